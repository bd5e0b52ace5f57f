"""The library's host code against a stand-in HIP runtime (fake_hip.cpp): which
buffers reach the kernels after a refused allocation, what is still queued when
a call returns, and which memory a call works in.  No GPU: the scenarios run in
a process of their own, where the stand-in takes the place of libamdhip64.
"""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
OK, OOM = 0, -7   # DPA4C_ERR_OOM


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    from paper_2608_19041_amd import build
    out = str(tmp_path_factory.mktemp("hip") / "fake_hip.so")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", f"--offload-arch={build.ARCH}",
                    "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"),
                    "-o", out], check=True)
    return out


class Host:
    """The library on the stand-in runtime, called with plain addresses."""

    def __init__(self, runtime):
        self.rt = ctypes.CDLL(runtime, mode=ctypes.RTLD_GLOBAL)
        self.lib = ctypes.CDLL(os.path.join(ROOT, "paper_2608_19041_amd", "libdpa4c.so"))
        self.rt.fake_log.restype = ctypes.c_char_p
        self.lib.dpa4c_last_error.restype = ctypes.c_char_p

    def log(self):
        return self.rt.fake_log().decode().splitlines()

    def refuse_from(self, nbytes, after=0):
        self.rt.fake_refuse_from(ctypes.c_size_t(nbytes), after)

    def device(self, values):
        """Device memory with these values."""
        a = np.ascontiguousarray(values)
        p = ctypes.c_void_p()
        assert self.rt.hipMalloc(ctypes.byref(p), ctypes.c_size_t(max(a.nbytes, 1))) == 0
        ctypes.memmove(p, a.ctypes.data, a.nbytes)
        return p

    def create(self, name, **change):
        import dataclasses
        import synth
        spec, weights = synth.model_weights(name)
        blob = synth.pack_blob(dataclasses.replace(spec, **change), weights)
        h = ctypes.c_void_p()
        rc = self.lib.dpa4c_model_create(blob, ctypes.c_size_t(len(blob)), 0, ctypes.byref(h))
        return rc, h

    def system(self, species, pairs=None):
        n = len(species)
        pairs = 2 * n if pairs is None else pairs
        s = {"n": n, "pairs": pairs,
             "pos": self.device(np.zeros((n, 3))), "species": self.device(np.int32(species)),
             "rows": self.device(np.linspace(0, pairs, n + 1).astype(np.int64)),
             "j": self.device(np.zeros(pairs, np.int32)),
             "shift": self.device(np.zeros(pairs, np.int32)),
             "vel": self.device(np.zeros((n, 3))), "force": self.device(np.zeros((n, 3))),
             "e": self.device(np.zeros(n)), "etot": self.device(np.zeros(1)),
             "chain": self.device(np.zeros(6)), "out": self.device(np.zeros((64, 9))),
             "cell": (ctypes.c_double * 9)(30, 0, 0, 0, 30, 0, 0, 0, 30),
             "pbc": (ctypes.c_int * 3)(1, 1, 1)}
        return s

    def energy(self, model, s, call="compute_energy_forces"):
        return getattr(self.lib, call)(
            model, s["pos"], s["species"], ctypes.c_int64(s["n"]), s["cell"], s["pbc"],
            ctypes.c_double(6.0), s["rows"], s["j"], s["shift"], ctypes.c_int64(s["pairs"]), s["e"],
            s["force"], s["etot"], None)

    def md(self, model, s, steps, nvt=False):
        mass = (ctypes.c_double * 128)(*([10.0] * 128))
        d, i64 = ctypes.c_double, ctypes.c_int64
        rebuilds = i64()
        head = (model, s["pos"], s["vel"], s["species"], mass, i64(s["n"]), s["cell"], s["pbc"],
                d(6.0), d(1.0), d(1.0), steps, 0)
        if nvt:
            return self.lib.nvt_step(*head, d(300.0), d(100.0), 3, s["chain"], s["out"], s["out"],
                                     s["out"], s["out"], s["force"], ctypes.byref(rebuilds), None)
        return self.lib.verlet_step(*head, s["out"], s["out"], s["force"], ctypes.byref(rebuilds),
                                    None)


def refused_allocation_fails_one_call(h):
    """A call that ran out of memory is refused; the next one is not."""
    rc, m = h.create("full")
    assert rc == OK
    two, five = h.system([28, 12] * 20), h.system([28, 12, 26, 21, 77] * 8)
    assert h.energy(m, two) == OK
    h.refuse_from(100 << 20)
    assert h.energy(m, five) == OOM
    h.refuse_from(0)
    assert h.energy(m, two) == OK, h.lib.dpa4c_last_error()


def tables_after_a_refused_allocation(h):
    """Five species' tables do not fit; the two or three species of before still run."""
    for before in ([28, 12], [28, 12, 26]):
        rc, m = h.create("full")
        assert rc == OK
        few, five = h.system(before * 20), h.system([28, 12, 26, 21, 77] * 8)
        assert h.energy(m, few) == OK
        h.refuse_from(100 << 20)
        assert h.energy(m, five) == OOM
        h.refuse_from(0)
        h.log()
        assert h.energy(m, few) == OK
        log = h.log()
        assert any("15backward_kernel" in x and x.endswith(" folded") for x in log), "not folded"
        assert h.rt.fake_bad() == 0, [x for x in log if x.startswith("bad")]


def first_call_gives_nothing_back(h):
    """A free waits for the device and unmaps: the first call of a model grows its
    buffers, whatever its species, without giving one up."""
    for name in ("mini", "full"):
        for species in ([28], [28, 12], [28, 12, 26], [28, 12, 26, 21, 77]):
            rc, m = h.create(name)
            s = h.system(species * 20)
            h.log()
            assert rc == OK and h.energy(m, s) == OK
            log = h.log()
            assert not any(x.startswith("free") for x in log), (name, len(species))
            assert h.energy(m, s) == OK
            assert not any(x.startswith(("malloc", "free")) for x in h.log())


def stages_after_the_tables_went(h):
    """The stages of the last evaluation read its tables: once another set took them
    they are refused, not recomputed from the wrong tables."""
    rc, m = h.create("full")
    one, two = h.system([28] * 40), h.system([28, 12] * 20)
    five, many = h.system([28, 12, 26, 21, 77] * 8), h.system([28, 12, 26, 21, 77, 45, 7, 63] * 5)
    stages = lambda: h.lib.dpa4c_debug_stages(m, ctypes.c_int64(40), None, None, None, None)  # noqa: E731
    assert rc == OK
    for other in (one, many):
        assert h.energy(m, two) == OK and stages() == OK
        assert h.energy(m, two, "compute_energy_forces_noalloc") == OK and stages() == OK
        assert h.energy(m, other, "compute_energy_forces_noalloc") == OK
        assert stages() != OK
        assert h.energy(m, other) == OK and stages() == OK
    assert h.energy(m, one, "compute_energy_forces_noalloc") == OK
    assert stages() == OK   # eight species ran on the separable tables, which stay
    assert h.energy(m, two) == OK
    h.refuse_from(100 << 20)
    assert h.energy(m, five) == OOM
    assert stages() != OK


def list_after_a_refused_workspace(h):
    """The list of the last dynamics call lost its buffers to a larger evaluation."""
    rc, m = h.create("small")
    s, large = h.system([28] * 40), h.system([28] * 40, pairs=400000)
    assert rc == OK and h.md(m, s, 3) == OK
    h.refuse_from(4 << 20)
    assert h.energy(m, large) == OOM
    h.refuse_from(0)
    h.log()
    assert h.lib.dpa4c_debug_stages(m, ctypes.c_int64(40), None, None, None, None) != OK
    assert h.md(m, s, 3) == OK
    log = h.log()
    assert h.rt.fake_bad() == 0, [x for x in log if x.startswith("bad")]
    assert any("12count_kernel" in x for x in log), "the list was not built again"


def list_after_a_refused_larger_system(h):
    """The rows of the list went to a larger system, which was refused."""
    rc, m = h.create("small")
    s, large = h.system([28] * 40), h.system([28] * 200000)
    assert rc == OK and h.md(m, s, 3) == OK
    h.refuse_from(1 << 20)
    assert h.md(m, large, 3) == OOM
    h.refuse_from(0)
    h.log()
    assert h.md(m, s, 3) == OK
    assert any("12count_kernel" in x for x in h.log()), "the list was not built again"


def list_after_a_half_refused_list(h):
    """Of the two arrays of a larger list the second was refused."""
    rc, m = h.create("small")
    s, large = h.system([28] * 1000), h.system([28] * 10000)
    assert rc == OK and h.md(m, s, 3) == OK
    entries = 20000 + 20000 // 8 + 16 * 10000   # with the list's head room
    h.refuse_from(4 * entries, after=1)
    assert h.md(m, large, 3) == OOM
    h.refuse_from(0)
    assert h.md(m, s, 3) == OK
    log = h.log()
    assert h.rt.fake_bad() == 0, [x for x in log if x.startswith("bad")]


def creation_without_room_for_tables(h):
    """A model whose folded tables have no room yet runs on the separable ones."""
    tables = 4 * 4 * 3000 * (3 * 128 + 32)   # two species at full width
    h.refuse_from(tables, after=1)           # the parameter block is as large
    rc, m = h.create("full")
    assert rc == OK, h.lib.dpa4c_last_error()
    s = h.system([28, 12] * 20)
    assert h.energy(m, s, "compute_energy_forces_noalloc") == OK
    h.refuse_from(0)
    assert any("backward_kernel" in x and x.endswith(" separable") for x in h.log())
    assert h.energy(m, s) == OK
    assert any("backward_kernel" in x and x.endswith(" folded") for x in h.log())
    assert h.rt.fake_bad() == 0


def creation_reserves_only_tables_it_would_use(h):
    """At this spacing two species' tables are above the limit for any use."""
    rc, m = h.create("full", delta=1.2e-4)
    assert rc == OK
    tables = 4 * 4 * 50000 * (3 * 128 + 32)
    assert not any(x.startswith("malloc") and int(x.split()[1]) >= tables for x in h.log())


def refused_creation_keeps_no_memory(h):
    """A creation that ran out of memory gives back what it had taken."""
    for granted in (1, 2):   # the parameters; those and the split weights
        h.refuse_from(1 << 20, after=granted)
        rc, _ = h.create("full")
        assert rc == OOM
        log = h.log()
        assert any(x.startswith("malloc") for x in log)
        assert (sorted(x.split()[1] for x in log if x.startswith("malloc"))
                == sorted(x.split()[1] for x in log if x.startswith("free")))
    h.refuse_from(0)
    assert h.create("full")[0] == OK, h.lib.dpa4c_last_error()


def nothing_is_queued_after_the_last_wait(h):
    """A dynamics call has waited for all it queued, however it ended."""
    for nvt in (False, True):
        for steps in (0, 1, 2, 5, 30):
            rc, m = h.create("small")
            s = h.system([28] * 40)
            assert rc == OK and h.md(m, s, steps, nvt) == OK
            assert h.md(m, s, steps, nvt) == OK      # with the list carried over
            log = h.log()
            assert log[-1] == "sync", (nvt, steps, log[-2:])


def noalloc_works_outside_the_workspace(h):
    """The no-allocation call's rows are the device's own, and hold its atoms at once."""
    rc, m = h.create("full")
    s, many = h.system([28, 12] * 20), h.system([28, 12] * 6000)
    assert rc == OK and h.energy(m, s) == OK
    rows = lambda log: [x.split(" rows ")[1] for x in log if " rows " in x]  # noqa: E731
    assert rows(h.log()) == ["MM atoms 40", "MM", "M"]
    for x in (s, many):
        assert h.energy(m, x, "compute_energy_forces_noalloc") == OK, h.lib.dpa4c_last_error()
        log = h.log()
        assert rows(log) == [f"VV atoms {x['n']}", "VV", "V"], rows(log)
        assert not any(y.startswith(("malloc", "free", "memset")) for y in log)


SCENARIOS = [refused_allocation_fails_one_call, tables_after_a_refused_allocation,
             stages_after_the_tables_went, first_call_gives_nothing_back,
             list_after_a_refused_workspace, list_after_a_refused_larger_system,
             list_after_a_half_refused_list,
             creation_without_room_for_tables, creation_reserves_only_tables_it_would_use,
             refused_creation_keeps_no_memory,
             nothing_is_queued_after_the_last_wait, noalloc_works_outside_the_workspace]


@pytest.mark.parametrize("name", [f.__name__ for f in SCENARIOS])
def test_host_path(runtime, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, name],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    globals()[sys.argv[2]](Host(sys.argv[1]))
