// A HIP runtime without a GPU, for tests of the library's host code: device
// memory is host memory, copies are done at once, and a kernel launch does
// nothing but log its name, except for the few kernels whose results the host
// reads back.  Loaded with global symbols before libdpa4c.so, it stands in for
// libamdhip64.  The log holds, in order, what was queued ("launch", "copy"),
// waited for ("sync"), allocated and refused.
//
// The edge kernels' buffers are checked at every launch: an address that is
// not inside a live allocation (or a device variable) counts as bad.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <sstream>
#include <string>

#include "../paper_2608_19041_amd/csrc/common.h"
#include "../paper_2608_19041_amd/csrc/compact.h"

namespace {

std::map<char*, size_t> g_live;                  // hipMalloc
std::map<char*, size_t> g_vars;                  // device variables
std::map<const void*, std::pair<char*, size_t>> g_var_of;
std::map<const void*, std::string> g_name;       // kernels
std::ostringstream g_log;
std::string g_log_text;
size_t g_refuse_from = SIZE_MAX, g_free = size_t(200) << 30;
int g_refuse_after = 0, g_bad = 0;
hipError_t g_last = hipSuccess;
struct { dim3 grid, block; size_t shm; hipStream_t st; } g_cfg;

bool inside(const std::map<char*, size_t>& m, const void* p) {
  char* q = static_cast<char*>(const_cast<void*>(p));
  auto it = m.upper_bound(q);
  if (it == m.begin()) return false;
  --it;
  return q < it->first + it->second;
}
// M: allocated, V: device variable, 0: null, ?: neither
char region(const void* p) {
  return !p ? '0' : inside(g_live, p) ? 'M' : inside(g_vars, p) ? 'V' : '?';
}
void need(const char* kernel, const char* what, const void* p) {
  const char r = region(p);
  if (r == 'M' || r == 'V') return;
  ++g_bad;
  g_log << "bad " << kernel << " " << what << " " << r << "\n";
}
template <class T>
T arg(void** a, int k) { return *static_cast<T*>(a[k]); }

// the first template flag of an edge kernel: folded tables
bool folded(const std::string& name) { return name[name.find("Lb") + 2] == '1'; }

}  // namespace

extern "C" {

// refuses requests of ``bytes`` or more (0: none) once ``after`` of them were granted
void fake_refuse_from(size_t bytes, int after) {
  g_refuse_from = bytes ? bytes : SIZE_MAX;
  g_refuse_after = after;
}
void fake_free_bytes(size_t bytes) { g_free = bytes; }
int fake_bad() { return g_bad; }
const char* fake_log() {
  g_log_text = g_log.str();
  g_log.str("");
  return g_log_text.c_str();
}

hipError_t hipMalloc(void** p, size_t n) {
  if (n >= g_refuse_from && g_refuse_after-- <= 0) {
    g_log << "refused " << n << "\n";
    return g_last = hipErrorOutOfMemory;
  }
  char* q = static_cast<char*>(calloc(n, 1));
  g_live[q] = n;
  g_log << "malloc " << n << "\n";
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  g_log << "free " << g_live[static_cast<char*>(p)] << "\n";
  g_live.erase(static_cast<char*>(p));
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = g_free; *t = size_t(288) << 30; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  g_log << "copy " << n << "\n";
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t) {
  return hipSuccess;   // of the stage checks only
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  g_log << "memset " << n << "\n";
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { g_log << "sync\n"; return hipSuccess; }
hipError_t hipDeviceSynchronize() { g_log << "sync\n"; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "an error of the stand-in runtime"; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  auto& v = g_var_of[symbol];
  if (!v.first) {
    v.first = static_cast<char*>(calloc(v.second, 1));
    g_vars[v.first] = v.second;
  }
  *p = v.first;
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  g_name[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t bytes, int, int) {
  g_var_of[var] = {nullptr, bytes};
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t st) {
  g_cfg = {g, b, shm, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, hipStream_t* st) {
  *g = g_cfg.grid; *b = g_cfg.block; *shm = g_cfg.shm; *st = g_cfg.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** a, size_t, hipStream_t) {
  using dpa4c::CompactArgs;
  using dpa4c::ModelDev;
  const std::string& name = g_name[f];
  auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
  g_log << "launch " << name;
  if (is("15backward_kernel") || is("14forward_kernel")) {
    const bool fw = is("14forward_kernel");
    const char* k = fw ? "forward" : "backward";
    const ModelDev md = arg<ModelDev>(a, 0);
    g_log << (folded(name) ? " folded\n" : " separable\n");
    if (folded(name)) need(k, "tables", md.ftab);
    need(k, "species", arg<void*>(a, 2));
    need(k, "rows", arg<void*>(a, 3));
    if (fw) {
      const CompactArgs ca = arg<CompactArgs>(a, 4);
      need(k, "list", ca.nbr_j);
      need(k, "shifts", ca.nbr_shift);
      need(k, "counts", ca.ecount);
      need(k, "edges", ca.edge);
      need(k, "places", ca.cskin);
      need(k, "node state", arg<void*>(a, 5));
    } else {
      need(k, "counts", arg<void*>(a, 4));
      need(k, "edges", arg<void*>(a, 5));
      need(k, "places", arg<void*>(a, 6));
      need(k, "gradient", arg<void*>(a, 7));
    }
  } else if (is("18row_readout_kernel")) {
    g_log << " rows " << region(arg<void*>(a, 5)) << region(arg<void*>(a, 6)) << " atoms "
          << arg<int64_t>(a, 2) << "\n";
  } else if (is("12chain_kernel")) {
    g_log << " rows " << region(arg<void*>(a, 3)) << region(arg<void*>(a, 4)) << "\n";
  } else if (is("14row_vjp_kernel")) {
    g_log << " rows " << region(arg<void*>(a, 3)) << "\n";
  } else {
    g_log << "\n";
  }
  if (is("18list_finish_kernel")) {   // the species present and a symmetric list
    const int32_t* species = arg<const int32_t*>(a, 2);
    uint32_t* host = arg<uint32_t*>(a, 8);
    memset(host, 0, 16);
    for (int64_t i = 0; i < arg<int64_t>(a, 3); ++i) host[species[i] >> 5] |= 1u << (species[i] & 31);
    if (const int64_t* size = arg<const int64_t*>(a, 7)) {
      const int64_t h[2] = {*size, *size / 2};
      memcpy(host + 4, h, sizeof(h));
    }
  } else if (is("15scan_one_kernelIl")) {   // a count of two neighbours for each atom
    struct Report { int64_t *flags, *host; };
    const Report r = arg<Report>(a, 3);
    const int64_t n = arg<int64_t>(a, 1);
    for (int64_t i = 0; i <= n; ++i) arg<int64_t*>(a, 2)[i] = 2 * i;
    if (r.flags) {
      r.host[0] = 2 * n;
      r.host[1] = r.flags[0];
      r.host[2] = 2;
    }
  } else if (is("18batch_start_kernel")) {   // no violation
    int64_t* flags = arg<int64_t*>(a, 8);
    flags[4] = INT64_MAX;
    flags[5] = 0;
  }
  return hipSuccess;
}

}  // extern "C"
