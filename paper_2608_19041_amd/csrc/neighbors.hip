// Cell-list neighbour search and the reverse index of a skin list, Methods
// Eq. (neighbor-set), integer arithmetic only.
//
// Positions are mapped to fixed point Q(x) = rint(x * 2^20) (int64) and the
// membership test |Q(r_j) + sum_b n_b Q(h_b) - Q(r_i)|^2 < Q(r)^2 is exact, so
// every list built here is a deterministic function of the float64 positions.
// Rows come out in canonical order (ascending j, then n_x, n_y, n_z).
//
// Binning: positions are wrapped into the cell by integer multiples of the
// quantised lattice vectors, which keeps the test exact.  A diagonal cell is
// binned in integers; a triclinic cell by fractional coordinates in float64,
// which only decides the candidate set: its stencil reach carries a 1e-6 A
// margin, far above the rounding of the fractional coordinates, so every
// pair within the radius is visited and the integer test decides.
//
// Bins are about half the radius wide (reach 2), so a centre's stencil
// covers ~15.6 r^3 instead of 27 r^3 with radius-wide bins, of which a diagonal
// cell visits the bins that the sphere touches, 10.5 r^3.  After binning,
// each atom's fixed-point position and index are copied into a record in bin
// order, so the atoms of consecutive bins along the third axis are one
// contiguous run: the stencil of a centre is a few dozen such runs, which a
// wave reads with coalesced loads as one list of candidates, 64 at a time.
//
// Work mapping: one 64-lane wavefront per centre atom, waves striding over
// centres.  The count kernel counts a row; the fill kernel collects the
// accepted keys (j, packed n) of a row in LDS and writes each at its rank,
// the number of smaller keys in the row: canonical order without a sort
// network.  Rows longer than kMaxRow are ranked the same way from a global
// scratch the host provides once the count has shown them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "../../include/dpa4c.h"
#include "launch.h"

namespace dpa4c {

namespace {

constexpr int kBlock = 256;            // 4 waves
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxRow = 512;           // longest row the fill kernel ranks in LDS
constexpr int kRankBlock = 8;          // keys compared per step of the bucketed rank
constexpr int kMaxSeg = kWave;         // stencil runs a wave holds at once
constexpr int64_t kFlagCapacity = 1, kFlagRowTooLong = 2, kFlagShift = 4, kFlagNonFinite = 8;
// Atoms up to which the four waves of a workgroup search a row: a row's
// searches are two rounds of a chain of eight loads for one wave.  A wave
// against a workgroup in us: 108 atoms 11.7, 5.9; 500 11.5, 6.4; 1,372 12.7, 8.9;
// 2,916 14.0, 15.5; 4,000 15.4, 20.2.
constexpr int64_t kSplitSearch = 2048;
constexpr int64_t kPresenceOne = 8192; // atoms whose species one block looks through
constexpr int kFlagMaxRow = 3;         // flags[3]: the longest row of the last count

__device__ inline int64_t floor_div(int64_t a, int64_t b) {
  int64_t q = a / b;
  return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q;
}

__device__ inline int64_t qfix(double x) { return static_cast<int64_t>(__builtin_rint(x * kQScale)); }

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

// exclusive prefix count of ``pred`` over the lanes below this one
__device__ inline int ballot_prefix(bool pred, uint64_t* mask_out) {
  uint64_t m = __ballot(pred);
  *mask_out = m;
  return __popcll(m & ((uint64_t(1) << lane_id()) - 1));
}

__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The same for LDS alone: outstanding global loads and stores of the wave
// are not waited for.
__device__ inline void wave_local_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// the union of the threads' bitmasks over the block, to out[0..3]
__device__ inline void block_or(uint32_t (&m)[4], uint32_t* out) {
  __shared__ uint32_t sh[kWavesPerBlock][4];
  for (int off = 1; off < kWave; off <<= 1)
    for (int w = 0; w < 4; ++w) m[w] |= __shfl_xor(m[w], off);
  if (lane_id() == 0)
    for (int w = 0; w < 4; ++w) sh[threadIdx.x / kWave][w] = m[w];
  __syncthreads();
  if (threadIdx.x < 4) {
    uint32_t v = sh[0][threadIdx.x];
    for (int k = 1; k < kWavesPerBlock; ++k) v |= sh[k][threadIdx.x];
    out[threadIdx.x] = v;
  }
  __syncthreads();
}

// bitmask of the species among share ``b`` of ``nb`` of the atoms
__device__ inline void block_presence(const int32_t* __restrict__ species, int64_t n, int n_types1,
                                      int64_t b, int64_t nb, uint32_t* out) {
  uint32_t m[4] = {0u, 0u, 0u, 0u};
  for (int64_t i = b * kBlock + threadIdx.x; i < n; i += nb * kBlock) {
    int a = species[i];
    a = static_cast<unsigned>(a) < static_cast<unsigned>(n_types1) ? a : n_types1 - 1;
#pragma unroll
    for (int w = 0; w < 4; ++w) m[w] |= (a >> 5) == w ? 1u << (a & 31) : 0u;
  }
  block_or(m, out);
}

struct GridDev {
  int64_t qh[9];          // Q(h_b) in row b
  double inv[9];          // inverse lattice matrix (triclinic binning)
  int nc0, nc1, nc2;
  int re0, re1, re2;
  int64_t rq;
  double r0, r1, r2;      // 1 / nc0, 1 / nc1, 1 / nc2
  double r12, rn1;        // 1 / (nc1 nc2), 1 / (2 re1 + 1)
  double bpq0, bpq1, bpq2;   // bins per fixed-point unit (diagonal cells)
  float bw0, bw1, bw2;    // bin width over the radius (diagonal cells)
  int trim;               // runs are cut to the sphere (diagonal cells)
  int wide;               // differences to a candidate may need more than 31 bits
};

// floor(t / d) from the double inverse r = 1 / d: (t + 1/2) / d stays at least
// 1 / (2 d) away from an integer, and the product is off by 2^-52 of itself at
// most, so the floor is exact for all 32-bit t and d
__device__ inline int div_by(int t, double r) {
  return static_cast<int>(floor((t + 0.5) * r));
}

GridDev to_dev(const CellGrid& g) {
  GridDev d;
  for (int k = 0; k < 9; ++k) {
    d.qh[k] = g.qh[k];
    d.inv[k] = g.inv[k];
  }
  d.nc0 = g.nc[0];
  d.nc1 = g.nc[1];
  d.nc2 = g.nc[2];
  d.re0 = g.reach[0];
  d.re1 = g.reach[1];
  d.re2 = g.reach[2];
  d.rq = g.rq;
  d.r0 = 1.0 / d.nc0;
  d.r1 = 1.0 / d.nc1;
  d.r2 = 1.0 / d.nc2;
  d.r12 = 1.0 / (double(d.nc1) * d.nc2);
  d.rn1 = 1.0 / (2.0 * d.re1 + 1.0);
  const double bpq[3] = {d.nc0 / double(g.qh[0]), d.nc1 / double(g.qh[4]), d.nc2 / double(g.qh[8])};
  d.bpq0 = bpq[0];
  d.bpq1 = bpq[1];
  d.bpq2 = bpq[2];
  d.bw0 = static_cast<float>(1.0 / (bpq[0] * double(g.rq)));
  d.bw1 = static_cast<float>(1.0 / (bpq[1] * double(g.rq)));
  d.bw2 = static_cast<float>(1.0 / (bpq[2] * double(g.rq)));
  // the float arithmetic of the cut holds its margin of 10^-3 bins for any
  // reach of a few dozen bins
  d.trim = !g.tric && std::max({d.re0, d.re1, d.re2}) <= 64;
  // a candidate lies within reach + 1 bins of the centre along every axis
  // (and a margin far above the rounding of fractional coordinates)
  double most = 0.0;
  for (int k = 0; k < 3; ++k) {
    double span = kQScale;
    for (int b = 0; b < 3; ++b)
      span += (g.reach[b] + 1.0) / g.nc[b] * std::fabs(double(g.qh[3 * b + k]));
    most = std::max(most, span);
  }
  d.wide = most >= 1073741824.0;   // 2^30: three squares stay below 2^63
  return d;
}

// within (strictly) the fixed-point radius; no overflow: components are
// rejected before squaring
__device__ inline bool within(int64_t dx, int64_t dy, int64_t dz, int64_t rq) {
  if (dx >= rq || dx <= -rq || dy >= rq || dy <= -rq || dz >= rq || dz <= -rq) return false;
  return dx * dx + dy * dy + dz * dz < rq * rq;
}

// ---------------------------------------------------------------------------
// clears the bin counts and, when given, the eight flag words of a build
__global__ void __launch_bounds__(kBlock) build_zero_kernel(int32_t* __restrict__ p, int64_t n,
                                                            int64_t* __restrict__ flags) {
  int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (i < n) p[i] = 0;
  if (flags && i < 8) flags[i] = 0;
}

// qpos = the position wrapped into the cell, Q(x) - sum_b m_b Q(h_b);
// wrap = m; cell_of = its bin
template <bool TRIC>
__global__ void __launch_bounds__(kBlock) bin_kernel(const double* __restrict__ pos, int64_t n,
                                                     GridDev g, int64_t* __restrict__ qpos,
                                                     int32_t* __restrict__ wrap,
                                                     int32_t* __restrict__ cell_of,
                                                     int32_t* __restrict__ cell_cnt,
                                                     int64_t* __restrict__ flags) {
  int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (i >= n) return;
  const int nc[3] = {g.nc0, g.nc1, g.nc2};
  int c[3];
  bool bad = false;
  double x[3];
  for (int a = 0; a < 3; ++a) {
    x[a] = pos[3 * i + a];
    if (!isfinite(x[a]) || fabs(x[a]) > 1.0e12) {
      bad = true;
      x[a] = 0.0;
    }
  }
  if (!TRIC) {
    for (int a = 0; a < 3; ++a) {
      const int64_t L = g.qh[4 * a];
      int64_t q = qfix(x[a]);
      int64_t m = floor_div(q, L);
      int64_t qw = q - m * L;
      qpos[3 * i + a] = qw;
      wrap[3 * i + a] = static_cast<int32_t>(m);
      c[a] = static_cast<int>((qw * nc[a]) / L);
    }
  } else {
    int64_t m[3];
    double fw[3];
    for (int b = 0; b < 3; ++b) {
      const double f = x[0] * g.inv[b] + x[1] * g.inv[3 + b] + x[2] * g.inv[6 + b];
      const double fl = floor(f);
      m[b] = static_cast<int64_t>(fl);
      fw[b] = f - fl;
    }
    for (int a = 0; a < 3; ++a) {
      qpos[3 * i + a] = qfix(x[a]) - m[0] * g.qh[a] - m[1] * g.qh[3 + a] - m[2] * g.qh[6 + a];
      wrap[3 * i + a] = static_cast<int32_t>(m[a]);
      int cb = static_cast<int>(fw[a] * nc[a]);
      c[a] = cb < 0 ? 0 : (cb >= nc[a] ? nc[a] - 1 : cb);
    }
  }
  if (bad) atomicOr(reinterpret_cast<unsigned long long*>(flags), (unsigned long long)kFlagNonFinite);
  int cid = (c[0] * nc[1] + c[1]) * nc[2] + c[2];
  cell_of[i] = cid;
  atomicAdd(&cell_cnt[cid], 1);
}

// One candidate record per atom, in bin order: the low words of the wrapped
// fixed-point position and the atom index, read by one 16-byte load; the wrap
// counts of the same atoms follow in an array of their own, in the same order.
struct alignas(16) CellRec {
  int32_t q[3];
  int32_t j;
};
static_assert(sizeof(CellRec) == 16 && sizeof(int4) == 16, "record size");
constexpr size_t kRecBytes = sizeof(CellRec) + sizeof(int4);   // of one atom

// the atom's record at a free slot of its bin, taken by counting the bin down
// (slot order inside a bin does not matter: rows are ranked by key afterwards)
__global__ void __launch_bounds__(kBlock) place_kernel(int64_t n, const int32_t* __restrict__ cell_of,
                                                       const int64_t* __restrict__ qpos,
                                                       const int32_t* __restrict__ wrap,
                                                       const int32_t* __restrict__ start,
                                                       int32_t* __restrict__ left,
                                                       CellRec* __restrict__ rec) {
  int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (i >= n) return;
  int cid = cell_of[i];
  const int64_t at = start[cid] + (atomicSub(&left[cid], 1) - 1);
  CellRec r;
  r.q[0] = static_cast<int32_t>(qpos[3 * i]);
  r.q[1] = static_cast<int32_t>(qpos[3 * i + 1]);
  r.q[2] = static_cast<int32_t>(qpos[3 * i + 2]);
  r.j = static_cast<int32_t>(i);
  rec[at] = r;
  reinterpret_cast<int4*>(rec + n)[at] = make_int4(wrap[3 * i], wrap[3 * i + 1], wrap[3 * i + 2], 0);
}

// exclusive-to-inclusive prefix sum over the 64 lanes of a wave
__device__ inline int wave_inclusive_scan(int v) {
  const int lane = lane_id();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int t = __shfl_up(v, off);
    if (lane >= off) v += t;
  }
  return v;
}

// The stencil of one centre as runs of bins: a run is the bins of one
// (axis-0, axis-1) offset whose axis-2 bins are consecutive with one image
// index, so its atoms are one contiguous range of the bin-ordered records.
struct SegLds {
  int4 a[kMaxSeg];           // low words of the image displacement sum_b s_b Q(h_b) minus Q(r_i);
                             // record of candidate k of the centre's list minus k
  int4 s[kMaxSeg];           // image indices of the run
  int32_t vend[kMaxSeg];     // end of the run in the centre's list of candidates
  int32_t aux[kMaxSeg];      // for the ranking
};

// Visits every candidate (record, image) of the stencil of centre i and
// calls f(record, j, run, pred) on chunks of 64 (one per lane, pred false on
// idle lanes); pred is the exact membership test with the centre itself
// (j = i, n = 0: the one candidate at distance zero with its index) excluded.
// The image index of a pair is n = s - m_j + m_i with m the wrap counts of
// binning.  Wave-uniform control flow.
//
// The kernels around it are bound by their instructions, so: divisions go
// through inverses; in a diagonal cell each run is cut to the bins that the
// sphere reaches past the run's own distance along axes 0 and 1 (10.5 r^3 of
// candidates instead of 15.6 r^3); and a candidate is tested on 32-bit
// differences, which are exact where the host found that no candidate can be
// 2^30 units away, else on the 64-bit positions.  Count and fill of a million
// atoms within 7 A: 1.61 + 3.23 ms -> 0.98 + 2.33 ms.
template <bool TRIC, class Fn>
__device__ inline void for_stencil(const GridDev& g, int i, const int64_t* __restrict__ qpos,
                                   const int32_t* __restrict__ cell_of,
                                   const int32_t* __restrict__ start,
                                   const CellRec* __restrict__ rec, SegLds& sg, Fn&& f) {
  const int lane = lane_id();
  const int64_t qi0 = qpos[3 * int64_t(i)], qi1 = qpos[3 * int64_t(i) + 1],
                qi2 = qpos[3 * int64_t(i) + 2];
  const int cid_i = cell_of[i];
  const int ci0 = div_by(cid_i, g.r12);
  const int rem = cid_i - ci0 * (g.nc1 * g.nc2);
  const int ci1 = div_by(rem, g.r2);
  const int ci2 = rem - ci1 * g.nc2;
  const int lo2 = ci2 - g.re2, hi2 = ci2 + g.re2;
  const int s2lo = div_by(lo2, g.r2);
  const int nr = div_by(hi2, g.r2) - s2lo + 1;   // image runs along axis 2
  const int n1 = 2 * g.re1 + 1;
  const int nseg = (2 * g.re0 + 1) * n1 * nr;
  // the centre's place in its bin, in bins
  const float f0 = static_cast<float>(double(qi0) * g.bpq0 - ci0);
  const float f1 = static_cast<float>(double(qi1) * g.bpq1 - ci1);
  const float f2 = static_cast<float>(double(qi2) * g.bpq2 - ci2);
  // its distance to the bins o away, in bins, short of 10^-3 bins
  auto gap = [](int o, float f0) {
    const float d = o > 0 ? static_cast<float>(o) - f0 : f0 - static_cast<float>(o + 1);
    return o == 0 ? 0.0f : fmaxf(d - 1e-3f, 0.0f);
  };
  const int64_t rq2 = g.rq * g.rq;
  for (int sb = 0; sb < nseg; sb += kMaxSeg) {
    const int q = sb + lane;
    int len = 0, beg = 0;
    int4 at = make_int4(0, 0, 0, 0);
    if (q < nseg) {
      const int p = nr == 1 ? q : nr == 2 ? q >> 1 : q / nr, r = q - p * nr;
      const int p0 = div_by(p, g.rn1);
      const int o0 = p0 - g.re0, o1 = p - p0 * n1 - g.re1;
      const int t0 = ci0 + o0, t1 = ci1 + o1;
      const int s0 = div_by(t0, g.r0), s1 = div_by(t1, g.r1), s2 = s2lo + r;
      const int w0 = t0 - s0 * g.nc0, w1 = t1 - s1 * g.nc1;
      int lo = lo2, hi = hi2;
      if (!TRIC && g.trim) {
        const float gx = gap(o0, f0) * g.bw0, gy = gap(o1, f1) * g.bw1;
        const float h2 = 1.0f - gx * gx - gy * gy;
        const float h = __builtin_amdgcn_sqrtf(fmaxf(h2, 0.0f)) / g.bw2 + 2e-3f;
        lo = max(lo, ci2 + static_cast<int>(floorf(f2 - h)));
        hi = h2 < 0.0f ? lo - 1 : min(hi, ci2 + static_cast<int>(floorf(f2 + h)));
      }
      const int a = max(lo, s2 * g.nc2) - s2 * g.nc2;
      const int b = min(hi, s2 * g.nc2 + g.nc2 - 1) - s2 * g.nc2;
      if (a <= b) {
        const int base = (w0 * g.nc1 + w1) * g.nc2;
        beg = start[base + a];
        len = start[base + b + 1] - beg;
      }
      if (!TRIC) {
        at.x = static_cast<int>(s0 * g.qh[0] - qi0);
        at.y = static_cast<int>(s1 * g.qh[4] - qi1);
        at.z = static_cast<int>(s2 * g.qh[8] - qi2);
      } else {
        at.x = static_cast<int>(s0 * g.qh[0] + s1 * g.qh[3] + s2 * g.qh[6] - qi0);
        at.y = static_cast<int>(s0 * g.qh[1] + s1 * g.qh[4] + s2 * g.qh[7] - qi1);
        at.z = static_cast<int>(s0 * g.qh[2] + s1 * g.qh[5] + s2 * g.qh[8] - qi2);
      }
      sg.s[lane] = make_int4(s0, s1, s2, 0);
    }
    const int vend = wave_inclusive_scan(len);
    at.w = beg - (vend - len);
    sg.a[lane] = at;
    sg.vend[lane] = vend;
    const int total = __builtin_amdgcn_readlane(vend, kWave - 1);
    wave_local_sync();
    int seg = 0;   // the run of this lane's candidate (candidates advance, so does the run)
    for (int k0 = 0; k0 < total; k0 += kWave) {
      const int k = k0 + lane;
      bool pred = false;
      int32_t j = 0, slot = 0;
      if (k < total) {
        while (sg.vend[seg] <= k) ++seg;
        const int4 o = sg.a[seg];
        slot = o.w + k;
        const CellRec c = rec[slot];
        j = c.j;
        if (!g.wide) {
          const int dx = static_cast<int>(unsigned(c.q[0]) + unsigned(o.x));
          const int dy = static_cast<int>(unsigned(c.q[1]) + unsigned(o.y));
          const int dz = static_cast<int>(unsigned(c.q[2]) + unsigned(o.z));
          const int64_t d2 = int64_t(dx) * dx + int64_t(dy) * dy + int64_t(dz) * dz;
          pred = d2 < rq2 && !(d2 == 0 && j == i);
        } else {
          const int4 im = sg.s[seg];
          int64_t d[3];
          for (int x = 0; x < 3; ++x)
            d[x] = qpos[3 * int64_t(j) + x] + im.x * g.qh[x] + im.y * g.qh[3 + x] +
                   im.z * g.qh[6 + x] - qpos[3 * int64_t(i) + x];
          pred = within(d[0], d[1], d[2], g.rq) && !(j == i && im.x == 0 && im.y == 0 && im.z == 0);
        }
      }
      f(slot, j, seg, pred);
    }
    wave_local_sync();   // the next batch of runs overwrites the table
  }
}

template <bool TRIC>
__global__ void __launch_bounds__(kBlock) count_kernel(int64_t n, GridDev g,
                                                       const int64_t* __restrict__ qpos,
                                                       const int32_t* __restrict__ cell_of,
                                                       const int32_t* __restrict__ start,
                                                       const CellRec* __restrict__ rec,
                                                       int64_t* __restrict__ counts) {
  __shared__ SegLds segs[kWavesPerBlock];
  SegLds& sg = segs[threadIdx.x / kWave];
  const int64_t nwaves = int64_t(gridDim.x) * kWavesPerBlock;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (int64_t i = xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock + w; i < n; i += nwaves) {
    int64_t total = 0;
    for_stencil<TRIC>(g, static_cast<int>(i), qpos, cell_of, start, rec, sg,
                      [&](int, int, int, bool pred) { total += __popcll(__ballot(pred)); });
    if (lane_id() == 0) counts[i] = total;
  }
}

// ---------------------------------------------------------------------------
// Exclusive scan: out[0..n] with out[n] = total, in one block up to
// kScanOne elements and in three launches above.
constexpr int kScanPer = 8;
constexpr int kScanTile = kBlock * kScanPer;
constexpr int kScanOneThreads = 1024;
// one block takes 8,192 elements a turn, about 3 us each; three launches take
// about 12 us however few the elements
constexpr int64_t kScanOne = 4 * kScanOneThreads * kScanPer;

// What the scan of the row counts reports: the longest row goes to
// flags[kFlagMaxRow] (an atomic maximum per wave of the count kernel took
// 12 ns each, one after the other: 200 us of a build), and (total, flags[0],
// longest row) to three words of pinned host memory, read after the next
// synchronisation.
struct ScanReport {
  int64_t* flags;   // null: nothing is reported
  int64_t* host;
};

__device__ inline void scan_report(const ScanReport& r, int64_t total, int64_t most) {
  if (!r.flags) return;
  r.flags[kFlagMaxRow] = most;
  r.host[0] = total;
  r.host[1] = r.flags[0];
  r.host[2] = most;
}

__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t* sh, int64_t* total) {
  int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < kBlock; off <<= 1) {
    int64_t add = t >= off ? sh[t - off] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  int64_t incl = sh[t];
  *total = sh[kBlock - 1];
  __syncthreads();
  return incl - v;
}

__device__ inline int64_t block_max(int64_t v, int64_t* sh) {
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t o = __shfl_xor(v, off);
    v = o > v ? o : v;
  }
  if (lane_id() == 0) sh[threadIdx.x / kWave] = v;
  __syncthreads();
  v = sh[0];
  for (int k = 1; k < static_cast<int>(blockDim.x) / kWave; ++k) v = sh[k] > v ? sh[k] : v;
  __syncthreads();
  return v;
}

// block totals to partials[b] and block maxima to partials[gridDim.x + b]
template <class T>
__global__ void __launch_bounds__(kBlock) scan_partials_kernel(const T* __restrict__ in, int64_t n,
                                                               int64_t* __restrict__ partials) {
  __shared__ int64_t sh[kBlock];
  int64_t base = blockIdx.x * int64_t(kScanTile) + threadIdx.x * kScanPer;
  int64_t s = 0, most = 0;
  for (int k = 0; k < kScanPer; ++k)
    if (base + k < n) {
      const int64_t v = in[base + k];
      s += v;
      most = v > most ? v : most;
    }
  int64_t tot;
  block_exclusive_scan(s, sh, &tot);
  most = block_max(most, sh);
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = tot;
    partials[gridDim.x + blockIdx.x] = most;
  }
}

__global__ void __launch_bounds__(kBlock) scan_top_kernel(int64_t* __restrict__ partials,
                                                          int64_t nparts, ScanReport report) {
  __shared__ int64_t sh[kBlock];
  int64_t carry = 0, most = 0;
  for (int64_t b = 0; b < nparts; b += kBlock) {
    int64_t idx = b + threadIdx.x;
    int64_t v = idx < nparts ? partials[idx] : 0;
    if (idx < nparts && partials[nparts + idx] > most) most = partials[nparts + idx];
    int64_t tot;
    int64_t ex = block_exclusive_scan(v, sh, &tot);
    if (idx < nparts) partials[idx] = ex + carry;
    carry += tot;
  }
  most = block_max(most, sh);
  if (threadIdx.x == 0) scan_report(report, carry, most);
}

template <class T>
__global__ void __launch_bounds__(kBlock) scan_apply_kernel(const T* __restrict__ in, int64_t n,
                                                            const int64_t* __restrict__ partials,
                                                            T* __restrict__ out) {
  __shared__ int64_t sh[kBlock];
  int64_t base = blockIdx.x * int64_t(kScanTile) + threadIdx.x * kScanPer;
  int64_t v[kScanPer];
  int64_t s = 0;
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = base + k < n ? int64_t(in[base + k]) : 0;
    s += v[k];
  }
  int64_t tot;
  int64_t run = block_exclusive_scan(s, sh, &tot) + partials[blockIdx.x];
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) out[base + k] = static_cast<T>(run);
    run += v[k];
  }
  if (base <= n - 1 && n - 1 < base + kScanPer) out[n] = static_cast<T>(run);  // thread holding the last element
}

// the whole scan in one block
template <class T>
__global__ void __launch_bounds__(kScanOneThreads) scan_one_kernel(const T* __restrict__ in,
                                                                   int64_t n, T* __restrict__ out,
                                                                   ScanReport report) {
  constexpr int kWaves = kScanOneThreads / kWave;
  __shared__ int64_t sh[kWaves];
  const int lane = lane_id(), w = threadIdx.x / kWave;
  int64_t carry = 0, most = 0;
  for (int64_t first = 0; first < n; first += kScanOneThreads * kScanPer) {
    const int64_t base = first + threadIdx.x * kScanPer;
    int64_t v[kScanPer], s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = base + k < n ? int64_t(in[base + k]) : 0;
      s += v[k];
      most = v[k] > most ? v[k] : most;
    }
    int64_t incl = s;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int64_t o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    if (lane == kWave - 1) sh[w] = incl;
    __syncthreads();
    int64_t run = carry + incl - s, tot = 0;
    for (int k = 0; k < kWaves; ++k) {
      if (k < w) run += sh[k];
      tot += sh[k];
    }
    carry += tot;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (base + k < n) out[base + k] = static_cast<T>(run);
      run += v[k];
    }
  }
  if (report.flags) most = block_max(most, sh);
  if (threadIdx.x == 0) {
    out[n] = static_cast<T>(carry);
    scan_report(report, carry, most);
  }
}

// exclusive scan out[0..n] of in[0..n) with out[n] = the total (int32 or int64)
template <class T>
int exclusive_scan(const T* in, int64_t n, T* out, DevBuf& partials, const ScanReport& report,
                   hipStream_t st) {
  if (n <= kScanOne) {
    hipLaunchKernelGGL(scan_one_kernel<T>, dim3(1), dim3(kScanOneThreads), 0, st, in, n, out,
                       report);
    DPA4C_HIP_TRY(hipGetLastError());
    return 0;
  }
  int64_t nb = (n + kScanTile - 1) / kScanTile;
  DPA4C_TRY(partials.ensure(2 * sizeof(int64_t) * nb));
  hipLaunchKernelGGL(scan_partials_kernel<T>, dim3(nb), dim3(kBlock), 0, st, in, n,
                     partials.as<int64_t>());
  hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(kBlock), 0, st, partials.as<int64_t>(), nb,
                     report);
  hipLaunchKernelGGL(scan_apply_kernel<T>, dim3(nb), dim3(kBlock), 0, st, in, n,
                     partials.as<int64_t>(), out);
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

// ---------------------------------------------------------------------------
// Canonical key of a list entry: rows are sorted by it.
__device__ inline int64_t entry_key(int32_t j, int32_t sh) {
  return (int64_t(j) << 24) | int64_t(sh & 0xFFFFFF);
}

// Writes the keys kb[0, len) of a row at their ranks, the number of smaller
// keys in the row (keys of a row are distinct), PER keys per lane at a time
// against one broadcast read of every key; with ``jsamp`` also j of every
// entry at an absolute position 16 g, to jsamp[g].
template <int PER, class KB>
__device__ __forceinline__ void rank_row(int len, int64_t r0, KB* kb, int32_t* __restrict__ nbr_j,
                                         int32_t* __restrict__ nbr_shift,
                                         int32_t* __restrict__ jsamp) {
  const int lane = lane_id();
  for (int t0 = 0; t0 < len; t0 += kWave * PER) {
    int64_t mine[PER];
    int rank[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int t = t0 + lane + kWave * r;
      mine[r] = t < len ? kb[t] : INT64_MAX;
      rank[r] = 0;
    }
    for (int u = 0; u < len; ++u) {
      const int64_t ku = kb[u];
#pragma unroll
      for (int r = 0; r < PER; ++r) rank[r] += ku < mine[r] ? 1 : 0;
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int t = t0 + lane + kWave * r;
      if (t < len) {
        const int64_t at = r0 + rank[r];
        const int32_t j = static_cast<int32_t>(mine[r] >> 24);
        nbr_j[at] = j;
        nbr_shift[at] = static_cast<int32_t>(mine[r] & 0xFFFFFF);
        if (jsamp && (at & 15) == 0) jsamp[at >> 4] = j;
      }
    }
  }
}

typedef long long i64x2 __attribute__((ext_vector_type(2)));

// The same ranks for a row held in LDS, counted inside buckets: the keys
// are grouped by j into at most 64 buckets of one power-of-two width over
// the row's range of j, so a key's bucket never decreases as the key grows
// and its rank is the number of keys in lower buckets plus the number of
// smaller keys in its own bucket.  The keys are regrouped in place by bucket
// (in any order inside one); each lane then takes grouped keys and compares
// only with its bucket.  ``boff`` and ``bend`` are 64 ints of the wave's LDS;
// kb (16-byte aligned) has room for kRankBlock keys past the row.
template <int PER, class KB>
__device__ __forceinline__ void rank_row_lds(int len, int64_t r0, KB* kb, int32_t* boff,
                                             int32_t* bend, int32_t* __restrict__ nbr_j,
                                             int32_t* __restrict__ nbr_shift,
                                             int32_t* __restrict__ jsamp) {
  const int lane = lane_id();
  int64_t key[PER];
  int32_t jlo = INT32_MAX, jhi = INT32_MIN;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int t = lane + kWave * r;
    key[r] = t < len ? kb[t] : 0;
    if (t < len) {
      const int32_t j = static_cast<int32_t>(key[r] >> 24);
      jlo = j < jlo ? j : jlo;
      jhi = j > jhi ? j : jhi;
    }
  }
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) {
    const int32_t lo = __shfl_xor(jlo, off), hi = __shfl_xor(jhi, off);
    jlo = lo < jlo ? lo : jlo;
    jhi = hi > jhi ? hi : jhi;
  }
  jlo = __builtin_amdgcn_readfirstlane(jlo);
  jhi = __builtin_amdgcn_readfirstlane(jhi);
  // width 2^sh with (jhi - jlo) >> sh < 64
  const uint32_t span = static_cast<uint32_t>(jhi - jlo);
  const int sh = span < 64u ? 0 : 26 - __clz(span);
  auto bucket = [&](int64_t k) {
    return static_cast<int>(static_cast<uint32_t>(static_cast<int32_t>(k >> 24) - jlo) >> sh);
  };
  boff[lane] = 0;
  wave_local_sync();
  int bk[PER], slot[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    bk[r] = 0;
    slot[r] = 0;
    if (lane + kWave * r < len) {
      bk[r] = bucket(key[r]);
      slot[r] = atomicAdd(&boff[bk[r]], 1);
    }
  }
  wave_local_sync();
  const int cnt = boff[lane];
  const int incl = wave_inclusive_scan(cnt);
  wave_local_sync();
  boff[lane] = incl - cnt;
  bend[lane] = incl;
  wave_local_sync();
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (lane + kWave * r < len) kb[boff[bk[r]] + slot[r]] = key[r];
  if (lane < kRankBlock) kb[len + lane] = INT64_MAX;   // sentinels past the row
  wave_local_sync();
  // Every key before a bucket is smaller than the bucket's keys and every
  // key after it larger (or a sentinel), so a key's rank is counted over
  // whole aligned blocks of kRankBlock keys around its bucket.
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int t = lane + kWave * r;
    if (t < len) {
      const int64_t k = kb[t];
      const int b = bucket(k);
      const int lo = boff[b] & ~(kRankBlock - 1), hi = bend[b];
      int rank = lo;
      for (int u = lo; u < hi; u += kRankBlock) {
        const i64x2* q = reinterpret_cast<const i64x2*>(kb + u);
#pragma unroll
        for (int v = 0; v < kRankBlock / 2; ++v) {
          const i64x2 x = q[v];
          rank += (x.x < k ? 1 : 0) + (x.y < k ? 1 : 0);
        }
      }
      const int64_t at = r0 + rank;
      const int32_t j = static_cast<int32_t>(k >> 24);
      nbr_j[at] = j;
      nbr_shift[at] = static_cast<int32_t>(k & 0xFFFFFF);
      if (jsamp && (at & 15) == 0) jsamp[at >> 4] = j;
    }
  }
}

// One row: the accepted keys into kb[0, len) in candidate order, then
// each written at its rank.  ``kb`` is the wave's LDS row (LDS_ROW) or, for
// a row longer than kMaxRow, a global scratch row (inlined for each, so LDS
// rows use LDS instructions).
template <bool TRIC, bool LDS_ROW, class KB>
__device__ __forceinline__ void fill_row(const GridDev& g, int64_t n, int64_t i, int64_t r0, int len, KB* kb,
                                         const int64_t* __restrict__ qpos,
                                         const int32_t* __restrict__ wrap,
                                         const int32_t* __restrict__ cell_of,
                                         const int32_t* __restrict__ start,
                                         const CellRec* __restrict__ rec, SegLds& sg,
                                         int32_t* __restrict__ nbr_j,
                                         int32_t* __restrict__ nbr_shift,
                                         int32_t* __restrict__ jsamp, int64_t* __restrict__ flags) {
  const int mi0 = wrap[3 * i], mi1 = wrap[3 * i + 1], mi2 = wrap[3 * i + 2];
  int fill = 0;
  bool shift_bad = false;
  const int4* mj_all = reinterpret_cast<const int4*>(rec + n);
  for_stencil<TRIC>(g, static_cast<int>(i), qpos, cell_of, start, rec, sg,
                    [&](int slot_j, int32_t j, int seg, bool pred) {
    uint64_t m;
    const int pre = ballot_prefix(pred, &m);
    if (pred) {
      const int4 im = sg.s[seg], mj = mj_all[slot_j];
      const int nx = im.x - mj.x + mi0;
      const int ny = im.y - mj.y + mi1;
      const int nz = im.z - mj.z + mi2;
      if (nx < -127 || nx > 127 || ny < -127 || ny > 127 || nz < -127 || nz > 127) shift_bad = true;
      const int slot = fill + pre;
      if (slot < len) kb[slot] = entry_key(j, pack_shift(nx, ny, nz));
    }
    fill += __popcll(m);
  });
  if (shift_bad)
    atomicOr(reinterpret_cast<unsigned long long*>(flags), (unsigned long long)kFlagShift);
  if constexpr (LDS_ROW) {
    wave_local_sync();
    if (len <= kWave) rank_row<1>(len, r0, kb, nbr_j, nbr_shift, jsamp);
    else if (len <= 2 * kWave) rank_row_lds<2>(len, r0, kb, sg.aux, sg.vend, nbr_j, nbr_shift, jsamp);
    else if (len <= 4 * kWave) rank_row_lds<4>(len, r0, kb, sg.aux, sg.vend, nbr_j, nbr_shift, jsamp);
    else rank_row_lds<8>(len, r0, kb, sg.aux, sg.vend, nbr_j, nbr_shift, jsamp);
    wave_local_sync();   // the row's keys are read before the next row overwrites them
  } else {
    wave_lds_sync();     // the keys are global memory here: the stores are waited for
    if (len <= kWave) rank_row<1>(len, r0, kb, nbr_j, nbr_shift, jsamp);
    else if (len <= 2 * kWave) rank_row<2>(len, r0, kb, nbr_j, nbr_shift, jsamp);
    else if (len <= 4 * kWave) rank_row<4>(len, r0, kb, nbr_j, nbr_shift, jsamp);
    else rank_row<8>(len, r0, kb, nbr_j, nbr_shift, jsamp);
    wave_lds_sync();
  }
}

// Rows of the skin list: the accepted candidates of centre i as keys
// (j, packed n), each written at its rank in the row, so rows come out in
// canonical order.  With ``jsamp`` the neighbour index of every entry at an
// absolute position 16 g also goes to jsamp[g], for the reverse search.
// Rows longer than kMaxRow collect their keys in long_keys[row_ptr[i] ...]
// instead of LDS (the host passes it when the count found such rows;
// without it they are flagged).
template <bool TRIC>
__global__ void __launch_bounds__(kBlock) fill_kernel(int64_t n, GridDev g,
                                                      const int64_t* __restrict__ qpos,
                                                      const int32_t* __restrict__ wrap,
                                                      const int32_t* __restrict__ cell_of,
                                                      const int32_t* __restrict__ start,
                                                      const CellRec* __restrict__ rec,
                                                      const int64_t* __restrict__ row_ptr,
                                                      int32_t* __restrict__ nbr_j,
                                                      int32_t* __restrict__ nbr_shift, int64_t cap,
                                                      int32_t* __restrict__ jsamp,
                                                      int64_t* __restrict__ long_keys,
                                                      int64_t* __restrict__ flags) {
  __shared__ SegLds segs[kWavesPerBlock];
  __shared__ alignas(16) int64_t keys_all[kWavesPerBlock][kMaxRow + kRankBlock];
  if (row_ptr[n] > cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      atomicOr(reinterpret_cast<unsigned long long*>(flags), (unsigned long long)kFlagCapacity);
      atomicMax(reinterpret_cast<unsigned long long*>(flags + 2), (unsigned long long)row_ptr[n]);
    }
    return;
  }
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  SegLds& sg = segs[w];
  const int64_t nwaves = int64_t(gridDim.x) * kWavesPerBlock;
  for (int64_t i = xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock + w; i < n; i += nwaves) {
    const int64_t r0 = row_ptr[i];
    const int len = static_cast<int>(row_ptr[i + 1] - r0);
    if (len <= kMaxRow) {
      fill_row<TRIC, true>(g, n, i, r0, len, keys_all[w], qpos, wrap, cell_of, start, rec, sg, nbr_j,
                     nbr_shift, jsamp, flags);
    } else if (long_keys) {
      fill_row<TRIC, false>(g, n, i, r0, len, long_keys + r0, qpos, wrap, cell_of, start, rec, sg, nbr_j,
                     nbr_shift, jsamp, flags);
    } else if (lane_id() == 0) {
      atomicOr(reinterpret_cast<unsigned long long*>(flags), (unsigned long long)kFlagRowTooLong);
    }
  }
}

// ---------------------------------------------------------------------------
// What the reverse search and the evaluation need before they start: rev =
// -1 everywhere, with ``jsamp`` the neighbour index at every 16th position
// of the list, and with ``species`` the bitmask of the species present among
// the atoms of each of the first ``nmask`` blocks' shares.
__global__ void __launch_bounds__(kBlock) list_prep_kernel(const int64_t* __restrict__ row_ptr,
                                                           int64_t n,
                                                           const int32_t* __restrict__ nbr_j,
                                                           int64_t cap, int32_t* __restrict__ jsamp,
                                                           int64_t* __restrict__ rev,
                                                           const int32_t* __restrict__ species,
                                                           int n_types1,
                                                           uint32_t* __restrict__ masks, int nmask) {
  const int64_t t0 = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  const int64_t stride = int64_t(gridDim.x) * kBlock;
  for (int64_t i = t0; i < cap; i += stride) rev[i] = -1;
  if (jsamp) {
    int64_t total = row_ptr[n];
    total = total < cap ? (total < 0 ? 0 : total) : cap;
    for (int64_t g = t0; 16 * g < total; g += stride) jsamp[g] = nbr_j[16 * g];
  }
  if (species && static_cast<int>(blockIdx.x) < nmask)
    block_presence(species, n, n_types1, blockIdx.x, nmask, masks + 4 * blockIdx.x);
}

// The species and the list of a call, for the host: host[0..3] the bitmask of
// the species present (of ``nmask`` partial masks, or with none of all the
// atoms), and as int64 after it the list's size and the number of reverse
// pairs (the sum of ``npair`` partials).  One block.
__global__ void __launch_bounds__(kBlock) list_finish_kernel(const uint32_t* __restrict__ masks,
                                                             int nmask,
                                                             const int32_t* __restrict__ species,
                                                             int64_t n, int n_types1,
                                                             const unsigned long long* __restrict__ pairs,
                                                             int npair,
                                                             const int64_t* __restrict__ size,
                                                             uint32_t* __restrict__ host) {
  __shared__ uint32_t part[4];
  __shared__ unsigned long long sum[kWavesPerBlock];
  if (nmask > 0) {
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    for (int b = threadIdx.x; b < nmask; b += kBlock)
      for (int w = 0; w < 4; ++w) m[w] |= masks[4 * b + w];
    block_or(m, part);
  } else {
    block_presence(species, n, n_types1, 0, 1, part);
  }
  unsigned long long p = 0;
  for (int b = threadIdx.x; b < npair; b += kBlock) p += pairs[b];
  for (int off = 1; off < kWave; off <<= 1) p += __shfl_xor(p, off);
  if (lane_id() == 0) sum[threadIdx.x / kWave] = p;
  __syncthreads();
  if (threadIdx.x < 4) host[threadIdx.x] = part[threadIdx.x];
  if (threadIdx.x == 0 && size) {
    for (int k = 1; k < kWavesPerBlock; ++k) p += sum[k];
    int64_t* h = reinterpret_cast<int64_t*>(host + 4);
    h[0] = *size;
    h[1] = static_cast<int64_t>(p);
  }
}

__global__ void __launch_bounds__(kBlock) presence_kernel(const int32_t* __restrict__ species,
                                                          int64_t n, int n_types1,
                                                          uint32_t* __restrict__ masks) {
  block_presence(species, n, n_types1, blockIdx.x, gridDim.x, masks + 4 * blockIdx.x);
}

// A row outside [0, cap] (a malformed caller list) gets no reverse entries and
// is nobody's reverse row, like the compaction, which keeps nothing of it.
__device__ inline bool row_ok(int64_t b, int64_t e, int64_t cap) { return b >= 0 && e >= b && e <= cap; }

// The reverse search of entry s = (i -> j, n): the position of the entry
// (i, -n) of row j, written to rev[s], and s to rev of that entry (both
// positions in the whole list).  Row j is ordered by neighbour index,
// so the entries (i, m) of row j are consecutive and begin at the first
// entry with neighbour index >= i: the samples of row j (the neighbour
// index at every absolute position 16 g inside it) are bisected for the
// aligned block of 16 entries that holds it, that block is compared at once
// (four 16-byte loads with VEC, one load per entry without), and the entries
// (i, m) from there are matched on the image.
template <bool VEC>
__device__ inline bool reverse_search(int64_t n, int32_t i, int64_t s, int32_t j, int32_t sh,
                                      const int64_t* __restrict__ row_ptr,
                                      const int32_t* __restrict__ nbr_j,
                                      const int32_t* __restrict__ nbr_shift, int64_t cap,
                                      const int32_t* __restrict__ jsamp,
                                      int64_t* __restrict__ rev) {
  const int32_t want_sh = negate_shift(sh);
  if (j < 0 || j >= n) return false;
  const int64_t jb = row_ptr[j], je = row_ptr[j + 1];
  if (!row_ok(jb, je, cap) || je == jb) return false;
  const int64_t g0 = (jb + 15) >> 4, g1 = (je - 1) >> 4;   // samples inside the row
  int64_t l = g0;                                           // first sample >= i
  if (g0 <= g1) {
    int64_t h = g1 + 1;
    while (l < h) {
      const int64_t m = (l + h) >> 1;
      if (jsamp[m] < i) l = m + 1;
      else h = m;
    }
  }
  // the first entry >= i lies in [lo, hi), inside the aligned block [16 q, 16 q + 16)
  const int64_t lo = l > g0 ? 16 * (l - 1) : jb;
  const int64_t hi = l <= g1 ? 16 * l : je;
  const int64_t q16 = l > g0 ? 16 * (l - 1) : 16 * (g0 - 1);
  int64_t p = lo;
  if (VEC) {
    const int4* blk = reinterpret_cast<const int4*>(nbr_j + q16);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t t = q16 + 4 * v;
      if (t + 3 >= lo && t < hi) {
        const int4 x = blk[v];
        p += (t >= lo && t < hi && x.x < i) + (t + 1 >= lo && t + 1 < hi && x.y < i) +
             (t + 2 >= lo && t + 2 < hi && x.z < i) + (t + 3 >= lo && t + 3 < hi && x.w < i);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (lo + t < hi && nbr_j[lo + t] < i) ++p;
  }
  for (int64_t t = p; t < je && nbr_j[t] == i; ++t)
    if (nbr_shift[t] == want_sh) {
      rev[s] = t;
      rev[t] = s;
      return true;
    }
  return false;
}

// skin_rev[s] = position in the list of the reverse of entry s (i -> j, n),
// the entry (i, -n) of row j, or -1.  A symmetric list pairs every entry with its
// reverse, so only the canonical entry of a pair, the one with
// key(j, n) > key(i, -n) (that is j > i, or a periodic self image with the
// larger shift), searches and writes both indices.  One wave takes rows in
// turn and queues their canonical entries in LDS, so every search round
// runs 64 searches.  Entries whose partner is missing (a malformed caller
// list) keep the -1 of the fill before.  With ``paired`` each block writes
// the number of pairs it found to paired[block] (list_finish_kernel adds them
// up), so the caller can tell a symmetric list (2 x pairs = entries) from one
// that is not; one counter for all waves took 12 ns a wave, one after the
// other (13,718 atoms: 176 us of search, 20 without).  With ``order`` (the
// neighbour build's atom records in bin order) the rows are taken in that
// spatial order, so that centres searched close in time share their rows j
// in L2; the results do not depend on the order.  With ``parts`` > 1 a row is
// taken by that many waves, 64 entries each in turn.
template <bool VEC>
__global__ void __launch_bounds__(kBlock) skin_rev_kernel(int64_t n, const int64_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ nbr_j,
                                                          const int32_t* __restrict__ nbr_shift,
                                                          int64_t cap,
                                                          const int32_t* __restrict__ jsamp,
                                                          int64_t* __restrict__ rev,
                                                          unsigned long long* __restrict__ paired,
                                                          const CellRec* __restrict__ order,
                                                          int parts) {
  __shared__ int64_t qs_all[kWavesPerBlock][2 * kWave];
  __shared__ int32_t qi_all[kWavesPerBlock][2 * kWave];
  __shared__ int32_t qj_all[kWavesPerBlock][2 * kWave];   // (j, n) of each queued entry
  __shared__ int32_t qh_all[kWavesPerBlock][2 * kWave];
  const int w = threadIdx.x / kWave;
  int64_t* qs = qs_all[w];
  int32_t* qi = qi_all[w];
  int32_t* qj = qj_all[w];
  int32_t* qh = qh_all[w];
  const int64_t nwaves = int64_t(gridDim.x) * kWavesPerBlock;
  const int lane = lane_id();
  unsigned long long found = 0;
  int qn = 0;   // queued searches (wave-uniform)
  // runs the first ``count`` (<= 64) queued searches and moves the rest down
  auto run = [&](int count) {
    const bool hit = lane < count &&
                     reverse_search<VEC>(n, qi[lane], qs[lane], qj[lane], qh[lane], row_ptr, nbr_j,
                                         nbr_shift, cap,
                                         jsamp, rev);
    found += __popcll(__ballot(hit));
    const int rest = qn - count;
    int64_t ks = 0;
    int32_t ki = 0, kj = 0, kh = 0;
    if (lane < rest) {
      ks = qs[count + lane];
      ki = qi[count + lane];
      kj = qj[count + lane];
      kh = qh[count + lane];
    }
    wave_local_sync();
    if (lane < rest) {
      qs[lane] = ks;
      qi[lane] = ki;
      qj[lane] = kj;
      qh[lane] = kh;
    }
    wave_local_sync();
    qn = rest;
  };
  for (int64_t rp = xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock + w; rp < n * parts;
       rp += nwaves) {
    const int64_t r = parts == 1 ? rp : rp / parts;
    const int64_t i = order ? order[r].j : r;
    const int64_t b = row_ptr[i], e = row_ptr[i + 1];
    if (!row_ok(b, e, cap)) continue;
    for (int64_t s0 = b + (rp - r * parts) * kWave; s0 < e; s0 += parts * kWave) {
      const int64_t s = s0 + lane;
      bool canon = false;
      int32_t j = 0, sh = 0;
      if (s < e) {
        j = nbr_j[s];
        sh = nbr_shift[s];
        canon = entry_key(j, sh) > entry_key(static_cast<int32_t>(i), negate_shift(sh));
      }
      uint64_t m;
      const int pre = ballot_prefix(canon, &m);
      if (canon) {
        qs[qn + pre] = s;
        qi[qn + pre] = static_cast<int32_t>(i);
        qj[qn + pre] = j;
        qh[qn + pre] = sh;
      }
      qn += __popcll(m);
      wave_local_sync();
      if (qn >= kWave) run(kWave);
    }
  }
  if (qn > 0) run(qn);
  if (paired) {
    __shared__ unsigned long long sum[kWavesPerBlock];
    if (lane == 0) sum[w] = found;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 1; k < kWavesPerBlock; ++k) found += sum[k];
      paired[blockIdx.x] = found;
    }
  }
}

// per-axis minimum and maximum of the fixed-point positions (exact integer
// min/max, so independent of the order of the atomics); out = [min x, y, z,
// max x, y, z], initialised by the caller to (INT64_MAX, INT64_MIN)
__global__ void __launch_bounds__(kBlock) extent_kernel(const double* __restrict__ pos, int64_t n,
                                                        long long* __restrict__ out) {
  __shared__ long long sh[6][kWavesPerBlock];
  long long lo[3] = {INT64_MAX, INT64_MAX, INT64_MAX}, hi[3] = {INT64_MIN, INT64_MIN, INT64_MIN};
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock) {
    for (int a = 0; a < 3; ++a) {
      const double x = pos[3 * i + a];
      if (!isfinite(x) || fabs(x) > 1.0e12) continue;   // flagged by the build
      const long long q = qfix(x);
      lo[a] = q < lo[a] ? q : lo[a];
      hi[a] = q > hi[a] ? q : hi[a];
    }
  }
  for (int off = 1; off < kWave; off <<= 1)
    for (int a = 0; a < 3; ++a) {
      const long long l = __shfl_xor(lo[a], off), h = __shfl_xor(hi[a], off);
      lo[a] = l < lo[a] ? l : lo[a];
      hi[a] = h > hi[a] ? h : hi[a];
    }
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0)
    for (int a = 0; a < 3; ++a) {
      sh[a][w] = lo[a];
      sh[3 + a][w] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int a = threadIdx.x;
    long long v = sh[a][0];
    for (int k = 1; k < kWavesPerBlock; ++k) v = a < 3 ? (sh[a][k] < v ? sh[a][k] : v)
                                                       : (sh[a][k] > v ? sh[a][k] : v);
    if (a < 3) atomicMin(out + a, v);
    else atomicMax(out + a, v);
  }
}

__global__ void extent_init_kernel(long long* out) {
  if (threadIdx.x < 6) out[threadIdx.x] = threadIdx.x < 3 ? INT64_MAX : INT64_MIN;
}

__global__ void flag_out_kernel(const int64_t* __restrict__ flags, int64_t* __restrict__ host) {
  if (threadIdx.x == 0) *host = flags[0];
}

int waves_grid(int64_t n) {
  int64_t blocks = (n + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > 4096) blocks = 4096;
  return static_cast<int>(blocks < 1 ? 1 : blocks);
}

}  // namespace

int make_grid(const double cell[9], int64_t rq, CellGrid* g) {
  if (rq <= 0 || rq > int64_t(1000) * int64_t(kQScale)) {
    set_error("bad neighbour radius");
    return DPA4C_ERR_INVALID_ARG;
  }
  for (int k = 0; k < 9; ++k)
    if (!std::isfinite(cell[k]) || std::fabs(cell[k]) > 1.0e6) {
      set_error("cell entries must be finite and below 1e6 A");
      return DPA4C_ERR_INVALID_ARG;
    }
  g->rq = rq;
  g->ncell = 1;
  g->tric = 0;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      if (a != b && cell[3 * a + b] != 0.0) g->tric = 1;
  for (int k = 0; k < 9; ++k) {
    g->h[k] = cell[k];
    g->qh[k] = static_cast<int64_t>(std::rint(cell[k] * kQScale));
  }
  // inverse lattice matrix (rows of ``cell`` are the lattice vectors)
  const double* h = cell;
  const double det = h[0] * (h[4] * h[8] - h[5] * h[7]) - h[1] * (h[3] * h[8] - h[5] * h[6]) +
                     h[2] * (h[3] * h[7] - h[4] * h[6]);
  if (!g->tric) {
    for (int a = 0; a < 3; ++a)
      if (!(cell[4 * a] > 0)) {
        set_error("the diagonal of an orthorhombic cell must be positive");
        return DPA4C_ERR_INVALID_ARG;
      }
  }
  double vol = std::fabs(det);
  double hmax = 0.0;
  for (int k = 0; k < 9; ++k) hmax = std::max(hmax, std::fabs(cell[k]));
  if (!(vol > 1e-9 * hmax * hmax * hmax) || !(vol > 0)) {
    set_error("the cell is singular");
    return DPA4C_ERR_INVALID_ARG;
  }
  const double cof[9] = {h[4] * h[8] - h[5] * h[7], h[2] * h[7] - h[1] * h[8],
                         h[1] * h[5] - h[2] * h[4], h[5] * h[6] - h[3] * h[8],
                         h[0] * h[8] - h[2] * h[6], h[2] * h[3] - h[0] * h[5],
                         h[3] * h[7] - h[4] * h[6], h[1] * h[6] - h[0] * h[7],
                         h[0] * h[4] - h[1] * h[3]};
  for (int k = 0; k < 9; ++k) g->inv[k] = cof[k] / det;
  const double r = double(rq) / kQScale;
  // bins of about half the radius (sub = 2 per radius, stencil reach 2); a
  // grid of more than kMaxFineBins bins (a sparse system in a large cell)
  // falls back to radius-wide bins
  constexpr int64_t kMaxFineBins = int64_t(1) << 24;
  for (int sub = 2; sub >= 1; --sub) {
    g->ncell = 1;
    for (int a = 0; a < 3; ++a) {
      int64_t nc;
      if (!g->tric) {
        const int64_t L = g->qh[4 * a];
        nc = sub * L / g->rq;
        if (nc < 1) nc = 1;
        if (nc > 1024) nc = 1024;
        g->reach[a] = static_cast<int>((g->rq * nc + L - 1) / L);
      } else {
        // distance between the lattice planes of axis a: V / |h_b x h_c|
        const double* u = h + 3 * ((a + 1) % 3);
        const double* v = h + 3 * ((a + 2) % 3);
        const double cx = u[1] * v[2] - u[2] * v[1], cy = u[2] * v[0] - u[0] * v[2],
                     cz = u[0] * v[1] - u[1] * v[0];
        const double d = vol / std::sqrt(cx * cx + cy * cy + cz * cz);
        nc = static_cast<int64_t>(std::floor(sub * d / r));
        if (nc < 1) nc = 1;
        if (nc > 1024) nc = 1024;
        const double re = std::ceil((r + 1e-6) * double(nc) / d);
        if (re > 1024.0) {
          set_error("the cell is too thin for the neighbour radius");
          return DPA4C_ERR_UNSUPPORTED;
        }
        g->reach[a] = static_cast<int>(re);
      }
      g->nc[a] = static_cast<int>(nc);
      g->ncell *= nc;
    }
    if (g->ncell <= kMaxFineBins) break;
  }
  return 0;
}

int ensure_scratch(NeighborScratch& nb, int64_t n, const CellGrid& g) {
  DPA4C_TRY(nb.qpos.ensure(sizeof(int64_t) * 3 * n));
  DPA4C_TRY(nb.wrap.ensure(sizeof(int32_t) * 3 * n));
  DPA4C_TRY(nb.cell_of.ensure(sizeof(int32_t) * n));
  DPA4C_TRY(nb.cell_cnt.ensure(sizeof(int32_t) * g.ncell));
  DPA4C_TRY(nb.cell_start.ensure(sizeof(int32_t) * (g.ncell + 1)));
  DPA4C_TRY(nb.cell_rec.ensure(kRecBytes * n));
  DPA4C_TRY(nb.counts.ensure(sizeof(int64_t) * n));
  // the bin counts and the row counts are scanned with the same partials
  const int64_t most = std::max<int64_t>(n, g.ncell);
  DPA4C_TRY(nb.partials.ensure(2 * sizeof(int64_t) * size_t((most + kScanTile - 1) / kScanTile + 1)));
  return 0;
}

int build_skin_list(NeighborScratch& nb, const double* pos, int64_t n, const CellGrid& g,
                    int64_t* row_ptr, int64_t* flags, bool clear_flags, int64_t* host3,
                    hipStream_t st) {
  int rc = ensure_scratch(nb, n, g);
  if (rc) return rc;
  GridDev gd = to_dev(g);
  int blocks = static_cast<int>((n + kBlock - 1) / kBlock);
  int cblocks = static_cast<int>((g.ncell + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(build_zero_kernel, dim3(cblocks), dim3(kBlock), 0, st,
                     nb.cell_cnt.as<int32_t>(), g.ncell, clear_flags ? flags : nullptr);
  if (g.tric)
    hipLaunchKernelGGL(bin_kernel<true>, dim3(blocks), dim3(kBlock), 0, st, pos, n, gd,
                       nb.qpos.as<int64_t>(), nb.wrap.as<int32_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_cnt.as<int32_t>(), flags);
  else
    hipLaunchKernelGGL(bin_kernel<false>, dim3(blocks), dim3(kBlock), 0, st, pos, n, gd,
                       nb.qpos.as<int64_t>(), nb.wrap.as<int32_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_cnt.as<int32_t>(), flags);
  rc = exclusive_scan(nb.cell_cnt.as<int32_t>(), g.ncell, nb.cell_start.as<int32_t>(), nb.partials,
                      ScanReport{nullptr, nullptr}, st);
  if (rc) return rc;
  hipLaunchKernelGGL(place_kernel, dim3(blocks), dim3(kBlock), 0, st, n, nb.cell_of.as<int32_t>(),
                     nb.qpos.as<int64_t>(), nb.wrap.as<int32_t>(), nb.cell_start.as<int32_t>(),
                     nb.cell_cnt.as<int32_t>(), nb.cell_rec.as<CellRec>());
  if (g.tric)
    hipLaunchKernelGGL(count_kernel<true>, dim3(waves_grid(n)), dim3(kBlock), 0, st, n, gd,
                       nb.qpos.as<int64_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_start.as<int32_t>(), nb.cell_rec.as<CellRec>(),
                       nb.counts.as<int64_t>());
  else
    hipLaunchKernelGGL(count_kernel<false>, dim3(waves_grid(n)), dim3(kBlock), 0, st, n, gd,
                       nb.qpos.as<int64_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_start.as<int32_t>(), nb.cell_rec.as<CellRec>(),
                       nb.counts.as<int64_t>());
  DPA4C_HIP_TRY(hipGetLastError());
  return exclusive_scan(nb.counts.as<int64_t>(), n, row_ptr, nb.partials, ScanReport{flags, host3},
                        st);
}

int fill_skin_list(NeighborScratch& nb, int64_t n, const CellGrid& g, const int64_t* row_ptr,
                   int32_t* nbr_j, int32_t* nbr_shift, int64_t cap, int64_t* flags,
                   int64_t max_row, int32_t* jsamp, int64_t* host_flag, hipStream_t st) {
  GridDev gd = to_dev(g);
  int64_t* long_keys = nullptr;
  if (max_row > kMaxRow) {
    DPA4C_TRY(nb.long_keys.ensure(sizeof(int64_t) * size_t(cap < 1 ? 1 : cap)));
    long_keys = nb.long_keys.as<int64_t>();
  }
  if (g.tric)
    hipLaunchKernelGGL(fill_kernel<true>, dim3(waves_grid(n)), dim3(kBlock), 0, st, n, gd,
                       nb.qpos.as<int64_t>(), nb.wrap.as<int32_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_start.as<int32_t>(), nb.cell_rec.as<CellRec>(), row_ptr, nbr_j,
                       nbr_shift, cap, jsamp, long_keys, flags);
  else
    hipLaunchKernelGGL(fill_kernel<false>, dim3(waves_grid(n)), dim3(kBlock), 0, st, n, gd,
                       nb.qpos.as<int64_t>(), nb.wrap.as<int32_t>(), nb.cell_of.as<int32_t>(),
                       nb.cell_start.as<int32_t>(), nb.cell_rec.as<CellRec>(), row_ptr, nbr_j,
                       nbr_shift, cap, jsamp, long_keys, flags);
  if (host_flag)
    hipLaunchKernelGGL(flag_out_kernel, dim3(1), dim3(64), 0, st, flags, host_flag);
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

int position_extent(const double* pos, int64_t n, int64_t* dev6, int64_t* host6, hipStream_t st) {
  long long* d = reinterpret_cast<long long*>(dev6);
  hipLaunchKernelGGL(extent_init_kernel, dim3(1), dim3(64), 0, st, d);
  int64_t blocks = (n + kBlock - 1) / kBlock;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(extent_kernel, dim3(blocks), dim3(kBlock), 0, st, pos, n, d);
  DPA4C_HIP_TRY(hipGetLastError());
  DPA4C_HIP_TRY(hipMemcpyAsync(host6, dev6, 6 * sizeof(int64_t), hipMemcpyDeviceToHost, st));
  DPA4C_HIP_TRY(hipStreamSynchronize(st));
  return 0;
}

int launch_skin_rev(const int64_t* row_ptr, const int32_t* nbr_j, const int32_t* nbr_shift,
                    int64_t n, int64_t cap, int32_t* jsamp, bool jsamp_ready, int64_t* skin_rev,
                    const ListCheck* check, const NeighborScratch* order_of, hipStream_t st) {
  const CellRec* order = order_of ? order_of->cell_rec.as<CellRec>() : nullptr;
  if (n <= 0) return 0;
  int64_t sb = (cap + kBlock - 1) / kBlock;
  sb = sb < 1 ? 1 : (sb > 8192 ? 8192 : sb);
  // partial species masks only where one block would take long over the atoms
  int nmask = 0;
  if (check && n > kPresenceOne) {
    const int64_t want = std::min<int64_t>(256, (n + kBlock - 1) / kBlock);
    nmask = static_cast<int>(std::min(want, sb));
  }
  unsigned long long* pairs =
      check ? static_cast<unsigned long long*>(check->scratch) : nullptr;
  uint32_t* masks = nmask ? reinterpret_cast<uint32_t*>(pairs + 4096) : nullptr;
  hipLaunchKernelGGL(list_prep_kernel, dim3(static_cast<unsigned>(sb)), dim3(kBlock), 0, st,
                     row_ptr, n, nbr_j, cap, jsamp_ready ? nullptr : jsamp, skin_rev,
                     nmask ? check->species : nullptr, check ? check->n_types1 : 0, masks, nmask);
  // the block compare reads 16-byte groups of nbr_j: a list that is not
  // 16-byte aligned takes one load per entry
  const bool vec = (reinterpret_cast<uintptr_t>(nbr_j) & 15) == 0;
  const int parts = n <= kSplitSearch ? kWavesPerBlock : 1;
  const int grid = waves_grid(n * parts);
  if (vec)
    hipLaunchKernelGGL(skin_rev_kernel<true>, dim3(grid), dim3(kBlock), 0, st, n, row_ptr, nbr_j,
                       nbr_shift, cap, jsamp, skin_rev, pairs, order, parts);
  else
    hipLaunchKernelGGL(skin_rev_kernel<false>, dim3(grid), dim3(kBlock), 0, st, n, row_ptr, nbr_j,
                       nbr_shift, cap, jsamp, skin_rev, pairs, order, parts);
  if (check)
    hipLaunchKernelGGL(list_finish_kernel, dim3(1), dim3(kBlock), 0, st, masks, nmask,
                       check->species, n, check->n_types1, pairs, grid, row_ptr + n,
                       check->host);
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

int launch_presence(const int32_t* species, int64_t n, int n_types1, uint32_t* masks,
                    uint32_t* host, hipStream_t st) {
  const int nmask =
      n > kPresenceOne ? static_cast<int>(std::min<int64_t>(256, (n + kBlock - 1) / kBlock)) : 0;
  if (nmask)
    hipLaunchKernelGGL(presence_kernel, dim3(nmask), dim3(kBlock), 0, st, species, n, n_types1,
                       masks);
  hipLaunchKernelGGL(list_finish_kernel, dim3(1), dim3(kBlock), 0, st, masks, nmask, species, n,
                     n_types1, nullptr, 0, nullptr, host);
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace dpa4c
