// Pair-folded radial tables.
//
// For an ordered type pair (a, b) the amplitude of channel c is a function of
// rho alone (Eq. (amplitude)):
//     psi_c(rho) = gamma_c g_c(rho) + beta_c + sum_mu U_c,mu q_mu(rho).
// Quintic Hermite interpolation is linear in its knot data (value, first and
// second derivative at both ends), and a constant is reproduced exactly, so
// the interpolant of psi_c is gamma_c times the interpolant of g_c, plus
// beta_c, plus U times the interpolants of q (Supplementary Note "Quintic
// Hermite interpolation of the radial table").  Its normalised coefficients
// are that same linear combination of the tabulated ones.
//
// The channels c >= C1 enter degree zero alone, as chi psi_c, so their tables
// hold that product: its Taylor coefficients over an interval are those of psi
// convolved with those of the envelope at the knot.  The forward kernel then
// adds the interpolant as it is, and the backward kernel, which needs
// d(chi psi)/drho and no value, leaves c0 of these channels (7 of 8 at full
// width) in memory and takes 1,088 bytes an edge instead of 1,536.
//
// A row belongs to a knot and reaches half an interval to either side, since what
// a dropped or rounded coefficient c_n does to the value and the slope goes with
// |tau|^n and n |tau|^(n-1): |tau| <= 1/2 instead of tau < 1 halves the slope's
// error of c2 and takes that of c3 to a quarter, for the same bytes and
// operations.  Value, slope and curvature at a knot are those of the quintics on
// both sides; the cubic coefficient is the mean of theirs, which differ by c4.
// Forces of isolated pairs against 64 bits: 0.85 - 1.1 A 3.1 to 6.8e-6 of their
// norm before (rows from knot to knot, three models), 1.8 to 2.5e-6 now; 1.3 -
// 2 A 2.9 to 3.8e-6 before, 1.8 to 1.9e-6 now.
//
// Storage: c0 and c1 in float32, c2 and c3 as float16 scaled by fixed powers
// of two (one per coefficient, from a bound over every pair: |gamma| < 2 and
// |U| < 1 by their tanh forms, times the largest tabulated coefficient); c4
// and c5 are not stored.  With the normalised form c_n Delta^n the
// coefficients fall by about two orders of magnitude per power at
// Delta = 0.002 A, so the whole contribution of c4 and c5 together with the
// 2^-11 relative rounding of c2 and c3 stays below the float32 rounding of
// the value and below 2^-14 of the slope term (checked per model at set-up, for
// psi and for chi psi; a model that fails the check runs on the separable
// float32 tables), and a channel takes 12 bytes instead of 24.
//
// For the few species of an MD system the library keeps one such table per
// ordered pair present; the edge kernels then read one quintic per channel
// instead of a g quintic, R q quintics and the pair coefficients.  Systems
// with more than kMaxFoldTypes species, or whose folded tables would exceed
// kMaxFoldBytes, use the separable tables directly.  Five species at full
// width (128 channels, 3,000 rows at r_c = 6 A and Delta = 0.002 A) fold into
// 25 tables of 5.0 MB (125 MB, within the last-level cache); on the 5-species
// alloy the folded tables measured faster than the separable ones (backward
// 0.94 -> 0.70 ms at 31,250 atoms, when a folded channel still took 16 B),
// since every edge then reads one 12-byte entry per channel from one table
// instead of 24 B of g coefficients per channel plus the q rows and the pair
// coefficients.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "../../include/dpa4c.h"
#include "edge_math.h"
#include "launch.h"

namespace dpa4c {

namespace {

__global__ void fold_index_kernel(const int32_t* __restrict__ species, int64_t n, int n_types1,
                                  const int32_t* __restrict__ map, int32_t* __restrict__ fidx) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    fidx[i] = map[clamp_type(species[i], n_types1)];
}

struct FoldTypes {
  int t[kMaxFoldTypes];
};

// One block per (table row, folded type of the centre), thread = channel c: what
// does not depend on the pair, the coefficients of g and q around the knot and the
// envelope's, is formed once for the n_used pairs of a block.  For each pair anew,
// in 64 bits, it took the build of 25 tables at full width from 131 us (before chi
// psi and rows around knots) to 162; formed once 130 (five species of Mini 31, 40
// and 24, two of full width 27, 32 and 27).
__global__ void fold_build_kernel(const float* __restrict__ gtab, const float* __restrict__ qtab,
                                  const float* __restrict__ pair, FoldTypes used, int n_used,
                                  int n_types1, int C0, int R, int LPE, int intervals,
                                  double r_c, double delta, const float2 scale,
                                  float* __restrict__ ftab) {
  const int s = blockIdx.x;
  // the envelope at the row's knot, chi_n = chi^(n) Delta^n / n!:
  // chi = t^4 (1 + 4x + 10x^2 + 20x^3 + 35x^4), chi' = -280 x^4 t^3 / r_c
  // (a last knot past r_c, where no edge is: the same polynomials)
  const double h = delta / r_c, x = s * h, t = 1.0 - x;
  const double x2 = x * x, t2 = t * t;
  const double chi[4] = {
      t2 * t2 * (1.0 + x * (4.0 + x * (10.0 + x * (20.0 + x * 35.0)))),
      -280.0 * x2 * x2 * t2 * t * h,
      -140.0 * x2 * x * t2 * (4.0 * t - 3.0 * x) * h * h,
      -280.0 * x2 * t * (2.0 * t2 - 4.0 * x * t + x2) * h * h * h};
  // Around the knot the coefficients up to the third of one tabulated function
  // (coef(interval, power)): value, slope and curvature are those of both
  // intervals, the cubic coefficient is the mean of theirs; at either end of the
  // table those of the one interval there is (a Taylor shift from its end).
  auto around = [&](auto&& coef, double (&v)[4]) {
    if (s < intervals) {
      for (int q = 0; q < 4; ++q) v[q] = coef(s, q);
      if (s > 0)
        v[3] = 0.5 * (v[3] + coef(s - 1, 3) + 4.0 * coef(s - 1, 4) + 10.0 * coef(s - 1, 5));
    } else {
      double u[6];
      for (int q = 0; q < 6; ++q) u[q] = coef(s - 1, q);
      v[0] = u[0] + u[1] + u[2] + u[3] + u[4] + u[5];
      v[1] = u[1] + 2.0 * u[2] + 3.0 * u[3] + 4.0 * u[4] + 5.0 * u[5];
      v[2] = u[2] + 3.0 * u[3] + 6.0 * u[4] + 10.0 * u[5];
      v[3] = u[3] + 4.0 * u[4] + 10.0 * u[5];
    }
  };
  __shared__ double mode[kMaxModes][4];   // of the q functions, for all channels
  if (threadIdx.x < R) {
    double v[4];
    around([&](int i, int q) { return double(qtab[(size_t(i) * R + threadIdx.x) * 6 + q]); }, v);
    for (int q = 0; q < 4; ++q) mode[threadIdx.x][q] = v[q];
  }
  __syncthreads();
  const int PW = 2 + R, CPL = C0 / LPE;
  const float* pairs = pair + size_t(used.t[blockIdx.y]) * n_types1 * C0 * PW;
  for (int c = threadIdx.x; c < C0; c += blockDim.x) {
    const int k = c % LPE, j = c / LPE;
    const int at = fold_at(LPE, CPL, k, j);
    double g[4];
    around([&](int i, int q) { return double(gtab[((size_t(i) * CPL + j) * LPE + k) * 6 + q]); }, g);
    for (int b = 0; b < n_used; ++b) {
      const float* pc = pairs + ((size_t(used.t[b]) * CPL + j) * LPE + k) * PW;
      // row s of the pair, in the order the edge kernels read (load_fold_row)
      float* row = ftab + (size_t(blockIdx.y * n_used + b) * (intervals + 1) + s) * fold_pitch(C0, CPL);
      double v[4];
      for (int q = 0; q < 4; ++q) {
        v[q] = double(pc[0]) * g[q] + (q == 0 ? double(pc[1]) : 0.0);
        for (int mu = 0; mu < R; ++mu) v[q] += double(pc[2 + mu]) * mode[mu][q];
      }
      if (j > 0)   // times the envelope, from the highest power down
        for (int q = 3; q >= 0; --q) {
          double f = 0.0;
          for (int m = 0; m <= q; ++m) f += chi[m] * v[q - m];
          v[q] = f;
        }
      const float sc[2] = {scale.x, scale.y};
      uint16_t hb[2];
      for (int q = 0; q < 2; ++q)
        hb[q] = __builtin_bit_cast(uint16_t,
                                   static_cast<_Float16>(static_cast<float>(v[2 + q] * sc[q])));
      row[at] = static_cast<float>(v[0]);
      if (CPL > 2 && j == 0) row[3 * C0 + k] = static_cast<float>(v[0]);
      row[C0 + at] = static_cast<float>(v[1]);
      reinterpret_cast<uint32_t*>(row)[2 * C0 + at] = uint32_t(hb[0]) | (uint32_t(hb[1]) << 16);
    }
  }
}

int grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  return static_cast<int>(b < 4096 ? (b < 1 ? 1 : b) : 4096);
}

}  // namespace

int prepare_species(dpa4c_model* m, const uint32_t mask[4], const int32_t* species, int64_t n,
                    int32_t* fidx, bool may_alloc, bool* use_fold, hipStream_t st) {
  Workspace& w = m->ws;
  const int T1 = m->n_types + 1;
  *use_fold = false;
  if (n <= 0) return 0;
  // the type map and the pinned host words ([64, 64 + 4 T1): the type map) are
  // allocated with the model
  if (!w.fold_host || !w.fold_map.p) {
    set_error("prepare_species: the model's species buffers are missing");
    return DPA4C_ERR_INVALID_ARG;
  }
  const bool same = m->fold_n >= 0 && std::memcmp(mask, m->fold_types_mask, sizeof(m->fold_types_mask)) == 0;
  if (!same) {
    FoldTypes used{};
    int n_used = 0;
    std::vector<int32_t> map(T1, -1);
    for (int a = 0; a < T1; ++a)
      if (mask[a >> 5] >> (a & 31) & 1u) {
        if (n_used < kMaxFoldTypes) {
          used.t[n_used] = a;
          map[a] = n_used;
        }
        ++n_used;
      }
    const size_t need = fold_bytes(m->n_rows, m->C0, m->C[1], n_used);
    const bool folds = m->fold_allowed && n_used <= kMaxFoldTypes && need <= kMaxFoldBytes;
    if (folds && !may_alloc && need > std::max(w.ftab_first.bytes, w.ftab.bytes))
      return 0;        // this call only: separable tables, the folded state kept
    if (w.last_fidx) m->last_n = -1;   // its tables go: the stages cannot run again
    if (!folds) {
      std::memcpy(m->fold_types_mask, mask, sizeof(m->fold_types_mask));
      m->fold_n = 0;   // the separable tables are used
    } else {
      // no set has tables until these are built: a refused allocation has
      // already given the old ones back
      m->fold_n = -1;
      DevBuf& room = need <= w.ftab_first.bytes ? w.ftab_first : w.ftab;
      DPA4C_TRY(room.ensure(need));
      w.tables = room.as<float>();
      int32_t* hmap = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(w.fold_host) + 64);
      std::memcpy(hmap, map.data(), 4 * size_t(T1));
      DPA4C_HIP_TRY(hipMemcpyAsync(w.fold_map.p, hmap, 4 * size_t(T1), hipMemcpyHostToDevice, st));
      hipLaunchKernelGGL(fold_build_kernel, dim3(m->n_rows + 1, n_used),
                         dim3(m->C0 < 256 ? m->C0 : 256), 0, st, m->gtab, m->qtab, m->pair, used,
                         n_used, T1, m->C0, m->R, m->C[1], m->n_rows, m->r_c, m->delta,
                         make_float2(m->c_scale[0], m->c_scale[1]), w.tables);
      DPA4C_HIP_TRY(hipGetLastError());
      std::memcpy(m->fold_types_mask, mask, sizeof(m->fold_types_mask));
      m->fold_n = n_used;
    }
  }
  if (m->fold_n > 0) {
    hipLaunchKernelGGL(fold_index_kernel, dim3(grid_for(n)), dim3(256), 0, st, species, n, T1,
                       w.fold_map.as<int32_t>(), fidx);
    DPA4C_HIP_TRY(hipGetLastError());
    *use_fold = true;
  }
  return 0;
}

}  // namespace dpa4c
