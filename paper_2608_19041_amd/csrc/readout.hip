// The invariant readout (readout_row.h) as kernels of its own: node state in,
// calibrated descriptor out as the operand planes of the MLP (mlp_chain.hip),
// and dE/dD in, dE/d(node state) out.  Kept apart from the MLP, whose
// workgroups hold one CU each, the readouts run with as many atoms in flight
// as their descriptor rows in LDS allow.  Per 65,536 atoms at full width the
// readout takes 63 to 71 us and its VJP 72 to 76 us (degree four: 89 and 120 us),
// against 40 and 52 us for the bytes they move at the rate of a large copy; what bounds
// them is the chain of LDS reads and rotations of one atom, with three and two
// waves on a SIMD to hide it.
#include <hip/hip_runtime.h>

#include "../../include/dpa4c.h"
#include "launch.h"
#include "readout_row.h"

namespace dpa4c {

namespace {

constexpr int kThreads = 256;
constexpr int kRowAtoms = kThreads / kRow;   // atoms of a workgroup
// workgroups of a launch: each stages its tables once and strides over the
// atoms; about what runs at once
constexpr int64_t kRowGrid = 1024;
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// the lane's features of one atom
template <class P>
__device__ __forceinline__ void load_features(const float* y, const RowLane<P>& k, float (&y1)[3],
                                              float (&y2)[5], float (&y3)[P::L >= 3 ? 7 : 1],
                                              float (&y4)[P::L >= 4 ? 9 : 1]) {
#pragma unroll
  for (int m = 0; m < 3; ++m) y1[m] = y[P::Y1 + m * P::C1 + k.c];
#pragma unroll
  for (int m = 0; m < 5; ++m) y2[m] = y[P::Y2 + m * P::C2 + k.e];
  if constexpr (P::L >= 3) {
#pragma unroll
    for (int m = 0; m < 7; ++m) y3[m] = y[P::Y3 + m];
  }
  if constexpr (P::L >= 4) {
#pragma unroll
    for (int m = 0; m < 9; ++m) y4[m] = y[P::Y4 + m];
  }
}

template <class P, int KP>
__global__ void __launch_bounds__(kThreads, P::L >= 4 ? 2 : 3)
    row_readout_kernel(ModelDev md, MlpScales sc, int64_t n, const int32_t* __restrict__ species,
                       const float* __restrict__ node, float* __restrict__ desc,
                       float2* __restrict__ meta, float* __restrict__ desc_out) {
  __shared__ __align__(16) float rows[kRowAtoms][KP + 8];
  using T = RowTable<P>;
  __shared__ __align__(16) float tab[T::floats(T::kFwd)];
  const int ra = threadIdx.x / kRow;
  float* row = rows[ra];
  stage_table(tab, md.row_tab, T::kFwd, threadIdx.x, kThreads);
  RowLane<P> k;
  k.init();
  RowPlaces<P> at;
  at.init(k);
  __syncthreads();
  constexpr int kPieces = KP / 4, kEach = (kPieces + kRow - 1) / kRow;
  constexpr int kY0 = (P::C0 + kRow - 1) / kRow;
#pragma unroll 1
  for (int64_t g = blockIdx.x; g * kRowAtoms < n; g += gridDim.x) {
    // opaque: the tables are read from LDS for each atom, not kept in registers
    asm volatile("" : "+v"(k.l));
    const int64_t want = g * kRowAtoms + ra;
    const int64_t i = want < n ? want : n - 1;   // rows past n repeat the last atom, unstored
    const bool ok = want < n;
    const float* y = node + size_t(i) * P::NS;
    const float* x0 = md.type_embed + size_t(clamp_type(species[i], md.n_types1)) * P::C0;
    float y1[3], y2[5], y3[P::L >= 3 ? 7 : 1], y4[P::L >= 4 ? 9 : 1], y0[kY0], e0[kY0];
    load_features<P>(y, k, y1, y2, y3, y4);
#pragma unroll
    for (int q = 0; q < kY0; ++q) {
      const int t = k.l + q * kRow;
      y0[q] = t < P::C0 ? y[P::Y0 + t] : 0.0f;
      e0[q] = t < P::C0 ? x0[t] : 0.0f;
    }
    RowFwd<P> f;
    row_forward<P>(f, k, tab, y[0], y[1], y1, y2, y3, y4);
    row_descriptor<P>(f, k, at, row);
#pragma unroll
    for (int q = 0; q < kY0; ++q) {
      const int t = k.l + q * kRow;
      if (t < P::C0) {
        row[P::oX0 + t] = e0[q];
        row[P::oX + t] = y0[q] * f.i0;
      }
    }
    wave_sync();
    // calibration (Eq. (calibration)) in the descriptor's order, with the
    // row's norms
    float big = 0.0f, sq = 0.0f;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int t0 = (k.l + q * kRow) * 4;
      if (t0 < KP) {
        row_f4 x = *reinterpret_cast<const row_f4*>(row + t0);
        const row_f4 mu = *reinterpret_cast<const row_f4*>(md.mu + t0);
        const row_f4 is = *reinterpret_cast<const row_f4*>(md.inv_sigma + t0);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          x[w] = t0 + w < P::DOUT ? (x[w] - mu[w]) * is[w] : 0.0f;
          big = fmaxf(big, fabsf(x[w]));
          sq = fmaf(x[w], x[w], sq);
        }
        *reinterpret_cast<row_f4*>(row + t0) = x;
      }
    }
    big = row_max(big);
    sq = row_sum(sq);
    const int e = operand_exponent(big);
    const float up = __builtin_amdgcn_ldexpf(1.0f, e);
    wave_sync();
    if (ok) {
      _Float16* hi = reinterpret_cast<_Float16*>(desc + size_t(i) * KP);
#pragma unroll
      for (int q = 0; q < (KP / 8 + kRow - 1) / kRow; ++q) {
        const int t0 = (k.l + q * kRow) * 8;
        if (t0 < KP) {
          v8h a, b;
#pragma unroll
          for (int c = 0; c < 8; c += 4) {
            const row_f4 v = *reinterpret_cast<const row_f4*>(row + t0 + c);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const float x = v[w] * up;
              a[c + w] = static_cast<_Float16>(x);
              b[c + w] = static_cast<_Float16>(x - static_cast<float>(a[c + w]));
            }
          }
          *reinterpret_cast<v8h*>(hi + t0) = a;
          *reinterpret_cast<v8h*>(hi + KP + t0) = b;
        }
      }
      if (desc_out)
        for (int t = k.l; t < P::DOUT; t += kRow) desc_out[size_t(i) * P::DOUT + t] = row[t];
      if (k.l == 0)
        meta[i] = make_float2(__builtin_amdgcn_ldexpf(1.0f, -e),
                              fminf(big * sc.d_max, sqrtf(sq) * sc.d_norm) * 1.001f + sc.d_add);
    }
    wave_sync();   // the row is free for the next atom
  }
}

template <class P, int KP>
__global__ void __launch_bounds__(kThreads, 2)
    row_vjp_kernel(ModelDev md, int64_t n, const float* __restrict__ node,
                   const float* __restrict__ desc, float* __restrict__ node_grad) {
  __shared__ __align__(16) float rows[kRowAtoms][KP + 8];
  using T = RowTable<P>;
  __shared__ __align__(16) float tab[T::floats(T::kAll)];
  const int ra = threadIdx.x / kRow;
  float* row = rows[ra];
  stage_table(tab, md.row_tab, T::kAll, threadIdx.x, kThreads);
  RowLane<P> k;
  k.init();
  RowVjpPlaces<P> b;
  b.init(k);
  __syncthreads();
  constexpr int kPieces = KP / 4, kEach = (kPieces + kRow - 1) / kRow;
  constexpr int kY0 = (P::C0 + kRow - 1) / kRow;
#pragma unroll 1
  for (int64_t g = blockIdx.x; g * kRowAtoms < n; g += gridDim.x) {
    // opaque: the tables are read from LDS for each atom, not kept in registers
    asm volatile("" : "+v"(k.l));
    const int64_t want = g * kRowAtoms + ra;
    const int64_t i = want < n ? want : n - 1;
    const bool ok = want < n;
    const float* y = node + size_t(i) * P::NS;
    const float* nd = desc + size_t(i) * KP;
    float y1[3], y2[5], y3[P::L >= 3 ? 7 : 1], y4[P::L >= 4 ? 9 : 1], y0[kY0];
    load_features<P>(y, k, y1, y2, y3, y4);
    const float s0 = y[0], s1 = y[1];
#pragma unroll
    for (int q = 0; q < kY0; ++q) {
      const int t = k.l + q * kRow;
      y0[q] = t < P::C0 ? y[P::Y0 + t] : 0.0f;
    }
    // dE/dD~ = dE/dD / sigma, Eq. (calibration)
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int t0 = (k.l + q * kRow) * 4;
      if (t0 < KP)
        *reinterpret_cast<row_f4*>(row + t0) = *reinterpret_cast<const row_f4*>(nd + t0) *
                                               *reinterpret_cast<const row_f4*>(md.inv_sigma + t0);
    }
    RowFwd<P> f;
    row_forward<P>(f, k, tab, s0, s1, y1, y2, y3, y4);
    wave_sync();
    float xb1[3], xb2[5], xb3, xb4;
    row_vjp<P>(f, k, b, tab, row, xb1, xb2, xb3, xb4);
    formed(xb3);
    formed(xb4);
    // the normalisation X = Y / M: sums of Xbar Y per normaliser
    float part0 = 0.0f, part1 = 0.0f;
    float* go = node_grad + size_t(i) * P::NS;
#pragma unroll
    for (int q = 0; q < kY0; ++q) {
      const int t = k.l + q * kRow;
      if (t < P::C0) {
        const float xb = row[P::oX + t];
        part0 = fmaf(xb, y0[q], part0);
        if (ok) go[P::Y0 + t] = xb * f.i0;
      }
    }
    const bool own1 = k.l < P::C1, own2 = k.l < P::C2;   // not a repeated channel
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      part1 = fmaf(own1 ? xb1[m] : 0.0f, y1[m], part1);
      if (ok && own1) go[P::Y1 + m * P::C1 + k.c] = xb1[m] * f.i1;
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      part1 = fmaf(own2 ? xb2[m] : 0.0f, y2[m], part1);
      if (ok && own2) go[P::Y2 + m * P::C2 + k.e] = xb2[m] * f.i1;
    }
    if constexpr (P::L >= 3) {
      // z3l is the component of X; its Y is M1 times that
      part1 = fmaf(xb3, f.z3l * f.m1, part1);
      if (ok && k.l < 7) go[P::Y3 + k.l] = xb3 * f.i1;
    }
    if constexpr (P::L >= 4) {
      part1 = fmaf(xb4, f.z4l * f.m1, part1);
      if (ok && k.l < 9) go[P::Y4 + k.l] = xb4 * f.i1;
    }
    part0 = row_sum(part0);
    part1 = row_sum(part1);
    if (ok && k.l == 0) {
      go[0] = (row[P::oM0] - part0 * f.i0 * f.i0) * 0.5f * f.i0;   // M0 = sqrt(1/4 + S0)
      go[1] = (row[P::oM1] - part1 * f.i1 * f.i1) * 0.5f * f.i1;
    }
    wave_sync();   // the row is free for the next atom
  }
}

}  // namespace

size_t row_table_floats(const dpa4c_model* m) {
  size_t k = 0;
  with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto) {
    using P = decltype(p);
    k = RowTable<P>::floats(RowTable<P>::kAll);
    return 0;
  });
  return k;
}

void build_row_table(const dpa4c_model* m, const float* W1, const float* W2, const float* A1,
                     const float* A2, const float* cpl, float* out) {
  with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto) {
    using P = decltype(p);
    RowTable<P>::build(W1, W2, A1, A2, cpl, out);
    return 0;
  });
}

int launch_readout(const dpa4c_model* m, int64_t n, const int32_t* species, const float* node,
                   float* desc, float2* meta, float* desc_out, hipStream_t st) {
  const int64_t groups = (n + kRowAtoms - 1) / kRowAtoms;
  const unsigned grid = static_cast<unsigned>(groups < kRowGrid ? groups : kRowGrid);
  return with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto) {
    using P = decltype(p);
    hipLaunchKernelGGL((row_readout_kernel<P, mlp_width(P::DOUT)>), dim3(grid), dim3(kThreads), 0,
                       st, m->dev(), m->scales, n, species, node, desc, meta, desc_out);
    DPA4C_HIP_TRY(hipGetLastError());
    return 0;
  });
}

int launch_readout_vjp(const dpa4c_model* m, int64_t n, const float* node, const float* desc,
                       float* node_grad, hipStream_t st) {
  const int64_t groups = (n + kRowAtoms - 1) / kRowAtoms;
  const unsigned grid = static_cast<unsigned>(groups < kRowGrid ? groups : kRowGrid);
  return with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto) {
    using P = decltype(p);
    hipLaunchKernelGGL((row_vjp_kernel<P, mlp_width(P::DOUT)>), dim3(grid), dim3(kThreads), 0, st,
                       m->dev(), n, node, desc, node_grad);
    DPA4C_HIP_TRY(hipGetLastError());
    return 0;
  });
}

}  // namespace dpa4c
