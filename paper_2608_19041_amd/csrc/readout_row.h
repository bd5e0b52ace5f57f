// The invariant readout (Eqs. (alignment) .. (calibration)) and its
// vector-Jacobian product with sixteen lanes, one DPP row, per atom and the
// features in registers: lane l holds channel c = l mod C1 of degree one,
// e = l mod C2 of degree two and probe kappa = e of the half (l / K1) mod 2,
// which stands for the probe eta of degree two.  Narrower models repeat their
// channels around the row, so one rotation serves every width: ror<k> gives
// each lane what the lane k before it in its row holds, and the operand of a
// fused multiply-add can be rotated for free.  A product with a channel matrix
// is then a sum over rotations with that matrix read along its (wrapped)
// diagonals, which each lane keeps in registers; Gram and bispectrum blocks
// come out by diagonals too and go to the descriptor row in LDS through index
// tables that are the same for every atom.
//
// With S_eta the symmetric matrix of the (1,1,2) adjoints, s = S z, P the
// quartic adjoint and r = s + 2 P Q v, the adjoints of the probes are
//   dE/dv = 2 Q (s + P Q v),  dE/dQ + (dE/dQ)^T = sum_kappa v r^T + r v^T,
// so both come from the same three sums.
#pragma once

#include "common.h"
#include "edge_math.h"

namespace dpa4c {

constexpr int kRow = 16;   // lanes per atom

template <int K>
using IC = std::integral_constant<int, K>;

// fn(IC<0>{}), .., fn(IC<N - 1>{})
template <int N, class Fn>
__device__ __forceinline__ void unrolled(Fn&& fn) {
  if constexpr (N > 0) {
    unrolled<N - 1>(fn);
    fn(IC<N - 1>{});
  }
}

template <int Ctrl, class T>
__device__ __forceinline__ T dpp(T x) {
  static_assert(sizeof(T) == 4, "one register");
  const int v = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(v, Ctrl, 0xF, 0xF, true));
}
// the value K lanes before in the row (wrapped)
template <int K, class T>
__device__ __forceinline__ T ror(T x) {
  if constexpr (K % kRow == 0) return x;
  else return dpp<0x120 + K % kRow>(x);
}
// lane K of the row
template <int K, class T>
__device__ __forceinline__ T bcast(T x) { return dpp<0x150 + K>(x); }
// sum over the K1 lanes (4 or 8) of a half, and over the row; every lane gets
// the same bits
template <int K1>
__device__ __forceinline__ float half_row_sum(float x) {
  x += dpp<0xB1>(x);                          // quad_perm [1, 0, 3, 2]
  x += dpp<0x4E>(x);                          // quad_perm [2, 3, 0, 1]
  if constexpr (K1 == 8) x += dpp<0x141>(x);  // row_half_mirror
  return x;
}
__device__ __forceinline__ float row_sum(float x) {
  x = half_row_sum<8>(x);
  return x + ror<8>(x);
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, dpp<0xB1>(x));
  x = fmaxf(x, dpp<0x4E>(x));
  x = fmaxf(x, dpp<0x141>(x));
  return fmaxf(x, ror<8>(x));
}

// x formed here: without it the compiler moves the last multiply-adds of a
// sum past later conditional stores, or its first rotations far ahead, and
// keeps every rotated operand in a register in between
__device__ __forceinline__ void formed(float& x) { asm volatile("" : "+v"(x)); }

constexpr float kRowSqrt2 = 1.4142135623730951f;
constexpr float kRowInvSqrt2 = 0.7071067811865476f;
constexpr float kRowInvSqrt6 = 0.4082482904638631f;
constexpr float kRowInvSqrt5 = 0.4472135954999579f;
constexpr float kRowSqrt12_35 = 0.5855400437691199f;
constexpr float kRowSqrt3 = 1.7320508075688772f;

// index of the (a <= b) pair in row-major order over the upper triangle
__device__ __forceinline__ int row_tri(int a, int b, int C) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  return lo * C - lo * (lo - 1) / 2 + (hi - lo);
}

// which channels and probes a lane stands for
template <class P>
struct RowLane {
  int l, c, e, eta;
  __device__ __forceinline__ void init() {
    l = threadIdx.x & (kRow - 1);
    c = l & (P::C1 - 1);
    e = l & (P::C2 - 1);
    eta = (l / P::K1) & 1;
  }
};

// What the lanes of a row read for every atom, staged once per workgroup:
// the wrapped diagonals of the channel matrices (entry k of a lane belongs
// to the channel that ror<k> brings it) and the couplings of degree three.
// Rows of 16-byte pieces, [piece][lane], so that a row reads whole lines.
//   kW1:  W1[c_k][c]      kW2:  W2[e_k][e]     kA1:  A1[c_k][e]   kA2: A2[e_k][eta]
//   kW1T: W1[c][c_k]      kW2T: W2[e][e_k]     kA1T: A1[c][e_k]
//   kA2P: A2[e][eta], A2[e][1 - eta]
//   kCT: C123[o = l][.] (7, l < 15)   kCW: C233[m1][m2 = l][.] (5 rows of 7, l < 7)
//   kCZ: C123[.][m = l] (15, l < 7)
// and at degree four
//   k134: C134[m1][m3 = l][.] (3 rows of 9, l < 7)    k224: C224[m1][m2 = l][.] (5 of 9, l < 5)
//   k244: C244[m1][a = l][.] (5 of 9, l < 9)          k334: C334[a = l][b][.] (7 of 9, l < 7)
//   k444: C444[a = l][b][.] (9 of 9, l < 9)           k134Z: C134[m1][.][m4 = l] (3 of 7, l < 9)
//   k224Z: C224[m1][.][m4 = l] (5 of 5, l < 9)        k334Z: C334[a][.][m4 = l] (7 of 7, l < 9)
// zero elsewhere; rows begin a piece of their own
template <class P>
struct RowTable {
  static constexpr int C1 = P::C1, C2 = P::C2, K1 = P::K1;
  static constexpr int kW1 = 0, kW2 = kW1 + C1 / 4, kA1 = kW2 + C2 / 4;
  static constexpr int kA2 = kA1 + (P::kHasA1 ? C1 / 4 : 0);
  static constexpr int kCT = kA2 + C2 / 4, kCW = kCT + (P::L >= 3 ? 2 : 0);
  static constexpr bool k4 = P::L >= 4;
  static constexpr int k134 = kCW + (P::L >= 3 ? 10 : 0), k224 = k134 + (k4 ? 9 : 0);
  static constexpr int k244 = k224 + (k4 ? 15 : 0), k334 = k244 + (k4 ? 15 : 0);
  static constexpr int k444 = k334 + (k4 ? 21 : 0);
  static constexpr int kFwd = k444 + (k4 ? 27 : 0);   // pieces of the forward pass
  static constexpr int kW1T = kFwd, kW2T = kW1T + C1 / 4, kA1T = kW2T + C2 / 4;
  static constexpr int kA2P = kA1T + (P::kHasA1 ? K1 / 4 : 0), kCZ = kA2P + 1;
  static constexpr int k134Z = kCZ + (P::L >= 3 ? 4 : 0), k224Z = k134Z + (k4 ? 6 : 0);
  static constexpr int k334Z = k224Z + (k4 ? 10 : 0);
  static constexpr int kAll = k334Z + (k4 ? 14 : 0);
  static constexpr size_t floats(int pieces) { return size_t(pieces) * kRow * 4; }

  // the table, from the parameters on the host (cpl null below degree three)
  static void build(const float* W1, const float* W2, const float* A1, const float* A2,
                    const float* cpl, float* out) {
    auto put = [&](int piece, int l, int q, float v) {
      out[((piece + q / 4) * kRow + l) * 4 + q % 4] = v;
    };
    for (int t = 0; t < kAll * kRow * 4; ++t) out[t] = 0.0f;
    for (int l = 0; l < kRow; ++l) {
      const int c = l & (C1 - 1), e = l & (C2 - 1), eta = (l / K1) & 1;
      for (int q = 0; q < C1; ++q) {
        const int o = (c - q) & (C1 - 1);
        put(kW1, l, q, W1[o * C1 + c]);
        put(kW1T, l, q, W1[c * C1 + o]);
        if (P::kHasA1) put(kA1, l, q, A1[o * K1 + e]);
      }
      for (int q = 0; q < C2; ++q) {
        const int o = (e - q) & (C2 - 1);
        put(kW2, l, q, W2[o * C2 + e]);
        put(kW2T, l, q, W2[e * C2 + o]);
        put(kA2, l, q, A2[o * P::K2 + eta]);
        if (P::kHasA1) put(kA1T, l, q, A1[c * K1 + o]);
      }
      put(kA2P, l, 0, A2[e * P::K2 + eta]);
      put(kA2P, l, 1, A2[e * P::K2 + 1 - eta]);
      if (P::L >= 3) {
        for (int q = 0; q < 7 && l < 15; ++q) put(kCT, l, q, cpl[l * 7 + q]);
        for (int q = 0; q < 35 && l < 7; ++q)
          put(kCW + q / 7 * 2, l, q % 7, cpl[kC123 + (q / 7 * 7 + l) * 7 + q % 7]);
        for (int q = 0; q < 15 && l < 7; ++q) put(kCZ, l, q, cpl[q * 7 + l]);
      }
      if (P::L >= 4) {
        const float *c134 = cpl + kO134, *c224 = cpl + kO224, *c244 = cpl + kO244,
                    *c334 = cpl + kO334, *c444 = cpl + kO444;
        for (int q = 0; q < 27 && l < 7; ++q)
          put(k134 + q / 9 * 3, l, q % 9, c134[(q / 9 * 7 + l) * 9 + q % 9]);
        for (int q = 0; q < 45 && l < 5; ++q)
          put(k224 + q / 9 * 3, l, q % 9, c224[(q / 9 * 5 + l) * 9 + q % 9]);
        for (int q = 0; q < 45 && l < 9; ++q)
          put(k244 + q / 9 * 3, l, q % 9, c244[(q / 9 * 9 + l) * 9 + q % 9]);
        for (int q = 0; q < 63 && l < 7; ++q) put(k334 + q / 9 * 3, l, q % 9, c334[l * 63 + q]);
        for (int q = 0; q < 81 && l < 9; ++q) put(k444 + q / 9 * 3, l, q % 9, c444[l * 81 + q]);
        for (int q = 0; q < 21 && l < 9; ++q) put(k134Z + q / 7 * 2, l, q % 7, c134[q * 9 + l]);
        for (int q = 0; q < 25 && l < 9; ++q) put(k224Z + q / 5 * 2, l, q % 5, c224[q * 9 + l]);
        for (int q = 0; q < 49 && l < 9; ++q) put(k334Z + q / 7 * 2, l, q % 7, c334[q * 9 + l]);
      }
    }
  }
};
typedef float row_f4 __attribute__((ext_vector_type(4)));

// the first ``pieces`` pieces of the table into LDS
__device__ __forceinline__ void stage_table(float* dst, const float* src, int pieces, int tid,
                                            int nthreads) {
  for (int t = tid; t < pieces * kRow; t += nthreads)
    reinterpret_cast<row_f4*>(dst)[t] = reinterpret_cast<const row_f4*>(src)[t];
}

// N floats of a lane from piece ``first`` of the table on.  Not before what
// comes ahead of it in the program: hoisted together the tables would fill the
// registers.
template <int N>
__device__ __forceinline__ void table_read(const float* tab, int first, int l, float (&out)[N]) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < (N + 3) / 4; ++q) {
    const row_f4 v = *reinterpret_cast<const row_f4*>(tab + ((first + q) * kRow + l) * 4);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (4 * q + w < N) out[4 * q + w] = v[w];
  }
}

// acc[m] += sum_k ror<k>(x[m]) w[k] over the N diagonals of a matrix
template <int N, int M>
__device__ __forceinline__ void row_product(float (&acc)[M], const float (&x)[M], const float* tab,
                                            int first, int l) {
  float w[N];
  table_read(tab, first, l, w);
  unrolled<N>([&](auto j) {
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = fmaf(ror<decltype(j)::value>(x[m]), w[j], acc[m]);
  });
#pragma unroll
  for (int m = 0; m < M; ++m) formed(acc[m]);
}

// the forward intermediates of an atom
template <class P>
struct RowFwd {
  float i0, i1, m0, m1;
  float xt1[3], xt2[5];                // aligned features of channels c and e
  float xt3[P::L >= 3 ? 7 : 1];        // degree three, the same in every lane
  float z1[3], z2[5];                  // probes kappa = e and eta
  float q[6];                          // STF of z2: xx, yy, zz, xy, yz, xz
  float qv[3];                         // Q_eta v_kappa
  // T123[o = l], W233[m1][m2 = l], V233[m1] and U123[m1][eta]
  float t123, w233[P::L >= 3 ? 5 : 1], v233[P::L >= 3 ? 5 : 1], u123[P::L >= 3 ? 3 : 1];
  float z3l;                           // degree-three component l (l < 7)
  // degree four (one channel, Z4 = X~4): all components and component l
  // (l < 9); by lane R134[m1] = C134[m1][l] : Z4, R244[m1] = C244[m1][l] : Z4,
  // R334 = C334[l] : Z3 Z4 and R444 = C444[l] : Z4 Z4; in every lane T134[m1],
  // T244[m1] and V224[m1] = T224[m1] : Z2 of this half's eta
  static constexpr int n4 = P::L >= 4 ? 1 : 0;
  float xt4[n4 ? 9 : 1], z4l, r134[n4 ? 3 : 1], r244[n4 ? 5 : 1], r334, r444;
  float t134[n4 ? 3 : 1], t244[n4 ? 5 : 1], v224[n4 ? 5 : 1];
};

// y: the features of the lane (degree one, degree two, all of degree three)
template <class P>
__device__ __forceinline__ void row_forward(RowFwd<P>& f, const RowLane<P>& k, const float* tab,
                                            float s0, float s1, const float (&y1)[3],
                                            const float (&y2)[5],
                                            const float (&y3)[P::L >= 3 ? 7 : 1],
                                            const float (&y4)[P::L >= 4 ? 9 : 1]) {
  f.m0 = sqrtf(0.25f + s0);
  f.m1 = sqrtf(0.25f + s1);
  f.i0 = 1.0f / f.m0;
  f.i1 = 1.0f / f.m1;
  using T = RowTable<P>;
#pragma unroll
  for (int m = 0; m < 3; ++m) f.xt1[m] = 0.0f;
#pragma unroll
  for (int m = 0; m < 5; ++m) f.xt2[m] = 0.0f;
  row_product<P::C1>(f.xt1, y1, tab, T::kW1, k.l);
  row_product<P::C2>(f.xt2, y2, tab, T::kW2, k.l);
  // (I + W) y as y + (W y): the small sum rounds at its own size
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    f.xt1[m] = (y1[m] + f.xt1[m]) * f.i1;
    f.z1[m] = P::kHasA1 ? 0.0f : f.xt1[m];
  }
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    f.xt2[m] = (y2[m] + f.xt2[m]) * f.i1;
    f.z2[m] = 0.0f;
  }
  if constexpr (P::L >= 3) {
#pragma unroll
    for (int m = 0; m < 7; ++m) f.xt3[m] = y3[m] * f.i1;
  }
  if constexpr (P::kHasA1) row_product<P::C1>(f.z1, f.xt1, tab, T::kA1, k.l);
  row_product<P::C2>(f.z2, f.xt2, tab, T::kA2, k.l);
  // STF(z2), Eq. (stf), in the basis order (xy, yz, z^2, xz, x^2 - y^2)
  f.q[0] = -f.z2[2] * kRowInvSqrt6 + f.z2[4] * kRowInvSqrt2;
  f.q[1] = -f.z2[2] * kRowInvSqrt6 - f.z2[4] * kRowInvSqrt2;
  f.q[2] = 2.0f * f.z2[2] * kRowInvSqrt6;
  f.q[3] = f.z2[0] * kRowInvSqrt2;
  f.q[4] = f.z2[1] * kRowInvSqrt2;
  f.q[5] = f.z2[3] * kRowInvSqrt2;
  f.qv[0] = f.q[0] * f.z1[0] + f.q[3] * f.z1[1] + f.q[5] * f.z1[2];
  f.qv[1] = f.q[3] * f.z1[0] + f.q[1] * f.z1[1] + f.q[4] * f.z1[2];
  f.qv[2] = f.q[5] * f.z1[0] + f.q[4] * f.z1[1] + f.q[2] * f.z1[2];
  if constexpr (P::L >= 3) {
    float ct[7];
    table_read(tab, T::kCT, k.l, ct);
    f.t123 = 0.0f;
    f.z3l = 0.0f;
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      f.t123 = fmaf(ct[m], f.xt3[m], f.t123);
      f.z3l = k.l == m ? f.xt3[m] : f.z3l;
    }
#pragma unroll
    for (int m1 = 0; m1 < 5; ++m1) {
      float acc = 0.0f, cw[7];
      table_read(tab, T::kCW + 2 * m1, k.l, cw);
#pragma unroll
      for (int m3 = 0; m3 < 7; ++m3) acc = fmaf(cw[m3], f.xt3[m3], acc);
      f.w233[m1] = acc;
      f.v233[m1] = row_sum(acc * f.z3l);
      formed(f.v233[m1]);
    }
    unrolled<3>([&](auto m1) {
      float acc = 0.0f;
      unrolled<5>([&](auto m2) {
        acc = fmaf(bcast<decltype(m1)::value * 5 + decltype(m2)::value>(f.t123), f.z2[m2], acc);
      });
      f.u123[m1] = acc;
      formed(f.u123[m1]);
    });
  }
  if constexpr (P::L >= 4) {
    f.z4l = 0.0f;
#pragma unroll
    for (int m = 0; m < 9; ++m) {
      f.xt4[m] = y4[m] * f.i1;
      f.z4l = k.l == m ? f.xt4[m] : f.z4l;
    }
    // one row of nine couplings against Z4
    auto dot4 = [&](int piece) {
      float c[9], acc = 0.0f;
      table_read(tab, piece, k.l, c);
#pragma unroll
      for (int e = 0; e < 9; ++e) acc = fmaf(c[e], f.xt4[e], acc);
      return acc;
    };
#pragma unroll
    for (int m1 = 0; m1 < 3; ++m1) {
      f.r134[m1] = dot4(T::k134 + 3 * m1);
      f.t134[m1] = row_sum(f.r134[m1] * f.z3l);
      formed(f.t134[m1]);
    }
#pragma unroll
    for (int m1 = 0; m1 < 5; ++m1) {
      const float t = dot4(T::k224 + 3 * m1);   // T224[m1][m2 = l]
      float acc = 0.0f;
      unrolled<5>([&](auto m2) { acc = fmaf(bcast<decltype(m2)::value>(t), f.z2[m2], acc); });
      f.v224[m1] = acc;
      formed(f.v224[m1]);
    }
#pragma unroll
    for (int m1 = 0; m1 < 5; ++m1) {
      f.r244[m1] = dot4(T::k244 + 3 * m1);
      f.t244[m1] = row_sum(f.r244[m1] * f.z4l);
      formed(f.t244[m1]);
    }
    f.r334 = f.r444 = 0.0f;
#pragma unroll
    for (int b = 0; b < 7; ++b) f.r334 = fmaf(dot4(T::k334 + 3 * b), f.xt3[b], f.r334);
#pragma unroll
    for (int b = 0; b < 9; ++b) f.r444 = fmaf(dot4(T::k444 + 3 * b), f.xt4[b], f.r444);
    formed(f.r334);
    formed(f.r444);
  }
}

// x (symmetric, six entries) times itself
__device__ __forceinline__ void sym_square(const float (&q)[6], float (&s)[6]) {
  s[0] = q[0] * q[0] + q[3] * q[3] + q[5] * q[5];
  s[1] = q[3] * q[3] + q[1] * q[1] + q[4] * q[4];
  s[2] = q[5] * q[5] + q[4] * q[4] + q[2] * q[2];
  s[3] = q[0] * q[3] + q[3] * q[1] + q[5] * q[4];
  s[4] = q[3] * q[5] + q[1] * q[4] + q[4] * q[2];
  s[5] = q[0] * q[5] + q[3] * q[4] + q[5] * q[2];
}
// tr(A B) of symmetric matrices
__device__ __forceinline__ float sym_trace(const float (&a)[6], const float (&b)[6]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] +
         2.0f * (a[3] * b[3] + a[4] * b[4] + a[5] * b[5]);
}

// places of a lane's descriptor entries (offsets into the descriptor)
template <class P>
struct RowPlaces {
  static constexpr int N1 = P::C1 / 2 + 1, N2 = P::C2 / 2 + 1, N3 = P::K1 / 2 + 1;
  int g1[N1], g2[N2], j112[N3];
  __device__ __forceinline__ void init(const RowLane<P>& k) {
#pragma unroll
    for (int j = 0; j < N1; ++j) g1[j] = P::oG1 + row_tri(k.c, (k.c - j) & (P::C1 - 1), P::C1);
#pragma unroll
    for (int j = 0; j < N2; ++j) g2[j] = P::oG2 + row_tri(k.e, (k.e - j) & (P::C2 - 1), P::C2);
#pragma unroll
    for (int j = 0; j < N3; ++j)
      j112[j] = P::o112 + row_tri(k.e, (k.e - j) & (P::K1 - 1), P::K1) * P::K2 + k.eta;
  }
};

// The descriptor before calibration, but for its first 2 C0 entries, into the
// atom's row ``d``.  Lanes that hold the same entry write the same bits.
template <class P>
__device__ __forceinline__ void row_descriptor(const RowFwd<P>& f, const RowLane<P>& k,
                                               const RowPlaces<P>& at, float* d) {
  unrolled<RowPlaces<P>::N1>([&](auto j) {
    constexpr int J = decltype(j)::value;
    float acc = 0.0f;
#pragma unroll
    for (int m = 0; m < 3; ++m) acc = fmaf(ror<J>(f.xt1[m]), f.xt1[m], acc);
    d[at.g1[J]] = J == 0 ? acc : acc * kRowSqrt2;
  });
  unrolled<RowPlaces<P>::N2>([&](auto j) {
    constexpr int J = decltype(j)::value;
    float acc = 0.0f;
#pragma unroll
    for (int m = 0; m < 5; ++m) acc = fmaf(ror<J>(f.xt2[m]), f.xt2[m], acc);
    d[at.g2[J]] = J == 0 ? acc : acc * kRowSqrt2;
  });
  // (1,1,2): -(f / sqrt 5) v_k1 . Q_eta v_k2, from the lane of k2
  unrolled<RowPlaces<P>::N3>([&](auto j) {
    constexpr int J = decltype(j)::value;
    float acc = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) acc = fmaf(ror<J>(f.z1[a]), f.qv[a], acc);
    acc *= J == 0 ? -kRowInvSqrt5 : -kRowInvSqrt5 * kRowSqrt2;
    // the half-way diagonal holds each pair twice, as v_k1 . Q v_k2 and
    // v_k2 . Q v_k1, equal but for rounding: the lane of the larger index writes
    if (2 * J < P::K1 || k.e >= J) d[at.j112[J]] = acc;
  });
  // (2,2,2): -sqrt(12/35) w tr(Q Q Q) with this half's Q at least twice
  {
    float qo[6], s[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) qo[t] = ror<P::K1>(f.q[t]);
    sym_square(f.q, s);
    d[P::o222 + 3 * k.eta] = -kRowSqrt12_35 * sym_trace(s, f.q);
    d[P::o222 + 1 + k.eta] = -kRowSqrt12_35 * kRowSqrt3 * sym_trace(s, qo);
  }
  // quartic, Eq. (quartic), eta-major
  d[P::oPi + k.eta * P::K1 + k.e] = f.qv[0] * f.qv[0] + f.qv[1] * f.qv[1] + f.qv[2] * f.qv[2];
  if constexpr (P::L >= 3) {
    float g = 0.0f, j = 0.0f;
#pragma unroll
    for (int m = 0; m < 7; ++m) g = fmaf(f.xt3[m], f.xt3[m], g);
    d[P::oG3] = g;
#pragma unroll
    for (int m = 0; m < 3; ++m) j = fmaf(f.z1[m], f.u123[m], j);
    d[P::o123 + k.e * P::K2 + k.eta] = j;
    float v = 0.0f;
#pragma unroll
    for (int m = 0; m < 5; ++m) v = fmaf(f.z2[m], f.v233[m], v);
    d[P::o233 + k.eta] = v;
  }
  if constexpr (P::L >= 4) {
    float g = 0.0f, j134 = 0.0f, own = 0.0f, off = 0.0f, j244 = 0.0f;
#pragma unroll
    for (int m = 0; m < 9; ++m) g = fmaf(f.xt4[m], f.xt4[m], g);
    d[P::oG4] = g;
#pragma unroll
    for (int m = 0; m < 3; ++m) j134 = fmaf(f.z1[m], f.t134[m], j134);
    d[P::o134 + k.e] = j134;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      own = fmaf(f.z2[m], f.v224[m], own);
      off = fmaf(f.z2[m], ror<P::K1>(f.v224[m]), off);
      j244 = fmaf(f.z2[m], f.t244[m], j244);
    }
    // (k1, k2) = (0, 0), (0, 1), (1, 1); the mixed one from the lanes of eta 0
    d[P::o224 + 2 * k.eta] = own;
    if (k.eta == 0) d[P::o224 + 1] = off * kRowSqrt2;
    d[P::o244 + k.eta] = j244;
    d[P::o334] = row_sum(f.r334 * f.z3l);
    d[P::o444] = row_sum(f.r444 * f.z4l);
  }
  d[P::oM0] = f.m0;
  d[P::oM1] = f.m1;
}

// places of the adjoints a lane reads, by rotation
template <class P>
struct RowVjpPlaces {
  int g1[P::C1], g2[P::C2], j112[P::K1];
  __device__ __forceinline__ void init(const RowLane<P>& k) {
#pragma unroll
    for (int j = 0; j < P::C1; ++j)
      g1[j] = P::oG1 + row_tri(k.c, (k.c - j) & (P::C1 - 1), P::C1);
#pragma unroll
    for (int j = 0; j < P::C2; ++j)
      g2[j] = P::oG2 + row_tri(k.e, (k.e - j) & (P::C2 - 1), P::C2);
#pragma unroll
    for (int j = 0; j < P::K1; ++j)
      j112[j] = P::o112 + row_tri(k.e, (k.e - j) & (P::K1 - 1), P::K1) * P::K2 + k.eta;
  }
};

// dE/dY of degrees one to three (lane entries), divided by nothing yet: xb =
// dE/dX of the normalised features, from dE/dD~ in the atom's row ``d``.
template <class P>
__device__ __forceinline__ void row_vjp(const RowFwd<P>& f, const RowLane<P>& k,
                                        const RowVjpPlaces<P>& b, const float* tab, const float* d,
                                        float (&xb1)[3], float (&xb2)[5], float& xb3,
                                        float& xb4) {
  using T = RowTable<P>;
  // s = S z with the (1,1,2) adjoints, this half's eta
  float s[3] = {0.0f, 0.0f, 0.0f};
  unrolled<P::K1>([&](auto j) {
    constexpr int J = decltype(j)::value;
    const float w = d[b.j112[J]] * (J == 0 ? -kRowInvSqrt5 : -kRowInvSqrt5 * kRowInvSqrt2);
#pragma unroll
    for (int m = 0; m < 3; ++m) s[m] = fmaf(ror<J>(f.z1[m]), w, s[m]);
  });
#pragma unroll
  for (int m = 0; m < 3; ++m) formed(s[m]);
  const float pb = d[P::oPi + k.eta * P::K1 + k.e];
  float t[3], r[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    t[m] = fmaf(pb, f.qv[m], s[m]);
    r[m] = fmaf(pb, f.qv[m], t[m]);
  }
  // dE/dv of this eta; the other half adds its own below
  float gz1[3];
  gz1[0] = 2.0f * (f.q[0] * t[0] + f.q[3] * t[1] + f.q[5] * t[2]);
  gz1[1] = 2.0f * (f.q[3] * t[0] + f.q[1] * t[1] + f.q[4] * t[2]);
  gz1[2] = 2.0f * (f.q[5] * t[0] + f.q[4] * t[1] + f.q[2] * t[2]);
  // dE/dz2 = E_m : dE/dQ
  float gz2[5];
  {
    const float g0 = f.z1[0] * r[0], g1 = f.z1[1] * r[1], g2 = f.z1[2] * r[2];
    gz2[0] = half_row_sum<P::K1>(f.z1[0] * r[1] + f.z1[1] * r[0]) * kRowInvSqrt2;
    gz2[1] = half_row_sum<P::K1>(f.z1[1] * r[2] + f.z1[2] * r[1]) * kRowInvSqrt2;
    gz2[2] = half_row_sum<P::K1>(2.0f * g2 - g0 - g1) * kRowInvSqrt6;
    gz2[3] = half_row_sum<P::K1>(f.z1[0] * r[2] + f.z1[2] * r[0]) * kRowInvSqrt2;
    gz2[4] = half_row_sum<P::K1>(g0 - g1) * kRowInvSqrt2;
  }
  {
    // (2,2,2): 3 a Q^2 + b (Q Q' + Q' Q) + c Q'^2, Q' the other half's
    const float w = -kRowSqrt12_35;
    const float ja = 3.0f * w * d[P::o222 + 3 * k.eta];
    const float jb = w * kRowSqrt3 * d[P::o222 + 1 + k.eta];
    const float jc = w * kRowSqrt3 * d[P::o222 + 2 - k.eta];
    float qo[6], ss[6], so[6], g[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) qo[i] = ror<P::K1>(f.q[i]);
    sym_square(f.q, ss);
    const float* q = f.q;
    float mm[6];   // the symmetric product Q Q' + Q' Q
    mm[0] = 2.0f * (q[0] * qo[0] + q[3] * qo[3] + q[5] * qo[5]);
    mm[1] = 2.0f * (q[3] * qo[3] + q[1] * qo[1] + q[4] * qo[4]);
    mm[2] = 2.0f * (q[5] * qo[5] + q[4] * qo[4] + q[2] * qo[2]);
    mm[3] = q[0] * qo[3] + q[3] * qo[1] + q[5] * qo[4] + qo[0] * q[3] + qo[3] * q[1] + qo[5] * q[4];
    mm[4] = q[3] * qo[5] + q[1] * qo[4] + q[4] * qo[2] + qo[3] * q[5] + qo[1] * q[4] + qo[4] * q[2];
    mm[5] = q[0] * qo[5] + q[3] * qo[4] + q[5] * qo[2] + qo[0] * q[5] + qo[3] * q[4] + qo[5] * q[2];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      so[i] = ror<P::K1>(ss[i]);
      g[i] = ja * ss[i] + jb * mm[i] + jc * so[i];
    }
    gz2[0] += 2.0f * g[3] * kRowInvSqrt2;
    gz2[1] += 2.0f * g[4] * kRowInvSqrt2;
    gz2[2] += (2.0f * g[2] - g[0] - g[1]) * kRowInvSqrt6;
    gz2[3] += 2.0f * g[5] * kRowInvSqrt2;
    gz2[4] += (g[0] - g[1]) * kRowInvSqrt2;
  }
#pragma unroll
  for (int m = 0; m < 5; ++m) formed(gz2[m]);
  xb3 = 0.0f;
  xb4 = 0.0f;
  if constexpr (P::L >= 3) {
    const float j123 = d[P::o123 + k.e * P::K2 + k.eta], j233 = d[P::o233 + k.eta];
    float cz[15];
    table_read(tab, T::kCZ, k.l, cz);
    float ub[3], vb[5];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      gz1[m] = fmaf(j123, f.u123[m], gz1[m]);
      ub[m] = half_row_sum<P::K1>(j123 * f.z1[m]);
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      vb[m] = j233 * f.z2[m];
      vb[m] += ror<P::K1>(vb[m]);
    }
    float gz3 = 0.0f;
#pragma unroll
    for (int m1 = 0; m1 < 3; ++m1)
#pragma unroll
      for (int m2 = 0; m2 < 5; ++m2) {
        float tb = ub[m1] * f.z2[m2];
        tb += ror<P::K1>(tb);
        gz3 = fmaf(tb, cz[5 * m1 + m2], gz3);
        formed(gz3);
      }
#pragma unroll
    for (int m1 = 0; m1 < 5; ++m1) gz3 = fmaf(2.0f * vb[m1], f.w233[m1], gz3);
    unrolled<5>([&](auto m) {
      float acc = gz2[m];
      unrolled<3>([&](auto m1) {
        acc = fmaf(bcast<decltype(m1)::value * 5 + decltype(m)::value>(f.t123), ub[m1], acc);
      });
      gz2[m] = fmaf(j233, f.v233[m], acc);
      formed(gz2[m]);
    });
    xb3 = fmaf(2.0f * d[P::oG3], f.z3l, gz3);
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) gz1[m] += ror<P::K1>(gz1[m]);   // both etas
  if constexpr (P::L >= 4) {
    const float j134 = d[P::o134 + k.e], j334 = d[P::o334], j444 = d[P::o444];
    const float jown = d[P::o224 + 2 * k.eta], joff = d[P::o224 + 1] * kRowSqrt2;
    const float j244 = d[P::o244 + k.eta];
    float gz4 = 0.0f, gz3 = 0.0f, z2o[5];
#pragma unroll
    for (int m1 = 0; m1 < 3; ++m1) {
      float c[7], r = 0.0f;
      table_read(tab, T::k134Z + 2 * m1, k.l, c);
      const float tb134 = half_row_sum<P::K1>(j134 * f.z1[m1]);
      gz1[m1] = fmaf(j134, f.t134[m1], gz1[m1]);
      gz3 = fmaf(tb134, f.r134[m1], gz3);
#pragma unroll
      for (int a = 0; a < 7; ++a) r = fmaf(c[a], f.xt3[a], r);
      gz4 = fmaf(tb134, r, gz4);
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) z2o[m] = ror<P::K1>(f.z2[m]);
    // the (2,2,4) adjoint of T224 made symmetric: this half's share is
    // Jbar z z + (Jbar_01 / 2) z z', the halves together the whole
#pragma unroll
    for (int m1 = 0; m1 < 5; ++m1) {
      float c[5];
      table_read(tab, T::k224Z + 2 * m1, k.l, c);
#pragma unroll
      for (int m2 = 0; m2 < 5; ++m2) {
        float tb = f.z2[m1] * fmaf(jown, f.z2[m2], 0.5f * joff * z2o[m2]);
        tb += ror<P::K1>(tb);
        gz4 = fmaf(tb, c[m2], gz4);
      }
      formed(gz4);
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      gz2[m] = fmaf(2.0f * jown, f.v224[m], gz2[m]);
      gz2[m] = fmaf(joff, ror<P::K1>(f.v224[m]), gz2[m]);
      gz2[m] = fmaf(j244, f.t244[m], gz2[m]);
      float tb = j244 * f.z2[m];
      tb += ror<P::K1>(tb);
      gz4 = fmaf(2.0f * tb, f.r244[m], gz4);
    }
    {
      float r = 0.0f;
#pragma unroll
      for (int a = 0; a < 7; ++a) {
        float c[7], q = 0.0f;
        table_read(tab, T::k334Z + 2 * a, k.l, c);
#pragma unroll
        for (int e = 0; e < 7; ++e) q = fmaf(c[e], f.xt3[e], q);
        r = fmaf(q, f.xt3[a], r);
      }
      gz4 = fmaf(j334, r, gz4);
    }
    gz3 = fmaf(2.0f * j334, f.r334, gz3);
    gz4 = fmaf(3.0f * j444, f.r444, gz4);
    xb3 += gz3;
    xb4 = fmaf(2.0f * d[P::oG4], f.z4l, gz4);
  }
  // dE/dX~ from the Gram blocks and the probes
  float gx1[3] = {0.0f, 0.0f, 0.0f}, gx2[5];
  unrolled<P::C1>([&](auto j) {
    constexpr int J = decltype(j)::value;
    const float w = d[b.g1[J]] * (J == 0 ? 2.0f : kRowSqrt2);
#pragma unroll
    for (int m = 0; m < 3; ++m) gx1[m] = fmaf(ror<J>(f.xt1[m]), w, gx1[m]);
  });
#pragma unroll
  for (int m = 0; m < 3; ++m) formed(gx1[m]);
  if constexpr (P::kHasA1) {
    row_product<P::K1>(gx1, gz1, tab, T::kA1T, k.l);
  } else {
#pragma unroll
    for (int m = 0; m < 3; ++m) gx1[m] += gz1[m];
  }
  float a2[2];
  table_read(tab, T::kA2P, k.l, a2);
#pragma unroll
  for (int m = 0; m < 5; ++m) gx2[m] = fmaf(gz2[m], a2[0], ror<P::K1>(gz2[m]) * a2[1]);
  unrolled<P::C2>([&](auto j) {
    constexpr int J = decltype(j)::value;
    const float w = d[b.g2[J]] * (J == 0 ? 2.0f : kRowSqrt2);
#pragma unroll
    for (int m = 0; m < 5; ++m) gx2[m] = fmaf(ror<J>(f.xt2[m]), w, gx2[m]);
  });
#pragma unroll
  for (int m = 0; m < 5; ++m) formed(gx2[m]);
  // through the alignment (I + W), W's share summed by itself
#pragma unroll
  for (int m = 0; m < 3; ++m) xb1[m] = 0.0f;
#pragma unroll
  for (int m = 0; m < 5; ++m) xb2[m] = 0.0f;
  row_product<P::C1>(xb1, gx1, tab, T::kW1T, k.l);
  row_product<P::C2>(xb2, gx2, tab, T::kW2T, k.l);
#pragma unroll
  for (int m = 0; m < 3; ++m) xb1[m] += gx1[m];
#pragma unroll
  for (int m = 0; m < 5; ++m) xb2[m] += gx2[m];
}

}  // namespace dpa4c
