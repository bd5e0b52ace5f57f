// The atomic-energy MLP, its head and its input gradient for tiles of atoms
// (Eqs. (atomic-energy), (fitting)):
//
//   h1 = SiLU(D Th1 + b1), h2 = SiLU(h1 Th2 + b2) + h1, h3 = SiLU(h2 Th3 + b3) + h2
//   E  = h3 . w + b + E_ref[a]
//   hb2 = w + (w * s3) Th3^T,  hb1 = hb2 + (hb2 * s2) Th2^T,  dE/dD = (hb1 * s1) Th1^T
//
// with s_t = SiLU'(pre_t).  One workgroup takes 16 RT atoms through all six
// products; the descriptor comes in from, and dE/dD goes out to, one row of
// 4 KP bytes per atom that the readout kernels fill and read.
//
// Products.  Every float32 operand x is carried as two float16 numbers,
// x 2^e = hi + lo with hi = f16(x 2^e), lo = f16(x 2^e - hi), and a product
// is three v_mfma_f32_16x16x32_f16 per 32 inputs, lo hi + hi lo + hi hi,
// accumulated in float32.  hi + lo holds x to one float32 ulp or better, the
// product of the two lo parts, at most 2^-22 of the whole, is left out, and
// the accumulation rounds every 32 inputs instead of every input: against
// 64 bits dE/dD from the same descriptor is off by 1.7 to 4.3e-7 of its norm
// (seven models, a crystal and a cluster), 0.65 to 0.87 of what float32
// products reach.  v_mfma_f32_16x16x4_f32 takes 5.3 times as long.  The
// exponents e are powers of two that keep |x 2^e| at or below 2^15: per matrix for the weights (model set-up), per atom for D, h1
// and h2 (from bounds that start at the row's own norms, MlpScales), per
// model for the backward operands.  Entries far below a row's bound lose
// relative, not absolute, precision: the float16 subnormals end 2^-39 below
// the bound.
//
// Layout.  The weights are the A operand and the atoms the B operand, so a
// lane ends up with four consecutive features of one atom and writes them to
// LDS (two planes, hi and lo, [atom][feature]) with two 8-byte stores.  Each
// wave owns NT fixed 16-feature tiles, streamed from L2 once for all RT atom
// tiles: at RT = 4 a 32-input block of the full width is 48 KB of weights
// for 1152 matrix-core cycles of a SIMD, under the 64 B per cycle that L1
// returns.
#include <hip/hip_runtime.h>

#include "../../include/dpa4c.h"
#include "edge_math.h"
#include "launch.h"

namespace dpa4c {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// logistic function with the hardware reciprocal (v_rcp_f32, within 1 ulp)
__device__ inline float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// x as a value the compiler knows nothing about: what is formed from it is
// formed here, and not kept in registers from an earlier use
__device__ inline float opaque(float x) {
  asm("" : "+v"(x));
  return x;
}

constexpr int kBufWord3 = 0x00020000;   // raw 32-bit buffer, gfx9 data format

// One 16-byte load through a buffer resource: descriptor and tile offset in
// scalar registers, only the lane offset in a vector register.
__device__ inline v8h load_frag(__amdgpu_buffer_rsrc_t rs, unsigned lane16, int soff) {
  const u4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, static_cast<int>(lane16), soff, 0);
  return __builtin_bit_cast(v8h, v);
}

// hi and lo planes of one feature tile's weights for one 32-input block
template <int NT>
struct WBlock {
  v8h hi[NT], lo[NT];
};

// The weight stream of one product: fragment order [tile][block][plane][lane]
// of 16 bytes; tiles first, first + stride, .. (tiles past the last repeat it).
template <int NT>
struct WStream {
  __amdgpu_buffer_rsrc_t rs;
  int toff[NT];
  __device__ inline void open(const void* w, int blocks, int first, int stride, int ntiles) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w), 0, ntiles * blocks * 2048,
                                           kBufWord3);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int T = first + t * stride < ntiles ? first + t * stride : ntiles - 1;
      toff[t] = T * blocks * 2048;
    }
  }
  __device__ inline void load(WBlock<NT>& b, unsigned lane16, int kb) const {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      b.hi[t] = load_frag(rs, lane16, toff[t] + kb * 2048);
      b.lo[t] = load_frag(rs, lane16, toff[t] + kb * 2048 + 1024);
    }
  }
};

// Blocks of weights in flight: requested D - 1 blocks ahead of their use.
// With 64 atoms a block's products last long enough to cover the L2 latency
// from one block ahead, and the registers hold no more; the smaller tiles
// take less time for a block and have the room for more of them.
constexpr int blocks_in_flight(int rt) { return rt == 1 ? 4 : rt == 2 ? 3 : 2; }

template <int NT, int D>
struct WRing {
  WBlock<NT> b[D];
  // the first D - 1 blocks of a product
  __device__ inline void start(const WStream<NT>& ws, unsigned lane16, int blocks) {
#pragma unroll
    for (int k = 0; k < D - 1; ++k)
      if (k < blocks) ws.load(b[k], lane16, k);
  }
};

// acc[t][r] += W tile t x activations of atom tile r over KB blocks of 32
// inputs; the ring holds the first D - 1 blocks of weights.
template <int NT, int RT, int KB, int D>
__device__ inline void product(v4f (&acc)[NT][RT], const WStream<NT>& ws, WRing<NT, D>& ring,
                               const _Float16* act, int ld, int plane, unsigned lane16) {
  v8h lo[RT], hi[RT];
  auto load_lo = [&](int kb) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
      lo[r] = *reinterpret_cast<const v8h*>(act + plane + r * 16 * ld + kb * 32);
  };
  auto load_hi = [&](int kb) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
      hi[r] = *reinterpret_cast<const v8h*>(act + r * 16 * ld + kb * 32);
  };
  auto mul = [&](const v8h* w, const v8h* a) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[t], a[r], acc[t][r], 0, 0, 0);
  };
  // one block's products; the activations of the next block replace this
  // block's as soon as they are consumed: its lo parts have two thirds of the
  // block to arrive, its hi parts the first third of the next
  auto step = [&](const WBlock<NT>& b, int kb, auto more_c) {
    constexpr bool more = decltype(more_c)::value;   // a block follows
    __builtin_amdgcn_sched_barrier(0);   // keep the requests ahead of the products
    mul(b.hi, lo);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (more) load_lo(kb + 1);
    __builtin_amdgcn_sched_barrier(0);
    mul(b.lo, hi);
    mul(b.hi, hi);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (more) load_hi(kb + 1);
  };
  load_lo(0);
  load_hi(0);
  // rounds of D blocks after which every request of the round is in range
  constexpr int kRounds = KB >= 2 * D - 1 ? (KB - (D - 1)) / D : 0;
#pragma unroll 1
  for (int p = 0; p < kRounds; ++p) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      ws.load(ring.b[(u + D - 1) % D], lane16, p * D + u + D - 1);
      step(ring.b[u], p * D + u, std::true_type{});
    }
  }
#pragma unroll
  for (int kb = kRounds * D; kb < KB - 1; ++kb) {
    if (kb + D - 1 < KB) ws.load(ring.b[(kb + D - 1) % D], lane16, kb + D - 1);
    step(ring.b[kb % D], kb, std::true_type{});
  }
  step(ring.b[(KB - 1) % D], KB - 1, std::false_type{});
}

struct ChainArgs {
  const void* W[3];       // Theta_t split in fragment order (inputs KP, F, F; F features)
  const void* WT[3];      // their transposes (F inputs; KP, F, F features)
  const float* bias[3];
  const float* w_head;
  const float* E_ref;
  float b_head;
  int n_types1;
  MlpScales sc;
};

template <int KP, int F, int RT, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
    chain_kernel(ChainArgs p, int64_t n, const int32_t* __restrict__ species,
                 float* __restrict__ desc, const float2* __restrict__ meta,
                 double* __restrict__ e_atom) {
  constexpr int R = 16 * RT;
  constexpr int LD = (KP > F ? KP : F) + 8;   // halves; LD / 2 = 4 x odd mod 64: no bank conflicts
  constexpr int PL = R * LD;                  // halves per plane
  constexpr int FT = F / 16, NT = FT / NW;
  static_assert(FT % NW == 0 && KP % 32 == 0 && F % 32 == 0, "tile split");
  constexpr int DT = KP / 16;                 // feature tiles of dE/dD
  constexpr int KBD = KP / 32, KBF = F / 32;
  __shared__ __align__(16) _Float16 act[2 * PL];
  __shared__ double epart[NW][R];
  __shared__ __align__(16) float vec[4][F];   // b1, b2, b3, w
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const unsigned lane16 = 16u * lane;
  const _Float16* act_rd = act + col * LD + 8 * grp;   // this lane's operand rows
  constexpr int D = blocks_in_flight(RT);
  WStream<NT> ws;
  WRing<NT, D> ring;
  for (int t = threadIdx.x; t < F; t += 64 * NW) {
#pragma unroll
    for (int v = 0; v < 3; ++v) vec[v][t] = p.bias[v][t];
    vec[3][t] = p.w_head[t];
  }
  const int64_t row0 = int64_t(blockIdx.x) * R;
  ws.open(p.W[0], KBD, wave, NW, FT);
  ring.start(ws, lane16, KBD);
  // ---- the tile's descriptor planes into LDS (rows past n: zeros)
  {
    constexpr int kPerRow = KP / 4;                       // 16-byte pieces of an atom's row
    constexpr int kPieces = R * kPerRow, kThreads = 64 * NW;
    constexpr int kEach = (kPieces + kThreads - 1) / kThreads;
    u4 v[kEach];
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int pc = threadIdx.x + q * kThreads;
      const int row = pc / kPerRow, at = pc % kPerRow;
      v[q] = u4{0u, 0u, 0u, 0u};
      if (pc < kPieces && row0 + row < n)
        v[q] = *reinterpret_cast<const u4*>(desc + (row0 + row) * size_t(KP) + at * 4);
    }
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int pc = threadIdx.x + q * kThreads;
      const int row = pc / kPerRow, at = pc % kPerRow;
      const int pl = at / (KP / 8), k8 = at % (KP / 8);
      if (pc < kPieces) *reinterpret_cast<u4*>(act + pl * PL + row * LD + k8 * 8) = v[q];
    }
  }
  // ---- the scales of this lane's atoms (one per atom tile)
  float undo[RT], bound[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int64_t i = row0 + r * 16 + col;
    const float2 mt = i < n ? meta[i] : make_float2(1.0f, 1.0f);
    undo[r] = mt.x * p.sc.w_undo[0];   // 2^-(e_D + e_W)
    bound[r] = mt.y;                   // of |h1|
  }
  __syncthreads();

  // pre-activations of the first two layers; the second's place is taken by
  // hbar2 on the way back
  v4f p1[NT][RT], p2[NT][RT];
  float part[RT];                      // this wave's share of h3 . w
#pragma unroll
  for (int r = 0; r < RT; ++r) part[r] = 0.0f;
  // four features of one atom as the next operand
  auto put = [&](int at, const v4f& x) {
    v4h hi, lo;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      hi[c] = static_cast<_Float16>(x[c]);
      lo[c] = static_cast<_Float16>(x[c] - static_cast<float>(hi[c]));
    }
    *reinterpret_cast<v4h*>(act + at) = hi;
    *reinterpret_cast<v4h*>(act + PL + at) = lo;
    __builtin_amdgcn_sched_barrier(0);   // one tile's values in registers at a time
  };
#pragma unroll
  for (int layer = 0; layer < 3; ++layer) {
    v4f acc[NT][RT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[t][r] = v4f{0.f, 0.f, 0.f, 0.f};
    if (layer == 0)
      product<NT, RT, KBD, D>(acc, ws, ring, act_rd, LD, PL, lane16);
    else
      product<NT, RT, KBF, D>(acc, ws, ring, act_rd, LD, PL, lane16);
    ws.open(layer < 2 ? p.W[layer + 1] : p.WT[2], KBF, wave, NW, FT);
    ring.start(ws, lane16, KBF);
    __syncthreads();   // everyone has read the operand planes
    // scales of the operands this layer writes, and of the next products
    float und[RT], up[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const float b = layer == 0 ? bound[r] : bound[r] * p.sc.h2_mul + p.sc.h2_add;
      const int e = operand_exponent(b);
      up[r] = layer == 2 ? p.sc.p_up[2] : __builtin_amdgcn_ldexpf(1.0f, e);
      und[r] = undo[r];
      if (layer < 2) undo[r] = __builtin_amdgcn_ldexpf(p.sc.w_undo[layer + 1], -e);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int f = (wave + NW * t) * 16 + 4 * grp;
      const v4f bias = *reinterpret_cast<const v4f*>(&vec[layer][f]);
      const v4f wh = *reinterpret_cast<const v4f*>(&vec[3][f]);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        v4f x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float pre = fmaf(acc[t][r][c], und[r], bias[c]);
          const float sg = sigm(pre);
          const float a = pre * sg;
          if (layer == 0) {
            p1[t][r][c] = pre;
            x[c] = a * up[r];
          } else if (layer == 1) {
            p2[t][r][c] = pre;
            const float z1 = opaque(p1[t][r][c]);
            const float h1 = z1 * sigm(z1);
            const float h2 = a + h1;   // identity residual
            part[r] = fmaf(h2, wh[c], part[r]);
            x[c] = h2 * up[r];
          } else {
            part[r] = fmaf(a, wh[c], part[r]);   // h3 = a + h2
            const float s = sg * (1.0f + pre * (1.0f - sg));
            x[c] = wh[c] * s * up[r];            // p3 = w s3
          }
        }
        put((r * 16 + col) * LD + f, x);
      }
    }
    if (layer == 2) {
      // head: fixed-order sums over this wave's features; from the lanes' shares
      // on in 64 bits, since those sums are of the size of E itself
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        double sum = part[r];
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (grp == 0) epart[wave][r * 16 + col] = sum;
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < R; i += 64 * NW) {
    if (row0 + i < n) {
      double e = epart[0][i];
#pragma unroll
      for (int w = 1; w < NW; ++w) e += epart[w][i];
      int a = species[row0 + i];
      a = static_cast<unsigned>(a) < static_cast<unsigned>(p.n_types1) ? a : p.n_types1 - 1;
      e_atom[row0 + i] = e + double(p.b_head) + double(p.E_ref[a]);
    }
  }
  // dE/dD: ND whole feature tiles for each wave, and what is left of them in
  // single (feature tile, atom tile) pairs
  constexpr int ND = DT / NW, kLeft = DT - ND * NW;
  WStream<ND> wd;
  WRing<ND, D> ringd;
  // ---- hbar_{t-1} = hbar_t + p_t Th_t^T,  p_{t-1} = hbar_{t-1} s_{t-1}
#pragma unroll
  for (int layer = 2; layer >= 1; --layer) {
    v4f acc[NT][RT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[t][r] = v4f{0.f, 0.f, 0.f, 0.f};
    product<NT, RT, KBF, D>(acc, ws, ring, act_rd, LD, PL, lane16);
    if (layer == 2) {
      ws.open(p.WT[1], KBF, wave, NW, FT);
      ring.start(ws, lane16, KBF);
    } else {
      wd.open(p.WT[0], KBF, wave, NW, DT);
      ringd.start(wd, lane16, KBF);
    }
    __syncthreads();
    const float und = p.sc.p_undo[layer], up = p.sc.p_up[layer - 1];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int f = (wave + NW * t) * 16 + 4 * grp;
      const v4f wh = *reinterpret_cast<const v4f*>(&vec[3][f]);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        v4f x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float pre = opaque(layer == 2 ? p2[t][r][c] : p1[t][r][c]);
          const float sg = sigm(pre);
          const float s = sg * (1.0f + pre * (1.0f - sg));
          const float hb = fmaf(acc[t][r][c], und, layer == 2 ? wh[c] : p2[t][r][c]);
          if (layer == 2) p2[t][r][c] = hb;
          x[c] = hb * s * up;
        }
        put((r * 16 + col) * LD + f, x);
      }
    }
    __syncthreads();
  }
  // ---- dE/dD = p1 Th1^T
  const float und = p.sc.p_undo[0];
  auto put_row = [&](int f, int r, const v4f& x) {
    const int64_t i = row0 + r * 16 + col;
    if (i < n) *reinterpret_cast<v4f*>(desc + i * size_t(KP) + f * 16 + 4 * grp) = x * und;
  };
  {
    v4f acc[ND][RT];
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[t][r] = v4f{0.f, 0.f, 0.f, 0.f};
    product<ND, RT, KBF, D>(acc, wd, ringd, act_rd, LD, PL, lane16);
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
      for (int r = 0; r < RT; ++r) put_row(wave + NW * t, r, acc[t][r]);
  }
  if constexpr (kLeft > 0) {
#pragma unroll 1
    for (int u = wave; u < kLeft * RT; u += NW) {
      const int f = ND * NW + u / RT, r = u % RT;
      constexpr int D1 = blocks_in_flight(1);
      WStream<1> w1;
      WRing<1, D1> r1;
      w1.open(p.WT[0], KBF, f, 1, DT);
      r1.start(w1, lane16, KBF);
      v4f acc[1][1] = {{v4f{0.f, 0.f, 0.f, 0.f}}};
      product<1, 1, KBF, D1>(acc, w1, r1, act_rd + r * 16 * LD, LD, PL, lane16);
      put_row(f, r, acc[0][0]);
    }
  }
}

// A matrix W [K][N] (entry (k, n) at w[k sk + n sn]) in split fragment order:
// for feature tile T, block kb and lane l eight halves
// W[kb*32 + 8*(l/16) + i][T*16 + l%16] 2^e, the plane of the hi parts before
// that of the lo parts; rows past K and columns past N are zero.
__global__ void split_weights_kernel(const float* __restrict__ w, int K, int N, int sk, int sn,
                                     int blocks, int tiles, float scale, v8h* __restrict__ out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= tiles * blocks * 64) return;
  const int l = idx & 63, kb = (idx >> 6) % blocks, T = (idx >> 6) / blocks;
  const int n = T * 16 + (l & 15);
  v8h hi, lo;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int k = kb * 32 + 8 * (l >> 4) + i;
    const float x = (k < K && n < N ? w[size_t(k) * sk + size_t(n) * sn] : 0.0f) * scale;
    hi[i] = static_cast<_Float16>(x);
    lo[i] = static_cast<_Float16>(x - static_cast<float>(hi[i]));
  }
  v8h* dst = out + (size_t(T) * blocks + kb) * 128 + l;
  dst[0] = hi;
  dst[64] = lo;
}

template <int KP, int F, int RT, int NW>
int launch_chain_shape(const dpa4c_model* m, int64_t n, const int32_t* species, float* desc,
                       const float2* meta, double* e_atom, hipStream_t st) {
  ChainArgs a{};
  for (int t = 0; t < 3; ++t) {
    a.W[t] = m->wsplit[t];
    a.WT[t] = m->wsplitT[t];
    a.bias[t] = m->bias[t];
  }
  a.w_head = m->w_head;
  a.b_head = m->b_head;
  a.E_ref = m->E_ref;
  a.n_types1 = m->n_types + 1;
  a.sc = m->scales;
  const int64_t tiles = (n + 16 * RT - 1) / (16 * RT);
  hipLaunchKernelGGL((chain_kernel<KP, F, RT, NW>), dim3(static_cast<unsigned>(tiles)),
                     dim3(64 * NW), 0, st, a, n, species, desc, meta, e_atom);
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

int launch_split_weights(const float* w, int K, int N, int sk, int sn, int blocks, int tiles,
                         float scale, void* out, hipStream_t st) {
  const int total = tiles * blocks * 64;
  hipLaunchKernelGGL(split_weights_kernel, dim3((total + 255) / 256), dim3(256), 0, st, w, K, N,
                     sk, sn, blocks, tiles, scale, static_cast<v8h*>(out));
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

// Atoms per workgroup.  A workgroup of 16 RT atoms takes about (2 + RT) units
// of time (the weights stream past whatever RT is, the rest grows with it;
// full width, 65,536 atoms: 46, 58, 72 and 101 us a round for RT = 1 .. 4),
// and kSlots of them run at once, so the RT with the least rounds x (2 + RT)
// is taken: 16 atoms while every workgroup still has a slot, 64 for many
// rounds, and in between what leaves the last round least empty.  Fitted at
// full width, it holds at every other: over eleven sizes from 500 to 65,000
// atoms for each of the six profiles the stage with the RT taken is within 3
// percent of the best of the four (1 percent but for widths 256 at 8,112
// atoms).  In us for RT = 1 .. 4: width 96 at 24,624 atoms 42, 42, 47, 56 (2
// taken), width 192 at 16,384 56, 49, 58, 56 (2), width 256 at 46,464 208, 160,
// 153, 163 (3), width 384 at 11,760 163, 138, 108, 123 (3).
int launch_chain(const dpa4c_model* m, int64_t n, const int32_t* species, float* desc,
                 const float2* meta, double* e_atom, hipStream_t st) {
  return with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto f) {
    using P = decltype(p);
    constexpr int F = decltype(f)::value, KP = mlp_width(P::DOUT);
    // waves of a workgroup, and workgroups at once (by registers: eight waves
    // of up to 256 on each of the chip's 256 CUs)
    constexpr int NW = F == 384 ? 8 : F == 96 ? 2 : 4;
    constexpr int64_t kSlots = 256 * (8 / NW);
    int best = 1;
    int64_t least = INT64_MAX;
    for (int rt = 1; rt <= 4; ++rt) {
      const int64_t tiles = (n + 16 * rt - 1) / (16 * rt);
      const int64_t cost = (tiles + kSlots - 1) / kSlots * (2 + rt);
      if (cost < least) {
        least = cost;
        best = rt;
      }
    }
    switch (best) {
      case 1: return launch_chain_shape<KP, F, 1, NW>(m, n, species, desc, meta, e_atom, st);
      case 2: return launch_chain_shape<KP, F, 2, NW>(m, n, species, desc, meta, e_atom, st);
      case 3: return launch_chain_shape<KP, F, 3, NW>(m, n, species, desc, meta, e_atom, st);
      default: return launch_chain_shape<KP, F, 4, NW>(m, n, species, desc, meta, e_atom, st);
    }
  });
}

int ensure_mlp_rows(dpa4c_model* m, int64_t n) {
  Workspace& w = m->ws;
  const size_t each = mlp_row_bytes(m->D_out);
  int64_t rows = n < kMlpRows ? (n + 63) / 64 * 64 : kMlpRows;
  if (rows <= w.mlp_rows) return 0;
  if (rows > kMlpRowsLeast) {
    size_t free_b = 0, total_b = 0;
    DPA4C_HIP_TRY(hipMemGetInfo(&free_b, &total_b));
    if (free_b < rows * each + (size_t(8) << 30)) rows = kMlpRowsLeast;
    if (rows <= w.mlp_rows) return 0;
  }
  DevBuf grown;
  const int rc = grown.ensure(rows * each);
  if (rc) return w.mlp_rows > 0 ? 0 : rc;
  w.mlp_buf.release();
  w.mlp_buf = grown;
  w.mlp_rows = rows;
  return 0;
}

int launch_atoms(const dpa4c_model* m, int64_t n, const int32_t* species, const float* node,
                 float* node_grad, double* e_atom, float* desc_out, const MlpRows& mid,
                 hipStream_t st) {
  if (n <= 0) return 0;
  if (m->n_layers != 3 || !m->wsplit[0]) {
    set_error("the per-atom kernels need three hidden layers");
    return DPA4C_ERR_UNSUPPORTED;
  }
  const int64_t rows = mid.rows;
  if (rows <= 0) {
    set_error("no rows between the readout and the MLP");
    return DPA4C_ERR_OOM;
  }
  const int64_t ns = m->S + 2;
  float* desc = mid.at;
  float2* meta = reinterpret_cast<float2*>(desc + rows * mlp_width(m->D_out));
  for (int64_t c = 0; c < n; c += rows) {
    const int64_t k = n - c < rows ? n - c : rows;
    DPA4C_TRY(launch_readout(m, k, species + c, node + c * ns, desc, meta,
                             desc_out ? desc_out + c * m->D_out : nullptr, st));
    DPA4C_TRY(launch_chain(m, k, species + c, desc, meta, e_atom + c, st));
    DPA4C_TRY(launch_readout_vjp(m, k, node + c * ns, desc, node_grad + c * ns, st));
  }
  return 0;
}

}  // namespace dpa4c
