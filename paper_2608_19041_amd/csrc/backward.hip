// Fused backward edge kernel: readout vector-Jacobian product followed by
// the edge recomputation of Methods "Fused execution and backward
// recomputation".
//
// One wavefront per centre above kSplitRows centres (four per 256-thread
// workgroup, never waiting for each other), up to that many the four waves of a
// workgroup for one centre, an even share of each round's edges each.  For
// centre i a wave reads the node-state gradient [dE/dS0, dE/dS1, dE/dY]
// (from the readout VJP), revisits the edges of row i, recomputes the tabulated
// radial maps (value and derivative), the pair coefficients and the envelope,
// and writes
//     dE/dr_ij = (dE/drho) u + (I - u u^T)(dE/du) / rho,
// with  dE/drho = sum_lmc Ybar_lmc B_lm d(chi_l psi_c)/drho
//               + Sbar0 d(chi^2)/drho + Sbar1 d(chi^4)/drho,
//       dE/du   = sum_lmc Ybar_lmc chi_l psi_c dB_lm/du.
//
// Lane k of an edge group owns the channels c = k + LPE*j.  For the
// non-scalar degrees the channel c = k contributes
//     psi_k * Q_k(u),  Q_k(u) = sum_{l>=1, m} Ybar_lmk B_lm(u),
// and Q_k is a fixed polynomial per centre: v.u (degree one), u.W u (degree
// two, W symmetric), a cubic (degree three) and a quartic (degree four).  Its
// coefficients are formed once per centre, so per edge each lane evaluates
// one short polynomial and its gradient instead of every harmonic.  The LPE
// partial sums of an edge are combined with a fixed DPP butterfly.
//
// The row is taken in passes of 64 edges: each lane first forms one edge's
// geometry, envelope and table row into the wave's LDS slice, so the groups
// do not repeat that work per lane; with folded tables a group requests the
// table entries of its next edge before it evaluates the current one.
//
// The gradient of an edge goes to the skin position of the edge (the force
// assembly finds a reverse gradient there with one lookup), over the
// compact records, and keeps j in the fourth component; a pass's gradients
// are stored together once its edges have run.  The passes run from the end
// of the row to its start: a skin position is never before its compact
// slot, so a gradient never lands on a record still to be read.  Where four
// waves share the row, one wave's gradients may land on records of its round
// that another wave reads, so the workgroup waits until all four have read
// theirs before any stores (round_sync).  With VIR the lane that forms a
// gradient also adds -g_e (x) r_e (float64) to its group's slot in LDS; the
// slots are summed in group order into the atom's term W_i of the virial of
// Eq. (forces).
//
// What bounds it is the stream of table entries into the CUs, so it reads only
// what a slope needs (fold.hip): 8 bytes a channel where the forward kernel
// reads 12.  Backward over 24,000 water atoms (four tables, more than an L2)
// 251 -> 166 us, 31,250 alloy atoms (25 tables) 435 -> 301 us, a million copper
// atoms (one table) 5.86 -> 4.97 ms, 7,056 carbon atoms with the virial 89 ->
// 83 us.
#include <hip/hip_runtime.h>

#include "../../include/dpa4c.h"
#include "edge_math.h"
#include "launch.h"

namespace dpa4c {

namespace {

constexpr int kTeam = 256;
constexpr int kWaves = kTeam / kWave;

// Four waves per SIMD for the degree-three variants on folded tables (at most 128
// registers, none spilled; the virial's get there by themselves), three with the
// pair coefficients of the separable tables; degree four would spill and keeps
// its natural three, two on separable tables.
template <class P, bool FOLD, bool VIR>
constexpr int backward_min_waves() { return P::L < 4 && !VIR ? (FOLD ? 4 : 3) : 1; }

// W = 4 as in the forward kernel: up to kSplitRows centres the four waves of a
// workgroup share a row.
template <class P, bool FOLD, bool VIR, int W>
__global__ void __launch_bounds__(kTeam, (backward_min_waves<P, FOLD, VIR>())) backward_kernel(ModelDev md, int64_t n,
                                                         const int32_t* __restrict__ typ,
                                                         const int64_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ ecount,
                                                         float4* edge,
                                                         const int32_t* __restrict__ cskin,
                                                         const float* __restrict__ node_grad,
                                                         double* __restrict__ w_atom) {
  static_assert(P::R == 0 || P::R == 4, "pair modes: 0 or 4");
  constexpr int G = kWave / P::LPE;   // edge groups in a wave
  __shared__ double wv_all[kWaves][VIR ? G : 1][9];
  // per edge of a pass: (u, 1/rho), (tau, chi, dchi, table row), (j, a_j);
  // the per-edge terms that do not depend on the lane's channel: (chi^2,
  // d chi^2/drho, the S0/S1 term, the degree-three/four part of Q_0), the
  // gradient of that part with the edge's skin position (bits), and with
  // folded tables the quintic weights (e2, e3, f2, f3)
  __shared__ float4 geo_all[kWaves][kWave];
  __shared__ float4 rad_all[kWaves][kWave];
  __shared__ int2 ids_all[kWaves][kWave];
  __shared__ float4 sc_all[kWaves][kWave];
  __shared__ float4 cb_all[kWaves][kWave];
  __shared__ float4 wt_all[kWaves][FOLD ? kWave : 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int grp = lane / P::LPE;
  const int k = lane % P::LPE;
  double (*wv)[9] = wv_all[wave];
  float4* geo = geo_all[wave];
  float4* rad = rad_all[wave];
  int2* ids = ids_all[wave];
  float4* scl = sc_all[wave];
  float4* cub = cb_all[wave];
  float4* wts = wt_all[wave];
  const int T1 = md.n_types1;
  const float inv_delta = md.inv_delta;
  const int nf = md.fold_n;
  // ``typ`` holds species (clamped here) or, with folded tables, the folded
  // index of every atom
  auto type_of = [&](int64_t a) { return FOLD ? typ[a] : clamp_type(typ[a], T1); };

  constexpr int kRows = kWaves / W;   // centres of a workgroup
  static_assert(W == 1 || W == kWaves, "a row per wave or per workgroup");
  // the records of a round are read before its gradients are stored
  auto round_sync = [] {
    if constexpr (W == 1) wave_sync();
    else __syncthreads();
  };
  for (int64_t blk = xcd_block(blockIdx.x, gridDim.x); blk * kRows < n; blk += gridDim.x) {
    const int64_t i = blk * kRows + (W == 1 ? wave : 0);
    if (i >= n) break;
    const int ai = type_of(i);
    const float* gyr = node_grad + size_t(i) * P::NS;
    // per-centre coefficients in the lane's channel layout
    float gy0[P::CPL];
#pragma unroll
    for (int j = 0; j < P::CPL; ++j) gy0[j] = gyr[P::Y0 + j * P::LPE + k];
    float v1[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) v1[m] = gyr[P::Y1 + m * P::C1 + k];
    float M2[6];
    {
      float w[5];
#pragma unroll
      for (int m = 0; m < 5; ++m) w[m] = k < P::C2 ? gyr[P::Y2 + m * P::C2 + k] : 0.0f;
      quad_form2(w, M2);
    }
    // channel 0's degree-three (and four) polynomial and the normaliser
    // gradients, in every lane: the per-edge pass evaluates them once per
    // edge, and only lane 0 of a group adds them
    float G3[3][6];
    {
      float w[7];
#pragma unroll
      for (int m = 0; m < 7; ++m) w[m] = P::L >= 3 ? gyr[P::Y3 + m] : 0.0f;
      cubic_form3(w, G3);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int qq = 0; qq < 6; ++qq) G3[a][qq] = wave_uniform(G3[a][qq]);
    }
    float G4[P::L >= 4 ? 3 : 1][10];   // gradient of the degree-four polynomial
    if constexpr (P::L >= 4) {
      float w[9], pc[15];
#pragma unroll
      for (int m = 0; m < 9; ++m) w[m] = gyr[P::Y4 + m];
      quartic_coeffs4(w, pc);
      quartic_grad4(pc, G4);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int qq = 0; qq < 10; ++qq) G4[a][qq] = wave_uniform(G4[a][qq]);
    }
    const float gs0 = wave_uniform(gyr[0]), gs1 = wave_uniform(gyr[1]);
    const float m0 = k == 0 ? 1.0f : 0.0f;

    const int64_t b = row_ptr[i];
    const int cnt = ecount[i];
    if (VIR && k == 0)
      for (int c = 0; c < 9; ++c) wv[grp][c] = 0.0;
    const float* pair_base = FOLD ? md.ftab + size_t(ai) * nf * (md.n_rows + 1) * fold_pitch(P::C0, P::CPL)
                                  : md.pair + size_t(ai) * T1 * (P::C0 * P::PW);

    // Separable tables: the coefficients of the lane's channels for the pair of
    // a_i and the type of the group's last edge.  The edges of a pass are taken
    // by type, so they are read once for a run of edges: 3 KB of the 6 KB that
    // an edge streams at full width (13,718 atoms of eight species 328 -> 280
    // us).  The forward kernel, with less work to cover the loads, gained nothing
    // from it (287 -> 303 us, three waves on a SIMD instead of five) and reads
    // them for every edge.
    float pp[FOLD ? 1 : P::CPL][FOLD ? 1 : P::PW];
    int pp_of = -1;

    // Entry x of the pass's np (compact slot c0 + x of the row): the edge
    // gradient from its LDS entry and, with folded tables, the lane's table
    // entries ``T`` of that edge.
    auto edge_work = [&](int x, int np, const FoldRow<P::CPL, false>& T) {
      const float4 ge = geo[x], ra = rad[x];
      const float x_ = ge.x, y = ge.y, z = ge.z, inv_rho = ge.w;
      const float tau = ra.x, chi = ra.y, dchi = ra.z;
      const bool valid = x < np;
      const float4 sc = scl[x];
      // sum of dE/dY0 with the amplitudes, with their slopes, and (folded tables)
      // with the slopes of amplitude times envelope
      float a0 = 0.0f, b0 = 0.0f, d0 = 0.0f, psi0 = 0.0f, dpsi0 = 0.0f;
      if constexpr (FOLD) {
        // the polynomials of the table of the pair (a_i, a_j) (c4 and c5
        // below float32 resolution, not stored), power form; the float16 c2,
        // c3 enter through their scaled weights (one mixed-precision FMA
        // each).  The lane's first channel is an amplitude, whose value the
        // higher degrees need too; the others hold amplitude times envelope
        // (fold.hip) and only their slope enters, so their c0 stays in
        // memory.  Their coefficients are contracted with dE/dY0 first,
        // A_p = sum_j Ybar0_j c_pj, then one slope in tau; d/drho's 1/Delta
        // is applied once to the sums.
        const float4 wt = wts[x];
        const float e2 = wt.x, e3 = wt.y, f2 = wt.z, f3 = wt.w;
        psi0 = fmaf(T.c1[0], tau, T.c0[0]);
        psi0 = fmaf(half_lo(T.w[0]), e2, psi0);
        psi0 = fmaf(half_hi(T.w[0]), e3, psi0);
        dpsi0 = fmaf(half_lo(T.w[0]), f2, T.c1[0]);
        dpsi0 = fmaf(half_hi(T.w[0]), f3, dpsi0) * inv_delta;
        float A1 = 0.0f, A2 = 0.0f, A3 = 0.0f;
#pragma unroll
        for (int jj = 1; jj < P::CPL; ++jj) {
          A1 = fmaf(gy0[jj], T.c1[jj], A1);
          A2 = fmaf(gy0[jj], half_lo(T.w[jj]), A2);
          A3 = fmaf(gy0[jj], half_hi(T.w[jj]), A3);
        }
        a0 = gy0[0] * psi0;
        b0 = gy0[0] * dpsi0;
        d0 = fmaf(A3, f3, fmaf(A2, f2, A1)) * inv_delta;
      } else {
        const float t2 = tau * tau, t3 = t2 * tau, t4 = t2 * t2, t5 = t4 * tau;
        const float d1 = 2.0f * tau, d2 = 3.0f * t2, d3 = 4.0f * t3, d4 = 5.0f * t4;
        const int row = __float_as_int(ra.w), aj = ids[x].y;
        float q[4] = {0.f, 0.f, 0.f, 0.f}, dq[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (P::R > 0) {
          float c[6];
          load6(md.qtab + (size_t(row) * P::R + (k < P::R ? k : 0)) * 6, c);
          const float qk = c[0] + c[1] * tau + c[2] * t2 + c[3] * t3 + c[4] * t4 + c[5] * t5;
          const float dqk = (c[1] + c[2] * d1 + c[3] * d2 + c[4] * d3 + c[5] * d4) * inv_delta;
#pragma unroll
          for (int mu = 0; mu < 4; ++mu) {
            q[mu] = __shfl(qk, mu, P::LPE);
            dq[mu] = __shfl(dqk, mu, P::LPE);
          }
        }
        if (aj != pp_of) {
          const float* pc = pair_base + size_t(aj) * (P::C0 * P::PW);
#pragma unroll
          for (int jj = 0; jj < P::CPL; ++jj)
#pragma unroll
            for (int v = 0; v < P::PW; v += 2) {
              const float2 a =
                  *reinterpret_cast<const float2*>(pc + (jj * P::LPE + k) * P::PW + v);
              pp[jj][v] = a.x;
              pp[jj][v + 1] = a.y;
            }
          pp_of = aj;
        }
        const float* gt = md.gtab + size_t(row) * (P::C0 * 6);
#pragma unroll
        for (int jj = 0; jj < P::CPL; ++jj) {
          float c[6];
          load6(gt + (jj * P::LPE + k) * 6, c);
          const float gv = c[0] + c[1] * tau + c[2] * t2 + c[3] * t3 + c[4] * t4 + c[5] * t5;
          const float gd = (c[1] + c[2] * d1 + c[3] * d2 + c[4] * d3 + c[5] * d4) * inv_delta;
          float psi = pp[jj][0] * gv + pp[jj][1];
          float dpsi = pp[jj][0] * gd;
          if constexpr (P::R > 0) {
            psi += pp[jj][2] * q[0] + pp[jj][3] * q[1] + pp[jj][4] * q[2] + pp[jj][5] * q[3];
            dpsi += pp[jj][2] * dq[0] + pp[jj][3] * dq[1] + pp[jj][4] * dq[2] + pp[jj][5] * dq[3];
          }
          a0 += gy0[jj] * psi;
          b0 += gy0[jj] * dpsi;
          if (jj == 0) {
            psi0 = psi;
            dpsi0 = dpsi;
          }
        }
      }
      // Q_k(u) and its gradient: the lane's degree-one and degree-two parts
      // here, channel 0's degree-three (and four) part from the pass
      float gq[3];
      gq[0] = M2[0] * x_ + M2[3] * y + M2[5] * z;
      gq[1] = M2[3] * x_ + M2[1] * y + M2[4] * z;
      gq[2] = M2[5] * x_ + M2[4] * y + M2[2] * z;
      const float4 cb = cub[x];
      // Q = v.u + (1/2) u.M u + (1/3) u.grad P3 + (1/4) u.grad P4 (Euler's
      // relation per degree)
      const float Q = (v1[0] * x_ + v1[1] * y + v1[2] * z) +
                      0.5f * (gq[0] * x_ + gq[1] * y + gq[2] * z) + m0 * sc.w;
      const float chi2 = sc.x, dchi2 = sc.y;
      float drho = dchi * a0 + chi * b0 + d0 + Q * (dchi2 * psi0 + chi2 * dpsi0) + m0 * sc.z;
      const float wu = chi2 * psi0;
      float dux = wu * (v1[0] + gq[0] + m0 * cb.x);
      float duy = wu * (v1[1] + gq[1] + m0 * cb.y);
      float duz = wu * (v1[2] + gq[2] + m0 * cb.z);
      if (!valid) drho = dux = duy = duz = 0.0f;
      drho = group_sum<P::LPE>(drho);
      dux = group_sum<P::LPE>(dux);
      duy = group_sum<P::LPE>(duy);
      duz = group_sum<P::LPE>(duz);
      if (valid && k == 0) {
        const float udu = x_ * dux + y * duy + z * duz;
        const float gx = drho * x_ + (dux - udu * x_) * inv_rho;
        const float gy_ = drho * y + (duy - udu * y) * inv_rho;
        const float gz = drho * z + (duz - udu * z) * inv_rho;
        // to the entry's LDS slot (its geometry is no longer needed): the
        // pass's gradients are stored together once every edge has run
        geo[x] = make_float4(gx, gy_, gz, __int_as_float(ids[x].x));
        if (VIR) {   // LDS adds to the group's own slot: one writer, program order
          const float rho = __builtin_amdgcn_rcpf(inv_rho);   // hardware reciprocal, 1 ulp
          const float ga[3] = {gx, gy_, gz};
          const float rb[3] = {x_ * rho, y * rho, z * rho};
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int c = 0; c < 3; ++c) atomicAdd(&wv[grp][3 * a + c], -(double(ga[a]) * double(rb[c])));
        }
      }
    };
    // the lane's folded table entries of entry x of the pass
    auto load_rows = [&](int x, FoldRow<P::CPL, false>& T) {
      load_fold_row<P::LPE, P::CPL, false>(pair_base, __float_as_uint(rad[x].w), k, T);
    };

    // The row in passes of 64 edges: each lane first reads one record and
    // forms its edge's geometry, envelope and table row into the wave's LDS
    // slice (entries past the row get chi = 0 and table row 0), then the
    // groups take the pass's edges.
    const int rounds = (cnt + W * kWave - 1) / (W * kWave);
    // edges of a wave in a round: 64, or an even share of the row
    const int share = W == 1 ? kWave : rounds > 0 ? (cnt + W * rounds - 1) / (W * rounds) : 0;
    for (int rd = rounds - 1; rd >= 0; --rd) {
      const int c0 = (rd * W + (W == 1 ? 0 : wave)) * share;
      const int np = cnt - c0 < share ? (cnt > c0 ? cnt - c0 : 0) : share;
      {
        float4 ge = make_float4(0.f, 0.f, 0.f, 1.0f), ra = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 sc = make_float4(0.f, 0.f, 0.f, 0.f), cb = sc, wt = sc;
        int2 id = make_int2(0, 0);
        int sk = 0;
        if (lane < np) {
          const float4 rec = edge[b + c0 + lane];
          sk = cskin[b + c0 + lane];
          const EdgeGeom g = edge_geom(rec.x, rec.y, rec.z);
          float chi, dchi, tau;
          envelope(g.rho, md.r_c, md.inv_rc, &chi, &dchi);
          const int row = table_row<FOLD>(g.rho, inv_delta, md.n_rows, &tau);
          const int j = __float_as_int(rec.w);
          const int aj = type_of(j);
          ge = make_float4(g.ux, g.uy, g.uz, g.inv_rho);
          ra = make_float4(tau, chi, dchi,
                           FOLD ? __uint_as_float(fold_offset<P::C0, P::CPL>(aj * (md.n_rows + 1) + row))
                                : __int_as_float(row));
          id = make_int2(j, aj);
          const float x_ = g.ux, y = g.uy, z = g.uz;
          const float chi2 = chi * chi, dchi2 = 2.0f * chi * dchi;
          float c3[3] = {0.f, 0.f, 0.f};
          if constexpr (P::L >= 3) {
            const float mono[6] = {x_ * x_, x_ * y, x_ * z, y * y, y * z, z * z};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
              for (int qq = 0; qq < 6; ++qq) c3[a] += G3[a][qq] * mono[qq];
            }
          }
          float c4[3] = {0.f, 0.f, 0.f};   // grad P4
          if constexpr (P::L >= 4) {
            float mono3[10];
            cubic_monomials(x_, y, z, mono3);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
              for (int qq = 0; qq < 10; ++qq) c4[a] += G4[a][qq] * mono3[qq];
            }
          }
          float q0 = (1.0f / 3.0f) * (c3[0] * x_ + c3[1] * y + c3[2] * z);
          if constexpr (P::L >= 4) q0 += 0.25f * (c4[0] * x_ + c4[1] * y + c4[2] * z);
          sc = make_float4(chi2, dchi2, gs0 * dchi2 + gs1 * 2.0f * chi2 * dchi2, q0);
          cb = make_float4(c3[0] + c4[0], c3[1] + c4[1], c3[2] + c4[2], __int_as_float(sk));
          if constexpr (FOLD) {
            const float t2 = tau * tau, t3 = t2 * tau;
            wt = make_float4(md.c_inv[0] * t2, md.c_inv[1] * t3, md.c_inv[0] * (2.0f * tau),
                             md.c_inv[1] * (3.0f * t2));
          }
        }
        int at = lane;
        if constexpr (!FOLD) {   // by type, then the entries past the pass
          const int rank = type_rank(lane < np, id.y);
          at = lane < np ? rank : lane;
        }
        geo[at] = ge;
        rad[at] = ra;
        ids[at] = id;
        scl[at] = sc;
        cub[at] = cb;
        if constexpr (FOLD) wts[at] = wt;
      }
      round_sync();
      if constexpr (FOLD) {
        // the table entries of a group's next edge are requested before its
        // current edge is evaluated (two register sets, used in turn)
        FoldRow<P::CPL, false> TA, TB;
        load_rows(grp, TA);
        for (int base = 0; base < np; base += 2 * G) {
          if (base + G < np) load_rows(base + G + grp, TB);
          edge_work(base + grp, np, TA);
          if (base + G >= np) break;
          if (base + 2 * G < np) load_rows(base + 2 * G + grp, TA);
          edge_work(base + G + grp, np, TB);
        }
      } else {
        // an even share of the pass for every group, one run of types each
        const int per = (np + G - 1) / G;
        for (int x = 0; x < per; ++x) edge_work(grp * per + x, np, {});
      }
      wave_sync();
      // every record of the pass was read before its edges ran
      if (lane < np) edge[b + __float_as_int(cub[lane].w)] = geo[lane];
      wave_sync();   // the LDS entries are rewritten by the next pass
    }
    if (VIR) {
      round_sync();
      if (lane < 9 && (W == 1 || wave == 0)) {
        double s = 0.0;
        for (int q = 0; q < W * G; ++q) s += W == 1 ? wv[q][lane] : wv_all[q / G][q % G][lane];
        w_atom[9 * i + lane] = s;
      }
      round_sync();   // the slots are cleared for the next row
    }
  }
}

template <class P>
int launch(const dpa4c_model* m, int64_t n, const int32_t* species, const int32_t* fidx,
           const int64_t* row_ptr, const int32_t* ecount, float4* edge, const int32_t* cskin,
           const float* node_grad, double* w_atom, hipStream_t st) {
  const bool split = n <= kSplitRows;   // a workgroup per centre, else a wave
  int64_t blocks = split ? n : (n + kWaves - 1) / kWaves;
  blocks = blocks < 65536 ? blocks : 65536;
  if (blocks < 1) return 0;
  const int32_t* typ = fidx ? fidx : species;
  auto go = [&](auto fold, auto vir) {
    constexpr bool F = decltype(fold)::value, V = decltype(vir)::value;
    const dim3 grid(static_cast<unsigned>(blocks)), block(kTeam);
    if (split)
      hipLaunchKernelGGL((backward_kernel<P, F, V, kWaves>), grid, block, 0, st, m->dev(), n, typ,
                         row_ptr, ecount, edge, cskin, node_grad, w_atom);
    else
      hipLaunchKernelGGL((backward_kernel<P, F, V, 1>), grid, block, 0, st, m->dev(), n, typ,
                         row_ptr, ecount, edge, cskin, node_grad, w_atom);
  };
  if (fidx && w_atom) go(std::true_type{}, std::true_type{});
  else if (fidx) go(std::true_type{}, std::false_type{});
  else if (w_atom) go(std::false_type{}, std::true_type{});
  else go(std::false_type{}, std::false_type{});
  DPA4C_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

int launch_backward(const dpa4c_model* m, int64_t n, const int32_t* species, const int32_t* fidx,
                    const int64_t* row_ptr, const int32_t* ecount, float4* edge,
                    const int32_t* cskin, const float* node_grad, double* w_atom, hipStream_t st) {
  const int rc = with_profile(m->C0, m->L, m->R, m->F, [&](auto p, auto) {
    return launch<decltype(p)>(m, n, species, fidx, row_ptr, ecount, edge, cskin, node_grad,
                               w_atom, st);
  });
  if (rc == kNoProfile) {
    set_error("backward: profile not compiled");
    return DPA4C_ERR_UNSUPPORTED;
  }
  return rc;
}

}  // namespace dpa4c
