// Discrete adjoint of the fixed-step RK4 map, one reverse step at a time.
//
// Forward step (joint state y = (m, a), f = (torque, cavity RHS)):
//   k1 = f(y1), y2 = y + h/2 k1, k2 = f(y2), y3 = y + h/2 k2, k3 = f(y3),
//   y4 = y + h k3, k4 = f(y4), z = y + h/6 (k1 + 2 k2 + 2 k3 + k4),
//   m' = z_m / |z_m| on magnetic cells, a' = z_a.
// Reverse step, given lambda' = dL/dy':
//   lambda_z = (I - m' m'^T) lambda'_m / |z_m| (a: unchanged),
//   lambda_y = lambda_z, lambda_k4 = h/6 lambda_z, then for s = 4..1:
//   mu_s = J_f(y_s)^T lambda_ks (+ parameter gradients), lambda_y += mu_s,
//   lambda_k(s-1) = h w_(s-1)/6 lambda_z + c_s mu_s  (w = 1,2,2,1; c = h/2, h/2, h).
// The stage inputs y_s, |z_m| and a_s were recorded by the forward kernels
// while the segment was recomputed from its checkpoint.
//
// Adaptive (DP45) runs are reversed as the replay of their accepted steps
// (the step sizes h held): z = y + h sum_{j<=6} b_j k_j with stage inputs
// y_s = y + h sum_{j<s} a_sj k_j.  Reverse: lambda_z as above, lambda_y =
// lambda_z, then for s = 6..1: mu_s = J_f(y_s)^T lambda_ks, lambda_y += mu_s,
// with lambda_ks = h (b_s lambda_z + sum_{q>s} a_qs mu_q); the mu_q of
// stages 3..6 are kept until the earlier stages have used them.
// Stage numbering of the launches: RK4 stages 1..4 and 5 for the step
// start; DP45 stages 1..6 and 7 for the step start.
//
// Per stage the VJP is split in two cell kernels around the demag
// convolution of lambda_B (the tensor is symmetric and even, so the same
// FFT convolution is its own transpose):
//   A: lambda_B = dtorque/dB^T lambda_k, the direct torque term, the m^-
//      term, partial sums for the cavity and the parameters, grad u_n;
//   B: exchange / anisotropy / demag / intersublattice transposes applied
//      to lambda_B, then the RK bookkeeping above.
#include "mm_internal.h"
#include "kernels_common.h"
#include "launch.h"
#include "xrows.h"

namespace mmk {

// The sums of stage kernel A over a workgroup.  Two values at a time go
// through the butterfly of a wavefront (wave_sum2), the wave sums of up to four
// modes meet in LDS, and one thread a sum adds them in wavefront order.  With
// a butterfly for each of the 16 sums of a four-mode film and two barriers a
// mode A took 28.4 us on 128x128x32 cells, 26.1 so; of its 140 bytes a cell 64
// are the update of grad u in double.
struct AdjSums {
  static constexpr int MODES = 4, NW = MMI_WG / 64;
  static constexpr int ROWS = 3 * MODES + 4;         // per mode fb, Re m^-, Im m^-; then alpha, B0
  double* sh;
  __device__ __forceinline__ void put2(int row0, int row1, double a, double b) const {
    const double w = wave_sum2(a, b);
    const int lane = threadIdx.x & 63;
    if ((lane & 31) == 0) sh[(lane ? row1 : row0) * NW + (threadIdx.x >> 6)] = w;
  }
  // sum of row threadIdx.x
  __device__ __forceinline__ double row() const {
    double r = sh[threadIdx.x * NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) r += sh[threadIdx.x * NW + w];
    return r;
  }
};

// size of the step being reversed: fixed (RK4) or the logged one (DP45)
template <class CtlPtr>
__device__ __forceinline__ double adj_step(const InstDesc& D, CtlPtr C) {
  if (D.method != MMI_DP45) return C->adj_h;
  return fabs(gbl(D.hlog)[C->adj_base + C->rec_index]);
}

// --------------------------------------------------------- cavity part
// RK4 (DP = false): ST = 5 step start, ST = 4..1 after the stage kernels of
// that stage.  DP45 (DP = true): ST = 7 step start, ST = 6..1.
// It needs the partial sums of stage kernel A and nothing of stage kernel B,
// which touches none of what it writes (but for the index of the recorded
// step at the end of a DP45 step), so one workgroup per instance runs it
// beside B's own, ahead of them in B's launch; the step start runs beside
// k_adj_start.  As launches of their own, each slot summed by the whole
// workgroup in turn, these took 27 us a stage on the 128x128x32 film (1024
// records, four modes) and 4 us and a launch on small grids: its reverse step
// 0.62 vs 0.74 ms.  Behind B's workgroups and with the modes one after the
// other in one lane (their mu_a in scratch memory, which the whole kernel then
// carries) it was what B waited for: B of the film 28.5 vs 23.5 us.
template <bool DP, int ST>
__device__ void adj_cav(const InstDesc* __restrict__ descs, int inst, double* tot) {
  constexpr bool kStart = DP ? ST == 7 : ST == 5;
  const InstDesc& D = descs[inst];
  InstCtl* C = D.ctl;
  if (C->done) return;
  const int N = D.N;
  const double h = adj_step(D, C);
  if (!kStart) {
    // every slot is summed in a fixed order: a wavefront takes slots in turn,
    // lane l records l, l + 64, ... (eight in flight), a butterfly joins them
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const MMG double* P = gbl(D.partials);
    for (int k = wv; k < 3 * N + 4; k += MMI_WG / 64) {
      const int q = k < N ? MMI_ASLOT_FB + k : k < 3 * N ? MMI_ASLOT_MM + (k - N) : MMI_ASLOT_ALPHA + (k - 3 * N);
      double v = 0.0;
      int w = lane;
      for (; w + 7 * 64 < D.nwg; w += 8 * 64) {
        double p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = P[(size_t)(w + u * 64) * MMI_PSTRIDE + q];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += p[u];
      }
      for (; w < D.nwg; w += 64) v += P[(size_t)w * MMI_PSTRIDE + q];
      v = wave_sum(v);
      if (lane == 0) tot[q] = v;
    }
    __syncthreads();
  }
  // then lane n of the first wavefront carries mode n
  if (threadIdx.x >= 64) return;
  const int n = threadIdx.x;
  const bool mode = n < N;
  if (kStart) {
    if (!mode) return;
    const double wl = DP ? h * DPCoef::b6 : h / 6.0;
    // a loss on the trace: its derivative at the end of the step being reversed
    const double* q = !DP && D.dla_trace ? D.dla_trace + ((size_t)(C->adj_base + C->rec_index + 1) * N + n) * 2 : nullptr;
    for (int r = 0; r < 2; ++r) {
      if (q) C->la[n][r] += q[r];
      C->lza[n][r] = C->la[n][r];
      C->lka[n][r] = wl * C->la[n][r];
    }
  } else {
    const int ri = C->rec_index;
    if (n == 0) {
      C->grad_alpha += tot[MMI_ASLOT_ALPHA];
      for (int c = 0; c < 3; ++c) C->grad_B0[c] += tot[MMI_ASLOT_B0 + c];
      if (ST == 1) C->rec_index = ri - 1;
    }
    if (!mode) return;
    const double* as = D.rec_a + (((size_t)ri * D.rec_nstg + (ST - 1)) * N + n) * 2;
    const double scale = D.inv_ngeo / (double)D.S;
    const double cst = (ST == 4) ? h : 0.5 * h;
    const double wprev = h * (ST == 2 ? 1.0 : 2.0) / 6.0;
    const double c = D.cphi[n], s = D.sphi[n], g = D.g[n];
    const double lr = C->lka[n][0], li = C->lka[n][1];
    const double ar = as[0], ai = as[1];
    const double fb = tot[MMI_ASLOT_FB + n];
    const double mr = tot[MMI_ASLOT_MM + 2 * n] * scale, mi = tot[MMI_ASLOT_MM + 2 * n + 1] * scale;
    // dF/dg = (s + i c) m^- ; feedback h0 = 2 g / gamma with Re[e^{-i Phi} a] = c ar + s ai
    const double fr = s * mr - c * mi, fi = s * mi + c * mr;
    C->grad_g[n] += lr * fr + li * fi + fb * (2.0 / D.gamma) * (c * ar + s * ai);
    // mu_a = conj(-kappa - i w) lambda_ka + h0 fb (c, s)
    const double w = D.omega[n], kp = D.kappa[n];
    double mu[2] = {-kp * lr - w * li + D.h0[n] * fb * c, w * lr - kp * li + D.h0[n] * fb * s};
    if (D.kerr_on) {
      // transpose of the Jacobian of -i K |a|^2 a at the stage amplitude
      const double K = D.kerr[n];
      const double q = K * (ar * ar + ai * ai), x = 2.0 * K * ar * ai;
      mu[0] += lr * x - li * (q + 2.0 * K * ar * ar);
      mu[1] += lr * (q + 2.0 * K * ai * ai) - li * x;
    }
    if (D.param_on) {
      // transpose of the Jacobian of -i Lam conj(a), Lam = lam e^{-2 i wp t}
      // at the stage time: [[Li, -Lr], [-Lr, -Li]] (symmetric)
      const double ts = DP ? gbl(D.rec_t)[ri] + DPCoef::c(ST) * h
                           : C->adj_t0 + (double)ri * h + (ST == 1 ? 0.0 : ST == 4 ? h : 0.5 * h);
      double sn, cs;
      sincos(2.0 * D.par_wp[n] * ts, &sn, &cs);
      const double Lr = D.par_re[n] * cs + D.par_im[n] * sn;
      const double Li = D.par_im[n] * cs - D.par_re[n] * sn;
      mu[0] += Li * lr - Lr * li;
      mu[1] -= Lr * lr + Li * li;
    }
    if (D.jcpl_on)
      // with direct mode coupling mu_a reads the lambda_ka of all modes (the
      // stores below come after these loads for the whole wavefront)
      for (int q = 0; q < N; ++q) {
        // -i sum_q J_qn a_n in the equation of mode q, J symmetric
        mu[0] -= D.jcpl[q][n] * C->lka[q][1];
        mu[1] += D.jcpl[q][n] * C->lka[q][0];
      }
    __builtin_amdgcn_wave_barrier();
    for (int r = 0; r < 2; ++r) {
      C->la[n][r] += mu[r];
      if (!DP) {
        if (ST > 1) C->lka[n][r] = wprev * C->lza[n][r] + cst * mu[r];
      } else if (ST > 1) {
        // lambda_ka(ST-1) = h (b_(ST-1) lambda_za + sum_{q>=ST} a_(q,ST-1) mu_a,q)
        if (ST >= 3) C->lmua[ST - 1][n][r] = mu[r];
        double acc = DPCoef::b(ST - 1) * C->lza[n][r] + DPCoef::a(ST, ST - 1) * mu[r];
        for (int q = ST + 1; q <= 6; ++q) acc += DPCoef::a(q, ST - 1) * C->lmua[q - 1][n][r];
        C->lka[n][r] = h * acc;
      }
    }
  }
  // adjoint of m^- for the next stage kernel A: conj(i g e^{-i Phi}) lambda_ka
  if (ST >= 2) {
    const double c = D.cphi[n], s = D.sphi[n], g = D.g[n];
    const double lr = C->lka[n][0], li = C->lka[n][1];
    // conj(g (s + i c)) = g (s - i c)
    C->lmm[n][0] = g * (s * lr + c * li);
    C->lmm[n][1] = g * (s * li - c * lr);
  }
}

// the same as a launch of its own (the last stage of a DP45 step)
template <bool DP, int ST>
__global__ __launch_bounds__(MMI_WG) void k_adj_cav(const InstDesc* __restrict__ descs, int count) {
  __shared__ double tot[MMI_PSTRIDE];
  if ((int)blockIdx.x < count) adj_cav<DP, ST>(descs, blockIdx.x, tot);
}

// ---------------------------------------------------------- step start
// lambda_z from the step-end adjoint (held in lam_y), lambda_y = lambda_z,
// lambda_k4 = h/6 lambda_z.
template <bool DP>
__global__ __launch_bounds__(MMI_WG) void k_adj_start(const InstDesc* __restrict__ descs,
                                                      const int* __restrict__ wg_inst, int nblocks, int count) {
  __shared__ double tot[MMI_PSTRIDE];
  const int lead = (int)gridDim.x - nblocks;
  if ((int)blockIdx.x < lead) {
    if ((int)blockIdx.x < count) adj_cav<DP, DP ? 7 : 5>(descs, blockIdx.x, tot);
    return;
  }
  const int lblk = xcd_block(nblocks, lead);
  const InstDesc& D = descs[wg_inst[lblk]];
  const MMG InstCtl* __restrict__ C = gbl(D.ctl);
  if (C->done) return;
  const int nc = D.ncell, S = D.S;
  const int i = wg_cell(D, lblk - D.wg0);
  if (i >= nc) return;
  const bool mag = !D.has_geom || gbl(D.geom)[i];
  const size_t vec = (size_t)3 * S * nc;
  const int ri = C->rec_index;
  const MMG float* Yn = gbl(D.rec_m) + ((size_t)(ri + 1) * D.rec_nstg) * vec;   // state after the step
  MMG float* const lam_y = gbl(D.lam_y);
  MMG float* const lam_z = gbl(D.lam_z);
  MMG float* const lam_k = gbl(D.lam_k);
  // weight of the last stage in the step-end combination: h/6 (RK4), h b_6 (DP45)
  const float c6 = (float)(D.method == MMI_DP45 ? adj_step(D, C) * DPCoef::b6 : C->adj_h / 6.0);
  for (int s = 0; s < S; ++s) {
    float l[3], y[3];
    for (int c = 0; c < 3; ++c) {
      l[c] = lam_y[(s * 3 + c) * nc + i];
      y[c] = Yn[(s * 3 + c) * nc + i];
    }
    float z[3] = {0.f, 0.f, 0.f};
    if (mag) {
      const float inv = 1.0f / gbl(D.rec_norm)[(size_t)ri * S * nc + s * nc + i];
      const float d = l[0] * y[0] + l[1] * y[1] + l[2] * y[2];
      for (int c = 0; c < 3; ++c) z[c] = (l[c] - y[c] * d) * inv;
    }
    for (int c = 0; c < 3; ++c) {
      const int idx = (s * 3 + c) * nc + i;
      lam_z[idx] = z[c];
      lam_y[idx] = z[c];
      lam_k[idx] = c6 * z[c];
    }
  }
}

// ------------------------------------------------------------ stage A
template <int ST>
__global__ __launch_bounds__(MMI_WG) __attribute__((amdgpu_num_sgpr(80))) void k_adj_a(const InstDesc* __restrict__ descs,
                                                  const int* __restrict__ wg_inst,
                                                  const float2* __restrict__ tw) {
  __shared__ double sh[AdjSums::ROWS * (MMI_WG / 64)];
  extern __shared__ float2 xl[];
  const int lblk = xcd_block();
  const InstDesc& D = descs[wg_inst[lblk]];
  const MMG InstCtl* __restrict__ C = gbl(D.ctl);
  if (C->done) return;
  const int lw = lblk - D.wg0;
  const int nc = D.ncell, S = D.S, N = D.N;
  const int i = wg_cell(D, lw);
  const bool valid = i < nc;
  const bool mag = valid && (!D.has_geom || gbl(D.geom)[i]);
  const int ri = C->rec_index;
  const Src src = stage_src(D, C, MMI_ADJ, ST);
  const MMG double* as = gbl(D.rec_a) + ((size_t)ri * D.rec_nstg + (ST - 1)) * N * 2;
  const MMG float* const u_ = gbl(D.u);
  MMG float* const lam_B = gbl(D.lam_B);
  int x = 0, yy = 0, zz = 0;
  if (valid) cell_xyz(D, i, x, yy, zz);

  float m[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
  if (valid)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (s < S)
#pragma unroll
        for (int c = 0; c < 3; ++c) m[s][c] = src.ld((s * 3 + c) * nc + i);

  // feedback value of this stage: sum_n h0_n u_n Re[e^{-i Phi_n} a_n]
  float fb = 0.f;
  if (mag)
    for (int n = 0; n < N; ++n) {
      const float b = (float)(D.h0[n] * (D.cphi[n] * as[2 * n] + D.sphi[n] * as[2 * n + 1]));
      fb = fmaf(b, D.profiled ? gat(u_ + (size_t)n * nc, i) : 1.f, fb);
    }
  const float gl = D.gl, al = D.alpha;
  const float dga = 2.f * al / (1.f + al * al);   // -d ln(gamma')/d alpha
  const float wmm = (float)(D.inv_ngeo / (double)S);
  double galpha = 0.0, gb0x = 0.0, gb0y = 0.0, gb0z = 0.0;
  float lbx[2] = {0.f, 0.f};
  float lb0[3] = {0.f, 0.f, 0.f};   // field adjoint of sublattice 0 (the R2C input)
  float mux[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
  // demag field of this stage input: recorded during the segment recompute,
  // else from the convolution just enqueued
  float bdv[3] = {0.f, 0.f, 0.f};
  const bool bd_recorded = D.rec_bd != nullptr;
  if (bd_recorded && valid) {
    const MMG float* RB = gbl(D.rec_bd) + ((size_t)ri * D.rec_nstg + (ST - 1)) * (size_t)(3 * nc);
#pragma unroll
    for (int c = 0; c < 3; ++c) bdv[c] = gat(RB, c * nc + i);
  }
  if (mag) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (s >= S) continue;
      float B[3];
      field_at(D, src, i, x, yy, zz, m, s, fb, D.demag == 2, B, bdv, bd_recorded);
      const float* ms = m[s];
      float l[3];
      for (int c = 0; c < 3; ++c) l[c] = gat(gbl(D.lam_k), (s * 3 + c) * nc + i);
      float P[3], Q[3], lm[3], t1[3], t2[3], t3[3], lB[3];
      cross3(ms, B, P);
      cross3(ms, P, Q);
      cross3(l, ms, lm);          // lambda x m
      cross3(lm, ms, t1);         // (lambda x m) x m
      for (int c = 0; c < 3; ++c) lB[c] = -gl * (lm[c] + al * t1[c]);
      cross3(B, l, t1);           // B x lambda
      cross3(P, l, t2);           // P x lambda
      cross3(B, lm, t3);          // B x (lambda x m)
      for (int c = 0; c < 3; ++c) mux[s][c] = -gl * (t1[c] + al * (t2[c] + t3[c]));
      // dL/dalpha: lambda . (-(2a/(1+a^2)) tau - gamma' Q), tau = -gamma' (P + a Q)
      float ga = 0.f;
      for (int c = 0; c < 3; ++c) {
        const float tau = -gl * (P[c] + al * Q[c]);
        ga += l[c] * (-dga * tau - gl * Q[c]);
      }
      galpha += ga;
      gb0x += lB[0];
      gb0y += lB[1];
      gb0z += lB[2];
      lbx[s] = lB[0];
      for (int c = 0; c < 3; ++c) gat(lam_B, (s * 3 + c) * nc + i) = lB[c];
      if (s == 0)
        for (int c = 0; c < 3; ++c) lb0[c] = lB[c];
    }
  } else if (valid) {
    for (int s = 0; s < S; ++s)
      for (int c = 0; c < 3; ++c) lam_B[(s * 3 + c) * nc + i] = 0.f;
  }
  // m^- transpose, the gradient of the mode profiles and the sums
  const AdjSums sums{sh};
  MMG double* const rec = gbl(D.partials) + (size_t)lw * MMI_PSTRIDE;
  sums.put2(3 * AdjSums::MODES, 3 * AdjSums::MODES + 1, galpha, gb0x);
  sums.put2(3 * AdjSums::MODES + 2, 3 * AdjSums::MODES + 3, gb0y, gb0z);
  int n0 = 0;
  do {
    if (n0) __syncthreads();
    double fbs[AdjSums::MODES] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < AdjSums::MODES; ++q) {
      const int n = n0 + q;
      if (n >= N) break;
      const float u = D.profiled ? (valid ? gat(u_ + (size_t)n * nc, i) : 0.f) : 1.f;
      const float lr = (float)C->lmm[n][0], li = (float)C->lmm[n][1];
      double fbn = 0.0, mr = 0.0, mi = 0.0, gu = 0.0;
      if (mag) {
        MMG double* const g = D.grad_u ? gbl(D.grad_u) + (size_t)n * nc : nullptr;
        const double g0 = g ? gat(g, i) : 0.0;
        const float arn = (float)as[2 * n], ain = (float)as[2 * n + 1];
        const float fbw = (float)(D.h0[n] * (D.cphi[n] * arn + D.sphi[n] * ain));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          if (s >= S) continue;
          const float cs = D.csign[s];
          mux[s][0] += wmm * cs * u * lr;
          mux[s][1] -= wmm * cs * u * li;
          fbn += (double)(cs * lbx[s] * u);
          mr += (double)(cs * m[s][0] * u);
          mi -= (double)(cs * m[s][1] * u);
          gu += (double)(cs * (lbx[s] * fbw + wmm * (lr * m[s][0] - li * m[s][1])));
        }
        if (g) gat(g, i) = g0 + gu;
      }
      fbs[q] = fbn;
      sums.put2(3 * q + 1, 3 * q + 2, mr, mi);
      if (q & 1) sums.put2(3 * (q - 1), 3 * q, fbs[q - 1], fbs[q]);
      else if (n == N - 1) sums.put2(3 * q, 3 * q + 3, fbs[q], 0.0);   // (row 3 q + 3 is of no mode)
    }
    __syncthreads();
    const int k = threadIdx.x, q = k / 3, r = k - 3 * q;
    if (k < 3 * AdjSums::MODES) {
      if (n0 + q < N) rec[r == 0 ? MMI_ASLOT_FB + n0 + q : MMI_ASLOT_MM + 2 * (n0 + q) + r - 1] = sums.row();
    } else if (n0 == 0 && k < AdjSums::ROWS) {
      rec[MMI_ASLOT_ALPHA + k - 3 * AdjSums::MODES] = sums.row();
    }
    n0 += AdjSums::MODES;
  } while (n0 < N);
  if (valid)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (s < S)
#pragma unroll
        for (int c = 0; c < 3; ++c) gat(gbl(D.mu), (s * 3 + c) * nc + i) = mux[s][c];
  if (D.xfused) {
    // R2C of the field adjoint of this workgroup's x-rows: the X rows of its
    // convolution (no separate x-forward pass)
    const XRows xq = xrows_setup(D, lw, xl);
    load_twiddles(xq.twl, xq.Px, tw, MMI_WG);
    xrows_r2c(D, xq, lb0, false);
  }
}

// ------------------------------------------------------------ stage B
// Stages 2 to 4 of the DP45 replay read up to four stored mu beside the
// stencil and need 68 to 76 registers: held to eight wavefronts per SIMD they
// spilled 9, 13 and 1, which made a reverse step up to 1.7 % longer (two
// sublattices, 128x128x16 cells: 1010 vs 993 us; nowhere shorter).
template <bool DP, int ST>
__global__ __launch_bounds__(MMI_WG) __attribute__((amdgpu_waves_per_eu(DP && ST >= 2 && ST <= 4 ? 6 : 8), amdgpu_num_sgpr(80))) void k_adj_b(const InstDesc* __restrict__ descs,
                                                  const int* __restrict__ wg_inst,
                                                  const float2* __restrict__ tw, int nblocks, int count) {
  __shared__ double tot[MMI_PSTRIDE];
  extern __shared__ float2 xl[];
  const int lead = (int)gridDim.x - nblocks;
  if ((int)blockIdx.x < lead) {
    if ((int)blockIdx.x < count) adj_cav<DP, ST>(descs, blockIdx.x, tot);
    return;
  }
  const int lblk = xcd_block(nblocks, lead);
  const InstDesc& D = descs[wg_inst[lblk]];
  const MMG InstCtl* __restrict__ C = gbl(D.ctl);
  if (C->done) return;
  const int nc = D.ncell, S = D.S;
  const int lw = lblk - D.wg0;
  // convolved field adjoint of this cell: C2R of the workgroup's X rows, or
  // the x-inverse pass's output
  float bdv[3] = {0.f, 0.f, 0.f};
  if (D.xfused) {
    const XRows xq = xrows_setup(D, lw, xl);
    load_twiddles(xq.twl, xq.Px, tw, MMI_WG);
    xrows_c2r(D, xq, bdv);
  }
  const int i = wg_cell(D, lw);
  if (i >= nc) return;   // no barrier below
  const bool mag = !D.has_geom || gbl(D.geom)[i];
  const MMG float* const L = gbl(D.lam_B);
  MMG float* const lam_y = gbl(D.lam_y);
  const MMG float* const lam_z = gbl(D.lam_z);
  const MMG float* const mu_ = gbl(D.mu);
  MMG float* const lam_k = gbl(D.lam_k);
  const double h = adj_step(D, C);
  // RK4: coefficient of k_(ST-1) in y_ST and the weight of k_(ST-1)
  const float cst = (float)(ST == 4 ? h : 0.5 * h);
  const float wprev = (float)(h * (ST == 2 ? 1.0 : 2.0) / 6.0);
  // DP45: lambda_k(ST-1) = h (b_(ST-1) lambda_z + sum_{q>=ST} a_(q,ST-1) mu_q)
  const size_t vec = (size_t)3 * S * nc;
  int x, y, z, jn[6];
  cell_xyz(D, i, x, y, z);
  neighbours(D, i, x, y, z, jn);
  const float cq[6] = {D.cex_x, D.cex_x, D.cex_y, D.cex_y, D.cex_z, D.cex_z};
  const float e[3] = {D.ex, D.ey, D.ez}, nl[3] = {D.nlx, D.nly, D.nlz};
  const bool bd_sep = D.demag == 2 && !D.xfused;
  // own field adjoints of both sublattices (they couple through local demag
  // and B_E)
  float lb[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (s < S)
#pragma unroll
      for (int c = 0; c < 3; ++c) lb[s][c] = gat(L, (s * 3 + c) * nc + i);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    if (s >= S) continue;
    // Every load before any store, so that they are in flight together, a
    // neighbour that is absent replaced by the cell itself: with a branch per
    // neighbour its loads were six round trips one after the other (128x128x32
    // film: 31.5 vs 28.5 us; it moves about 65 MB).
    float nb[6][3], mu[3], ly[3], lz[3], ms[4][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int base = (s * 3 + c) * nc;
#pragma unroll
      for (int q = 0; q < 6; ++q) nb[q][c] = gat(L, base + jn[q]);
      mu[c] = gat(mu_, base + i);
      ly[c] = gat(lam_y, base + i);
      lz[c] = ST > 1 ? gat(lam_z, base + i) : 0.f;
      if (bd_sep) bdv[c] = gat(gbl(D.bd), c * nc + i);
#pragma unroll
      for (int q = ST + 1; q <= 6; ++q)
        if (DP && ST > 1) ms[q < 3 ? 0 : q - 3][c] = gat(gbl(D.mu_st) + (size_t)(q - 3) * vec, base + i);
    }
    // exchange (a symmetric graph Laplacian over magnetic pairs)
    float ex[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) ex[c] = fmaf(cq[q], nb[q][c] - lb[s][c], ex[c]);
    const float le = lb[s][0] * e[0] + lb[s][1] * e[1] + lb[s][2] * e[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float v = mu[c] + ex[c] + D.cK * le * e[c];
      if (D.demag == 1) v += nl[c] * (S == 2 ? lb[0][c] + lb[1][c] : lb[0][c]);
      else if (D.demag == 2) v += bdv[c];
      if (S == 2) v -= D.BE * lb[1 - s][c];
      v = mag ? v : 0.f;
      const int idx = (s * 3 + c) * nc + i;
      gat(lam_y, idx) = ly[c] + v;
      if (!DP) {
        if (ST > 1) gat(lam_k, idx) = fmaf(wprev, lz[c], cst * v);
      } else if (ST > 1) {
        // keep mu of stages 3..6 for the stages below
        if (ST >= 3) gat(gbl(D.mu_st) + (size_t)(ST - 3) * vec, idx) = v;
        float acc = (float)(DPCoef::b(ST - 1)) * lz[c] + (float)DPCoef::a(ST, ST - 1) * v;
#pragma unroll
        for (int q = ST + 1; q <= 6; ++q) acc = fmaf((float)DPCoef::a(q, ST - 1), ms[q < 3 ? 0 : q - 3][c], acc);
        gat(lam_k, idx) = (float)h * acc;
      }
    }
  }
}

}  // namespace mmk

// kind 0: step start, 1: stage kernel A, 2: stage kernel B; dp: the DP45 replay.
// The cavity part of `count` instances rides on kinds 0 and 2, except on B of
// stage 1 of a DP45 step, whose workgroups read what it changes: there it is a
// launch of its own (kind 3).
hipError_t mmk_launch_adj(int kind, bool dp, int stage, int nblocks, int count, const InstDesc* d, const int* wg,
                          hipStream_t s, const float2* tw, size_t lds) {
  const int lead = (count + 7) & ~7;   // whole rounds over the XCDs, so that the cells' workgroups keep theirs
  if (kind == 0) {
    if (dp) MM_LAUNCH(mmk::k_adj_start<true>, dim3(lead + nblocks), dim3(MMI_WG), 0, s, d, wg, nblocks, count);
    else MM_LAUNCH(mmk::k_adj_start<false>, dim3(lead + nblocks), dim3(MMI_WG), 0, s, d, wg, nblocks, count);
    return hipGetLastError();
  }
  if (kind == 3 && dp && stage == 1) {
    MM_LAUNCH((mmk::k_adj_cav<true, 1>), dim3(count), dim3(MMI_WG), 0, s, d, count);
    return hipGetLastError();
  }
#define MM_ADJ_A(ST)                                                                                  \
  if (kind == 1 && stage == ST) {                                                                     \
    MM_LAUNCH(mmk::k_adj_a<ST>, dim3(nblocks), dim3(MMI_WG), lds, s, d, wg, tw);                      \
    return hipGetLastError();                                                                         \
  }
#define MM_ADJ_B(DP, ST)                                                                              \
  if (kind == 2 && dp == DP && stage == ST) {                                                         \
    MM_LAUNCH((mmk::k_adj_b<DP, ST>), dim3((DP && ST == 1 ? 0 : lead) + nblocks), dim3(MMI_WG), lds, s, d, wg, tw, \
              nblocks, count);                                                                        \
    return hipGetLastError();                                                                         \
  }
  MM_ADJ_A(1) MM_ADJ_A(2) MM_ADJ_A(3) MM_ADJ_A(4) MM_ADJ_A(5) MM_ADJ_A(6)
  MM_ADJ_B(false, 1) MM_ADJ_B(false, 2) MM_ADJ_B(false, 3) MM_ADJ_B(false, 4)
  MM_ADJ_B(true, 1) MM_ADJ_B(true, 2) MM_ADJ_B(true, 3) MM_ADJ_B(true, 4) MM_ADJ_B(true, 5) MM_ADJ_B(true, 6)
#undef MM_ADJ_A
#undef MM_ADJ_B
  return hipErrorInvalidValue;
}
