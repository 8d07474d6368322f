// Reverse steps of small instances: the discrete adjoint of whole RK4 steps
// (the map and its reverse are stated in kernels_adjoint.hip) in one kernel.
//
// The per-stage launches of the reverse pass (a start, and stage kernels A and
// B per stage: nine a step) cost an instance of at most 1024 cells without
// FFT demag the launch each, as its forward steps did.  Here one
// workgroup runs any number of reverse steps: the adjoints lambda_y, lambda_z
// and lambda_k of a cell stay with its thread (in registers, but for two
// sublattices with two cells per thread, which spill 61), its stage input and lambda_B are
// exchanged through LDS, the recorded stage inputs are fetched one stage
// ahead, and one further wavefront carries the cavity part, one mode per lane.
// A stage has two barriers: behind A (lambda_B and the wave sums are in LDS)
// and behind B (with the next stage input in LDS), beside which the cavity
// wavefront forms mu_a from the sums and publishes what the next A needs.
//
// What bounds it: the dependent chain of a stage (the butterfly sums of A, then
// the cavity's sums over the wavefronts and its update), not throughput.
// A reverse step of the 8x8x1 geometry with the recompute of its forward step:
// 9.6 us against 46.9 us in per-stage launches; the gradient of 256 of its
// steps through the autograd function 4.9 against 14.8 ms.
// The order of every sum is that of the per-stage kernels; the terms of mu_a
// are added in another order and the compiler contracts the rest as it likes,
// so the two agree to rounding.  Which of them an instance takes depends on it
// alone.
#include "mm_internal.h"
#include "kernels_common.h"
#include "launch.h"
#include "small_desc.h"

namespace mmk {

constexpr int SA_CELLS_T = 512;               // cell threads at most: cells t, t + 512, ... of thread t
constexpr int SA_T = SA_CELLS_T + 64;         // and the cavity wavefront
constexpr int SA_SLOTS = MMI_ASLOT_B0 + 3;

template <int C>
struct AdjShared {
  double sum[SA_SLOTS][C][SA_CELLS_T / 64];   // wave sums of A: [slot][block of 512 cells][wavefront]
  double lk[MMI_MAX_MODES][2];                // lambda_ka of all modes (cavity wavefront only)
  float fb[MMI_MAX_MODES], fbw[MMI_MAX_MODES];  // feedback weights of the stage: in the field, in grad u_n
  float lr[MMI_MAX_MODES], li[MMI_MAX_MODES];   // adjoint of m^-
};

// Cell wavefronts.  sm: [S][512 C] stage input, [S][512 C] lambda_B (16-byte
// entries, so that a neighbour is one read), then [N][ncell] grad u_n (double)
// and [N][ncell] profiles, where they are kept in LDS.
template <int S, int C>
__device__ __forceinline__ void adj_cells(const InstDesc& D, AdjShared<C>& sh, float4* sm, int steps, int ri0, bool g_lds,
                                          bool u_lds) {
  constexpr int NCP = C * SA_CELLS_T;
  const int nc = D.ncell, N = D.N;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool prof = D.profiled != 0;
  const int nsum = prof ? N : min(N, 1);
  float4* const sb = sm + S * NCP;
  double* const sg = (double*)(sb + S * NCP);
  float* const su = (float*)(sg + (g_lds ? (size_t)N * nc : 0));
  const MMG float* const gu = gbl(D.u);
  MMG double* const gg = gbl(D.grad_u);
  const MMG float* const rec = gbl(D.rec_m);
  const MMG float* const rnorm = gbl(D.rec_norm);
  const int vec = 3 * S * nc;
  const CellDesc<S> Q(D);
  const double h = D.ctl->adj_h;
  const float c6 = (float)(h / 6.0), wmm = (float)(D.inv_ngeo / (double)S);
  const float gl = Q.gl, al = Q.alpha;
  const float dga = 2.f * al / (1.f + al * al);      // -d ln(gamma')/d alpha
  const float e[3] = {Q.ex, Q.ey, Q.ez}, nl[3] = {Q.nlx, Q.nly, Q.nlz};
  const float cq[6] = {Q.cex_x, Q.cex_x, Q.cex_y, Q.cex_y, Q.cex_z, Q.cex_z};
  int jn[C][6];
  bool valid[C], mag[C];
  float ly[C][S][3], lz[C][S][3], lk[C][S][3], y[C][S][3], norm[C][S], pre[C][S][3];

  // the recorded input of stage st of step ri, into `pre`
  auto fetch = [&](int ri, int st) {
    const MMG float* R = rec + (size_t)(ri * 4 + st - 1) * vec;
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) pre[j][s][c] = valid[j] ? R[(s * 3 + c) * nc + j * SA_CELLS_T + threadIdx.x] : 0.f;
  };
  auto fetch_norm = [&](int ri) {
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s)
        norm[j][s] = mag[j] ? rnorm[(size_t)ri * (S * nc) + s * nc + j * SA_CELLS_T + threadIdx.x] : 1.f;
  };
  auto put_input = [&]() {
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s)
        sm[s * NCP + j * SA_CELLS_T + threadIdx.x] = make_float4(pre[j][s][0], pre[j][s][1], pre[j][s][2], 0.f);
  };

#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int i = j * SA_CELLS_T + threadIdx.x;
    valid[j] = i < nc;
    mag[j] = valid[j] && (!D.has_geom || gbl(D.geom)[i]);
    const int ic = valid[j] ? i : 0;
    int x, yy, zz;
    cell_xyz(D, ic, x, yy, zz);
    neighbours(D, ic, x, yy, zz, jn[j]);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ly[j][s][c] = valid[j] ? gbl(D.lam_y)[(s * 3 + c) * nc + i] : 0.f;
        y[j][s][c] = valid[j] ? rec[(size_t)((ri0 + 1) * 4) * vec + (s * 3 + c) * nc + i] : 0.f;
      }
    if (valid[j])
      for (int q = 0; q < N; ++q) {
        if (g_lds && gg) sg[q * nc + i] = gg[(size_t)q * nc + i];
        if (u_lds) su[q * nc + i] = gu[(size_t)q * nc + i];
      }
  }
  fetch_norm(ri0);
  fetch(ri0, 4);
  put_input();
  __syncthreads();
  for (int it = 0; it < steps; ++it) {
    const int ri = ri0 - it;
    // step start: lambda_z, lambda_y = lambda_z, lambda_k4 = h/6 lambda_z
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float inv = 1.0f / norm[j][s];
        const float d = ly[j][s][0] * y[j][s][0] + ly[j][s][1] * y[j][s][1] + ly[j][s][2] * y[j][s][2];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float z = mag[j] ? (ly[j][s][c] - y[j][s][c] * d) * inv : 0.f;
          lz[j][s][c] = z;
          ly[j][s][c] = z;
          lk[j][s][c] = c6 * z;
        }
      }
#pragma unroll 1
    for (int st = 4; st >= 1; --st) {
      const bool more = st > 1 || it + 1 < steps;
      float mu[C][S][3], lb[C][S][3];
      // stage A
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const int i = j * SA_CELLS_T + threadIdx.x;
        if (C > 1 && j * SA_CELLS_T >= nc) {
#pragma unroll
          for (int s = 0; s < S; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) mu[j][s][c] = lb[j][s][c] = 0.f;
          continue;
        }
        float m[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}}, nb[S][6][3];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float4 v = sm[s * NCP + i];
          m[s][0] = v.x;
          m[s][1] = v.y;
          m[s][2] = v.z;
#pragma unroll
          for (int q = 0; q < 6; ++q) {
            const float4 w = sm[s * NCP + jn[j][q]];
            nb[s][q][0] = w.x;
            nb[s][q][1] = w.y;
            nb[s][q][2] = w.z;
          }
        }
        if (st == 1)
#pragma unroll
          for (int s = 0; s < S; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) y[j][s][c] = m[s][c];
        auto prof_u = [&](int q) {
          return !prof ? 1.f : !valid[j] ? 0.f : u_lds ? su[q * nc + i] : gu[(size_t)q * nc + i];
        };
        float fb = 0.f;
        for (int q = 0; q < N; ++q) fb = fmaf(sh.fb[q], prof_u(q), fb);
        double galpha = 0.0, gb[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float B[3], P[3], R[3], lm[3], t1[3], t2[3], t3[3];
          field_nb(Q, i, nb[s], m, s, fb, false, B);
          const float(&l)[3] = lk[j][s];
          cross3(m[s], B, P);
          cross3(m[s], P, R);
          cross3(l, m[s], lm);         // lambda x m
          cross3(lm, m[s], t1);        // (lambda x m) x m
#pragma unroll
          for (int c = 0; c < 3; ++c) lb[j][s][c] = mag[j] ? -gl * (lm[c] + al * t1[c]) : 0.f;
          cross3(B, l, t1);            // B x lambda
          cross3(P, l, t2);            // P x lambda
          cross3(B, lm, t3);           // B x (lambda x m)
          // dL/dalpha: lambda . (-(2a/(1+a^2)) tau - gamma' R), tau = -gamma' (P + a R)
          float ga = 0.f;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            mu[j][s][c] = mag[j] ? -gl * (t1[c] + al * (t2[c] + t3[c])) : 0.f;
            const float tau = -gl * (P[c] + al * R[c]);
            ga += l[c] * (-dga * tau - gl * R[c]);
            gb[c] += lb[j][s][c];
          }
          galpha += mag[j] ? ga : 0.f;
          sb[s * NCP + i] = make_float4(lb[j][s][0], lb[j][s][1], lb[j][s][2], 0.f);
        }
        // m^- transpose, the gradient of the mode profiles and the sums
        auto put2 = [&](int slot, double a, double b) {
          const double w = wave_sum2(a, b);
          if ((lane & 31) == 0) sh.sum[slot + (lane >> 5)][j][wv] = w;
        };
        for (int q = 0; q < N; ++q) {
          const float u = prof_u(q), lr = sh.lr[q], li = sh.li[q], fbw = sh.fbw[q];
          double fbn = 0.0, mr = 0.0, mi = 0.0, g = 0.0;
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const float cs = Q.csign[s];
            mu[j][s][0] += mag[j] ? wmm * cs * u * lr : 0.f;
            mu[j][s][1] -= mag[j] ? wmm * cs * u * li : 0.f;
            fbn += (double)(cs * lb[j][s][0] * u);
            mr += (double)(cs * m[s][0] * u);
            mi -= (double)(cs * m[s][1] * u);
            g += (double)(cs * (lb[j][s][0] * fbw + wmm * (lr * m[s][0] - li * m[s][1])));
          }
          if (mag[j] && gg) {
            if (g_lds) sg[q * nc + i] += g;
            else gg[(size_t)q * nc + i] += g;
          }
          if (q < nsum) {
            put2(MMI_ASLOT_MM + 2 * q, mag[j] ? mr : 0.0, mag[j] ? mi : 0.0);
            const double w = wave_sum(mag[j] ? fbn : 0.0);
            if (lane == 0) sh.sum[MMI_ASLOT_FB + q][j][wv] = w;
          }
        }
        put2(MMI_ASLOT_ALPHA, galpha, gb[0]);
        put2(MMI_ASLOT_B0 + 1, gb[1], gb[2]);
      }
      // the next stage input, on its way during the barrier and B
      if (more) fetch(st > 1 ? ri : ri - 1, st > 1 ? st - 1 : 4);
      if (st == 1 && more) fetch_norm(ri - 1);
      __syncthreads();
      // stage B
      const float cst = (float)(st == 4 ? h : 0.5 * h);
      const float wprev = (float)(h * (st == 2 ? 1.0 : 2.0) / 6.0);
#pragma unroll
      for (int j = 0; j < C; ++j) {
        if (C > 1 && j * SA_CELLS_T >= nc) break;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float ex[3] = {0.f, 0.f, 0.f};
          // exchange (a symmetric graph Laplacian over magnetic pairs)
#pragma unroll
          for (int q = 0; q < 6; ++q) {
            const float4 w = sb[s * NCP + jn[j][q]];
            ex[0] = fmaf(cq[q], w.x - lb[j][s][0], ex[0]);
            ex[1] = fmaf(cq[q], w.y - lb[j][s][1], ex[1]);
            ex[2] = fmaf(cq[q], w.z - lb[j][s][2], ex[2]);
          }
          const float le = lb[j][s][0] * e[0] + lb[j][s][1] * e[1] + lb[j][s][2] * e[2];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            float v = mu[j][s][c] + ex[c] + Q.cK * le * e[c];
            if (Q.demag == 1) {
              float t = lb[j][0][c];
              if (S == 2) t += lb[j][S - 1][c];
              v += nl[c] * t;
            }
            if (S == 2) v -= Q.BE * lb[j][S - 1 - s][c];
            v = mag[j] ? v : 0.f;
            ly[j][s][c] += v;
            if (st > 1) lk[j][s][c] = fmaf(wprev, lz[j][s][c], cst * v);
          }
        }
      }
      if (more) put_input();
      __syncthreads();
    }
  }
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int i = j * SA_CELLS_T + threadIdx.x;
    if (!valid[j]) continue;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) gbl(D.lam_y)[(s * 3 + c) * nc + i] = ly[j][s][c];
    if (g_lds && gg)
      for (int q = 0; q < N; ++q) gg[(size_t)q * nc + i] = sg[q * nc + i];
  }
}

// The cavity wavefront: lane n < N carries mode n, lanes 32..35 the sums that
// are the gradients of alpha and B0.
template <int S, int C>
__device__ __forceinline__ void adj_cavity(const InstDesc& D, AdjShared<C>& sh, int steps, int ri0) {
  InstCtl* const K = D.ctl;
  const int N = D.N, lane = threadIdx.x & 63;
  const bool mode = lane < N, coupled = D.jcpl_on != 0, kerr = D.kerr_on != 0, pump = D.param_on != 0;
  const int n = mode ? lane : 0;
  const int nct = blockDim.x - 64;
  const MMG double* const ra = gbl(D.rec_a);
  const MMG double* const tr = gbl(D.dla_trace);
  const double h = K->adj_h, t0 = K->adj_t0, scale = D.inv_ngeo / (double)S;
  const long long base = K->adj_base;
  const double cp = D.cphi[n], sp = D.sphi[n], g = D.g[n], om = D.omega[n], kp = D.kappa[n], h0 = D.h0[n];
  const double two_gamma = 2.0 / D.gamma, kr = D.kerr[n];
  const double pre = D.par_re[n], pim = D.par_im[n], pwp = D.par_wp[n];
  double la[2] = {K->la[n][0], K->la[n][1]}, lza[2] = {0.0, 0.0}, lka[2] = {0.0, 0.0};
  double as[2], an[2], gacc = lane >= 32 && lane < 36 ? (lane == 32 ? K->grad_alpha : K->grad_B0[lane - 33]) : K->grad_g[n];
  const int pn = D.profiled ? n : 0;
  const int slot0 = lane >= 32 ? MMI_ASLOT_ALPHA + (lane & 3) : MMI_ASLOT_FB + pn;

  // stage amplitude of stage st of step ri
  auto fetch = [&](int ri, int st) {
    const MMG double* q = ra + ((size_t)ri * 4 + (st - 1)) * N * 2 + 2 * n;
    an[0] = q[0];
    an[1] = q[1];
  };
  // sum over wavefronts, then over the blocks of 512 cells, in the order of
  // the partial records and their gather
  auto total = [&](int slot) {
    double p[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < C; ++j) {
      double v[SA_CELLS_T / 64];
#pragma unroll
      for (int w = 0; w < SA_CELLS_T / 64; ++w) v[w] = sh.sum[slot][j][w];
      double x = v[0];
      if (nct > 64) {
#pragma unroll
        for (int w = 1; w < SA_CELLS_T / 64; ++w) x += v[w];
      }
      p[j] = 0.0 + x;
    }
    return p[0] + p[1];
  };
  auto start = [&](double d0, double d1) {
    la[0] += d0;
    la[1] += d1;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      lza[r] = la[r];
      lka[r] = h / 6.0 * la[r];
    }
  };
  // what the next stage kernel A reads
  auto publish = [&]() {
    as[0] = an[0];
    as[1] = an[1];
    if (!mode) return;
    // adjoint of m^-: conj(i g e^{-i Phi}) lambda_ka
    sh.lr[n] = (float)(g * (sp * lka[0] + cp * lka[1]));
    sh.li[n] = (float)(g * (sp * lka[1] - cp * lka[0]));
    sh.fb[n] = feedback_weight(h0, cp, sp, as[0], as[1]);
    sh.fbw[n] = feedback_weight(h0, cp, sp, (double)(float)as[0], (double)(float)as[1]);
  };
  // a loss on the trace: its derivative at the end of step ri
  double d[2] = {0.0, 0.0};
  auto fetch_trace = [&](int ri) {
    if (!tr) return;
    const MMG double* q = tr + (size_t)(base + ri + 1) * N * 2 + 2 * n;
    d[0] = q[0];
    d[1] = q[1];
  };

  if (N > 0) {
    fetch_trace(ri0);
    fetch(ri0, 4);
  }
  start(d[0], d[1]);
  publish();
  __syncthreads();
  for (int it = 0; it < steps; ++it) {
    const int ri = ri0 - it;
#pragma unroll 1
    for (int st = 4; st >= 1; --st) {
      const bool more = st > 1 || it + 1 < steps;
      if (N > 0) {
        if (more) fetch(st > 1 ? ri : ri - 1, st > 1 ? st - 1 : 4);
        if (st == 1 && more) fetch_trace(ri - 1);
      }
      double Lr = 0.0, Li = 0.0;
      if (pump) {
        // transpose of the Jacobian of -i Lam conj(a), Lam = lam e^{-2 i wp t}
        const double ts = t0 + (double)ri * h + (st == 1 ? 0.0 : st == 4 ? h : 0.5 * h);
        double sn, cs;
        sincos(2.0 * pwp * ts, &sn, &cs);
        Lr = pre * cs + pim * sn;
        Li = pim * cs - pre * sn;
      }
      double mur = -kp * lka[0] - om * lka[1], mui = om * lka[0] - kp * lka[1];
      if (kerr) {
        // transpose of the Jacobian of -i K |a|^2 a at the stage amplitude
        const double ar = as[0], ai = as[1];
        const double q = kr * (ar * ar + ai * ai), x = 2.0 * kr * ar * ai;
        mur += lka[0] * x - lka[1] * (q + 2.0 * kr * ar * ar);
        mui += lka[0] * (q + 2.0 * kr * ai * ai) - lka[1] * x;
      }
      mur += Li * lka[0] - Lr * lka[1];
      mui -= Lr * lka[0] + Li * lka[1];
      if (coupled) {
        wave_lds_order();
        if (mode) {
          sh.lk[n][0] = lka[0];
          sh.lk[n][1] = lka[1];
        }
        wave_lds_order();
        for (int q = 0; q < N; ++q) {
          // -i sum_q J_qn a_n in the equation of mode q, J symmetric
          mur -= D.jcpl[q][n] * sh.lk[q][1];
          mui += D.jcpl[q][n] * sh.lk[q][0];
        }
      }
      const double c = st == 4 ? h : 0.5 * h, wp = h * (st == 2 ? 1.0 : 2.0) / 6.0;
      __syncthreads();
      // the sums of stage kernel A
      const double fb = total(slot0), mr = total(MMI_ASLOT_MM + 2 * pn) * scale, mi = total(MMI_ASLOT_MM + 2 * pn + 1) * scale;
      mur += h0 * fb * cp;
      mui += h0 * fb * sp;
      // dF/dg = (s + i c) m^- ; feedback h0 = 2 g / gamma with Re[e^{-i Phi} a] = c ar + s ai
      const double fr = sp * mr - cp * mi, fi = sp * mi + cp * mr;
      gacc += lane >= 32 ? fb : lka[0] * fr + lka[1] * fi + fb * two_gamma * (cp * as[0] + sp * as[1]);
      la[0] += mur;
      la[1] += mui;
      if (st > 1) {
        lka[0] = wp * lza[0] + c * mur;
        lka[1] = wp * lza[1] + c * mui;
      } else if (more) {
        start(d[0], d[1]);
      }
      if (more) publish();
      __syncthreads();
    }
  }
  if (mode) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      K->la[n][r] = la[r];
      K->lza[n][r] = lza[r];
      K->lka[n][r] = lka[r];
    }
    K->grad_g[n] = gacc;
  }
  if (lane == 32) K->grad_alpha = gacc;
  if (lane > 32 && lane < 36) K->grad_B0[lane - 33] = gacc;
  if (lane == 0) K->rec_index = ri0 - steps;
}

// `steps` reverse steps of instance `inst` from the recorded step at
// rec_index downwards.  blockDim.x = cell threads + 64; the two roles meet at
// the same number of barriers, one at the start and two per stage.
template <int S, int C>
__global__ __launch_bounds__(SA_T) void k_small_adj(const InstDesc* __restrict__ descs, int inst, int steps, int g_lds,
                                                    int u_lds) {
  __shared__ AdjShared<C> sh;
  extern __shared__ float4 sm[];
  const InstDesc& D = descs[inst];
  const InstCtl* const C0 = D.ctl;
  if (C0->done) return;
  const int ri0 = C0->rec_index;
  if (steps > ri0 + 1) steps = ri0 + 1;
  // sums of wavefronts and blocks that the instance does not have stay zero
  for (int k = threadIdx.x; k < (int)(sizeof(sh.sum) / sizeof(double)); k += blockDim.x) (&sh.sum[0][0][0])[k] = 0.0;
  __syncthreads();                                 // (also: every wavefront has read the control block)
  const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (role == (int)(blockDim.x >> 6) - 1) {
    __builtin_amdgcn_s_setprio(3);                 // the cells wait for it
    adj_cavity<S, C>(D, sh, steps, ri0);
  } else {
    adj_cells<S, C>(D, sh, sm, steps, ri0, g_lds != 0, u_lds != 0);
  }
}

}  // namespace mmk

hipError_t mmk_launch_small_adj(int S, int ncell, size_t lds, bool g_lds, bool u_lds, const InstDesc* d, int inst, int steps,
                                hipStream_t s) {
  const int threads = (ncell < mmk::SA_CELLS_T ? (ncell + 63) / 64 * 64 : mmk::SA_CELLS_T) + 64;
  const int per = (ncell + mmk::SA_CELLS_T - 1) / mmk::SA_CELLS_T;
#define MM_SMALL_ADJ(A, B)                                                                                         \
  do {                                                                                                             \
    MM_LAUNCH((mmk::k_small_adj<A, B>), dim3(1), dim3(threads), lds, s, d, inst, steps, g_lds ? 1 : 0, u_lds ? 1 : 0); \
    return hipGetLastError();                                                                                      \
  } while (0)
  if (steps < 1 || per < 1 || per > 2 || S < 1 || S > 2) return hipErrorInvalidValue;
  if (S == 1 && per == 1) MM_SMALL_ADJ(1, 1);
  if (S == 1) MM_SMALL_ADJ(1, 2);
  if (per == 1) MM_SMALL_ADJ(2, 1);
  MM_SMALL_ADJ(2, 2);
#undef MM_SMALL_ADJ
}

hipError_t mmk_set_small_adj_lds_limits() {
  hipError_t e = hipSuccess;
#define MM_SMALL_ATTR(A, B)                                               \
  if (e == hipSuccess)                                                    \
    e = hipFuncSetAttribute((const void*)mmk::k_small_adj<A, B>, hipFuncAttributeMaxDynamicSharedMemorySize, MMI_SMALL_LDS);
  MM_SMALL_ATTR(1, 1) MM_SMALL_ATTR(1, 2) MM_SMALL_ATTR(2, 1) MM_SMALL_ATTR(2, 2)
#undef MM_SMALL_ATTR
  return e;
}
