// Fixed-step runs of small instances: whole RK4 steps inside one kernel.
//
// An instance of at most MMI_SMALL_CELLS cells without FFT demag (the
// paper's 8x8x1 geometry, the 8^3 cube) has microseconds of arithmetic per
// step, and a launch per stage and finalisation (eight per step) cost it
// about 30 us.  Here one workgroup owns the instance for as many steps as
// the launch is given: the state and the running sum of the stage
// derivatives stay with their threads (in registers; with more than one cell
// per thread, at the three wavefronts per SIMD of such a workgroup, in part in
// scratch memory: 14 to 20 spilled registers for two cells, 77 to 107 for
// four), the stage inputs are exchanged through LDS
// (two buffers, one barrier per stage), and one further wavefront carries
// the FP64 cavity modes, one per lane, beside the cell wavefronts.
//
// The cavity runs one stage behind without holding the cells up: stage s+1
// needs a_{s+1} = a + c h ka_s, and ka_s depends on m^- of the stage-s
// input, whose sums were complete one barrier earlier.  While the cells
// evaluate stage s the cavity wavefront therefore forms ka_s from those sums
// and publishes the feedback of stage s+1.  At the step end the same holds
// for a(t + h), the step plan and the end-of-run test; only ka_1 and the trace
// sample, which need m^- of the new state, fall into stage 1 of the next step.
//
// What bounds it: the dependent chain of a stage (LDS read of the neighbours,
// torque, the butterfly sums of m^-, one barrier: about 900 cycles for one to
// two cell wavefronts per SIMD) and beside it the cavity's (sums over the
// wavefronts, right-hand side, feedback), not throughput.  2000 steps of the
// 8x8x1 geometry with its pulse and a trace sample per step: 3.9 ms against
// 60.9 ms in per-stage launches; of the 8^3 cube 6.3 against 60.8 ms.  The
// first version, with the neighbours' components in separate arrays and the
// envelope's exponential, a division by 6 and the loads of the descriptor on
// the cavity's chain, took 7.8 and 11.5 ms.
// The arithmetic and the order of every sum are those of k_stage and
// finalize, with shared functions whose fused multiply-adds are written out:
// an instance's results do not depend on the batch it is in.
#include <type_traits>
#include "mm_internal.h"
#include "kernels_common.h"
#include "launch.h"
#include "stage_final.h"
#include "small_desc.h"

namespace mmk {

constexpr int SM_CELLS_T = 512;               // cell threads at most: cells t, t + 512, ... of thread t
constexpr int SM_T = SM_CELLS_T + 64;         // and the cavity wavefront

// One mode's parameters behind the names cav_rhs uses.
struct ModeDesc {
  struct One {
    double v;
    __device__ __forceinline__ double operator[](int) const { return v; }
  };
  struct Row {
    const MMG double* p;
    __device__ __forceinline__ const MMG double* operator[](int) const { return p; }
  };
  int N, kerr_on, jcpl_on, param_on, drive_on;
  One omega, kappa, g, cphi, sphi, kerr, eta_re, eta_im, eta_t0, eta_sigma, par_re, par_im, par_wp;
  Row jcpl;
  double env = 0.0;               // the drive's envelope at the time of the next cav_rhs
  __device__ __forceinline__ ModeDesc(const InstDesc& D, int n)
      : N(D.N), kerr_on(D.kerr_on), jcpl_on(D.jcpl_on), param_on(D.param_on), drive_on(D.drive_on), omega{D.omega[n]},
        kappa{D.kappa[n]}, g{D.g[n]}, cphi{D.cphi[n]}, sphi{D.sphi[n]}, kerr{D.kerr[n]}, eta_re{D.eta_re[n]},
        eta_im{D.eta_im[n]}, eta_t0{D.eta_t0[n]}, eta_sigma{D.eta_sigma[n]}, par_re{D.par_re[n]}, par_im{D.par_im[n]},
        par_wp{D.par_wp[n]}, jcpl{(const MMG double*)D.jcpl[n]} {}
};

__device__ __forceinline__ double cav_envelope(const ModeDesc& D, int, double) { return D.env; }
// sincos as a call: only the parametric pump uses it, and its argument
// reduction inlined would take the registers of everything else
__device__ __attribute__((noinline)) double2 sincos_call(double x) {
  double2 r;
  sincos(x, &r.y, &r.x);
  return r;
}
__device__ __forceinline__ void cav_sincos(const ModeDesc&, double x, double& sn, double& cs) {
  const double2 r = sincos_call(x);
  cs = r.x;
  sn = r.y;
}

struct Cplx {
  double r, i;
};
// the amplitude of the lane's own mode behind cav_rhs's A[mode][re/im]
struct OwnAmp {
  Cplx v;
  struct Row {
    Cplx v;
    __device__ __forceinline__ double operator[](int q) const { return q ? v.i : v.r; }
  };
  __device__ __forceinline__ Row operator[](int) const { return {v}; }
};

// What the two roles of a workgroup exchange through LDS.
template <int C>
struct SmallShared {
  // wave sums of m^-: [buffer][2 mode + re/im][block of 512 cells][wavefront]
  double sum[2][2 * MMI_MAX_MODES][C][SM_CELLS_T / 64];
  double amp[MMI_MAX_MODES][2];        // stage amplitudes of all modes (cavity wavefront only)
  float fb[2][MMI_MAX_MODES];          // feedback weights h0 Re[e^{-i Phi} a] of the next stage
  float fbu[2];                        // their sum in mode order (modes without profiles)
  double h;                            // step size
  float h6;                            // (float)(h / 6)
  int bad_m, bad_a, done;
};

// Cell wavefronts.  Stage ST (1..4) reads stage input buffer (ST - 1) & 1 and
// writes the next input to the other.  A cell's vector is one 16-byte LDS
// entry, so that a neighbour is one read; the buffers have a fixed size, so
// that their offset is part of the instruction.
template <int S, int C, bool PROF>
__device__ __forceinline__ void small_cells(const InstDesc& D, SmallShared<C>& sh, float4* sm, int steps, int ri0, int cur0) {
  constexpr int NCP = C * SM_CELLS_T;                // entries per sublattice and buffer
  const int nc = D.ncell, N = D.N;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool rec = ri0 >= 0, split = D.split != 0, u_lds = PROF && D.small_u != 0;
  float* const su = (float*)(sm + 2 * S * NCP);
  const MMG float* const gu = gbl(D.u);
  const CellDesc<S> Q(D);
  const int nsum = PROF ? N : min(N, 1);
  int jn[C][6];
  bool valid[C], mag[C];
  float y[C][S][3], acc[C][S][3];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int i = j * SM_CELLS_T + threadIdx.x;
    valid[j] = i < nc;
    mag[j] = valid[j] && (!D.has_geom || gat(gbl(D.geom), i));
    const int ic = valid[j] ? i : 0;
    int x, yy, zz;
    cell_xyz(D, ic, x, yy, zz);
    neighbours(D, ic, x, yy, zz, jn[j]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        y[j][s][c] = valid[j] ? gat(gbl(D.y[cur0]), (s * 3 + c) * nc + i) : 0.f;
        acc[j][s][c] = 0.f;
      }
      sm[s * NCP + i] = make_float4(y[j][s][0], y[j][s][1], y[j][s][2], 0.f);
    }
    if (u_lds && valid[j])
      for (int q = 0; q < N; ++q) su[q * nc + i] = gu[(size_t)q * nc + i];
  }
  __syncthreads();
  int ran = 0;
  double h = 0.0;
  float h6 = 0.f;
  // one stage of step `it`
  auto stage = [&](int it, int ST) {
    const int rb = (ST - 1) & 1, wb = ST & 1;
    const float4* const src = sm + rb * S * NCP;
    float4* const dst = sm + wb * S * NCP;
    const float cc = ST == 4 ? h6 : ST == 3 ? (float)h : (float)(0.5 * h);
    const size_t ri = (size_t)(ri0 + it);
    const float fbu = PROF ? 0.f : sh.fbu[rb];
    bool badm = false;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int i = j * SM_CELLS_T + threadIdx.x;
      if (C > 1 && j * SM_CELLS_T >= nc) break;
      float m[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
      float nx[S][3], k[S][3], nb[S][6][3];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float4 v = src[s * NCP + i];
        m[s][0] = v.x;
        m[s][1] = v.y;
        m[s][2] = v.z;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          const float4 w = src[s * NCP + jn[j][q]];
          nb[s][q][0] = w.x;
          nb[s][q][1] = w.y;
          nb[s][q][2] = w.z;
        }
      }
      if (rec && valid[j]) {
        MMG float* R = gbl(D.rec_m) + (ri * 4 + (ST - 1)) * (size_t)(3 * S * nc);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int c = 0; c < 3; ++c) R[(s * 3 + c) * nc + i] = m[s][c];
      }
      float fb = fbu;
      if (PROF && valid[j])
        for (int q = 0; q < N; ++q) fb = fmaf(sh.fb[rb][q], u_lds ? su[q * nc + i] : gu[(size_t)q * nc + i], fb);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        float B[3];
        field_nb(Q, i, nb[s], m, s, fb, false, B);
        ll_torque(Q, m[s], B, k[s]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float kk = mag[j] ? k[s][c] : 0.f;
          const float kw = ST == 4 ? acc[j][s][c] + kk : kk;
          acc[j][s][c] = ST == 1 ? kk : fmaf(2.f, kk, acc[j][s][c]);
          nx[s][c] = fmaf(cc, kw, y[j][s][c]);       // next stage input, or the step end
        }
      }
      if (ST == 4) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float v0 = nx[s][0], v1 = nx[s][1], v2 = nx[s][2];
          if (mag[j]) {
            const float nrm = sqrtf(v0 * v0 + v1 * v1 + v2 * v2);
            if (rec) gbl(D.rec_norm)[ri * (size_t)(S * nc) + s * nc + i] = nrm;
            const float inv = 1.0f / nrm;
            v0 *= inv;
            v1 *= inv;
            v2 *= inv;
          }
          if (valid[j] && !(isfinite(v0) && isfinite(v1) && isfinite(v2))) badm = true;
          nx[s][0] = v0;
          nx[s][1] = v1;
          nx[s][2] = v2;
        }
      }
      float vr = 0.f, vi = 0.f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        dst[s * NCP + i] = make_float4(nx[s][0], nx[s][1], nx[s][2], 0.f);
        vr = fmaf(Q.csign[s], nx[s][0], vr);
        vi = fmaf(-Q.csign[s], nx[s][1], vi);
      }
      // mode sums of the next stage input
      for (int q = 0; q < nsum; ++q) {
        const double u = PROF && valid[j] ? (double)(u_lds ? su[q * nc + i] : gu[(size_t)q * nc + i]) : 1.0;
        const double w = wave_sum2(mag[j] ? u * (double)vr : 0.0, mag[j] ? u * (double)vi : 0.0);
        if ((lane & 31) == 0) sh.sum[wb][2 * q + (lane >> 5)][j][wv] = w;
      }
    }
    if (badm) sh.bad_m = 1;
    __syncthreads();
  };
  for (int it = 0; it < steps; ++it) {
    h = sh.h;
    h6 = sh.h6;
    if constexpr (C * S <= 2) {
      stage(it, 1);
      stage(it, 2);
      stage(it, 3);
      stage(it, 4);
    } else {
#pragma unroll 1
      for (int ST = 1; ST <= 4; ++ST) stage(it, ST);
    }
    if (sh.bad_m || sh.bad_a) break;
    ran = it + 1;
    const bool done = sh.done;
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float4 v = sm[s * NCP + j * SM_CELLS_T + threadIdx.x];
        y[j][s][0] = v.x;
        y[j][s][1] = v.y;
        y[j][s][2] = v.z;
      }
    if (split) __syncthreads();
    if (done) break;
  }
  if (ran == 0) return;
  MMG float* const Y = gbl(D.y[cur0 ^ (ran & 1)]);
#pragma unroll
  for (int j = 0; j < C; ++j)
    if (valid[j])
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) gat(Y, (s * 3 + c) * nc + j * SM_CELLS_T + threadIdx.x) = y[j][s][c];
}

// The cavity wavefront: lane n < N carries mode n in FP64; scalars (time,
// step plan, counters) are the same in every lane.
template <int S, int C, bool PROF>
__device__ __forceinline__ void small_cavity(const InstDesc& D, SmallShared<C>& sh, int steps, int ri0, int cur0) {
  InstCtl* const C0 = D.ctl;
  const int N = D.N;
  const int lane = threadIdx.x & 63;
  // everything the loop needs of the descriptor, read once: a scalar load
  // behind each barrier would sit on the chain the cells wait for
  const bool rec = ri0 >= 0, split = D.split != 0, drive = D.drive_on != 0, coupled = D.jcpl_on != 0;
  MMG double* const rec_a = gbl(D.rec_a);
  MMG double* const trace_t = gbl(D.trace_t);
  MMG double* const trace_a = gbl(D.trace_a);
  MMG double* const trace_m = gbl(D.trace_m);
  const int nct = blockDim.x - 64;                   // cell threads
  const bool mode = lane < N;
  const int n = mode ? lane : 0;
  ModeDesc MD(D, n);
  MD.jcpl_on = 0;
  const double h0 = D.h0[n];
  const double scale = D.inv_ngeo / (double)S;
  Cplx a{C0->a[n][0], C0->a[n][1]}, as{C0->as[n][0], C0->as[n][1]};
  Cplx k0{C0->ka[0][n][0], C0->ka[0][n][1]}, ksum{0.0, 0.0}, mm{C0->mm1[n][0], C0->mm1[n][1]};
  double t = C0->t, h = C0->h, hmin = C0->dt_min_seen, hmax = C0->dt_max_seen;
  const double t_end = C0->t_end, dt_fixed = C0->dt_fixed;
  long long accepted = C0->accepted, trace_n = C0->trace_n, trace_steps = C0->trace_steps;
  const long long trace_max = C0->trace_max, stride = C0->trace_stride;
  const int trace_on = C0->trace_on;
  long long phase = trace_on ? trace_steps % stride : 0;
  int clipped = C0->clipped;

  auto publish = [&](int b, Cplx v) {
    const float f = feedback_weight(h0, MD.cphi.v, MD.sphi.v, v.r, v.i);
    if (PROF) {
      if (mode) sh.fb[b][n] = f;
    } else {
      float sum = 0.f + __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(f)));
      for (int q = 1; q < N; ++q) sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), q));
      if (lane == 0) sh.fbu[b] = sum;
    }
  };
  // the drive's envelope at time ts, for the next right-hand sides: a step
  // has three stage times, and its last is the next step's first
  double env_t = NAN;
  auto envelope = [&](double ts) {
    if (!drive || ts == env_t) return;
    env_t = ts;
    MD.env = gauss_envelope(ts, MD.eta_t0.v, MD.eta_sigma.v);
  };
  // m^- of this lane's mode from sum buffer b, in the order of the partial
  // records and their gather: wavefronts in turn, then the butterfly over
  // the blocks of 512 cells
  auto gather = [&](int b) -> Cplx {
    const int k = PROF ? n : 0;
    double p[2][4] = {};
    // (sums of wavefronts and blocks the instance does not have stay zero)
#pragma unroll
    for (int q = 0; q < C; ++q) {
      double v[2][SM_CELLS_T / 64];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int w = 0; w < SM_CELLS_T / 64; ++w) v[r][w] = sh.sum[b][2 * k + r][q][w];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        double x = v[r][0];
        if (nct > 64) {
#pragma unroll
          for (int w = 1; w < SM_CELLS_T / 64; ++w) x += v[r][w];
        }
        p[r][q] = 0.0 + x;
      }
      if (C > 1) __builtin_amdgcn_sched_barrier(0);  // one block's sums in registers at a time
    }
    return {((p[0][0] + p[0][2]) + (p[0][1] + p[0][3])) * scale, ((p[1][0] + p[1][2]) + (p[1][1] + p[1][3])) * scale};
  };
  // cavity right-hand side of this lane's mode at the stage amplitude v (all
  // modes' amplitudes through LDS, for direct mode coupling)
  auto rhs = [&](double ts, Cplx v, Cplx mv) -> Cplx {
    Cplx f;
    envelope(ts);
    cav_rhs(MD, n, ts, OwnAmp{v}, mv.r, mv.i, f.r, f.i);
    if (coupled) {
      ModeDesc MC = MD;
      MC.jcpl_on = 1;
      wave_lds_order();
      if (mode) {
        sh.amp[n][0] = v.r;
        sh.amp[n][1] = v.i;
      }
      wave_lds_order();
      cav_rhs(MC, n, ts, sh.amp, mv.r, mv.i, f.r, f.i);
    }
    return f;
  };
  auto sample = [&]() {
    if (!trace_on) return;
    trace_steps += 1;
    if (++phase == stride) phase = 0;
    if (phase != 0 || trace_n >= trace_max) return;
    if (lane == 0) trace_t[trace_n] = t;
    if (mode) {
      MMG double* ta = trace_a + (trace_n * N + n) * 2;
      MMG double* tm = trace_m + (trace_n * N + n) * 2;
      ta[0] = a.r;
      ta[1] = a.i;
      tm[0] = mm.r;
      tm[1] = mm.i;
    }
    trace_n += 1;
  };

  publish(0, as);
  publish(1, as);
  if (lane == 0) {
    sh.h = h;
    sh.h6 = (float)(h / 6.0);
    sh.bad_m = 0;
  }
  __syncthreads();
  int ran = 0;
  bool bad = false, done = false;
  double c6 = h / 6.0, next_h = h, next_c6 = c6;
  int next_clipped = 0;
  // Stage ST of step `it`: ka of this stage's input from its m^- sums (a run's
  // first one is in the control block), then the amplitude of the next stage.
  auto stage = [&](auto st, int it) {
    constexpr int ST = decltype(st)::value;
    constexpr int rb = (ST - 1) & 1, wb = ST & 1;
    if (!split) {
      if (rec && mode) {
        MMG double* ra = rec_a + ((size_t)(ri0 + it) * 4 + (ST - 1)) * N * 2;
        ra[2 * n] = ST == 1 ? a.r : as.r;
        ra[2 * n + 1] = ST == 1 ? a.i : as.i;
      }
      if (ST == 1) {
        ksum = k0;
        as = {a.r + 0.5 * h * k0.r, a.i + 0.5 * h * k0.i};
      } else {
        const Cplx f = rhs(ST == 4 ? t + h : t + 0.5 * h, as, gather(rb));
        const double w = ST < 4 ? 2.0 : 1.0;
        ksum.r += w * f.r;
        ksum.i += w * f.i;
        if (ST < 4) {
          const double cn = (ST == 3) ? h : 0.5 * h;
          as = {a.r + cn * f.r, a.i + cn * f.i};
        } else {
          as = {a.r + c6 * ksum.r, a.i + c6 * ksum.i};
        }
      }
      publish(wb, as);
      // the envelope of the stages to come, so that it is ready behind the sums
      if (ST == 1) envelope(t + 0.5 * h);
      if (ST == 3) envelope(t + h);
    }
    if (ST == 2) {
      // the plan of the next step, taken if this one is accepted
      const double tn = clipped ? t_end : t + h;
      const double rem = t_end - tn;
      next_h = dt_fixed;
      next_clipped = 0;
      if (next_h * (1.0 + 1e-9) >= rem) {
        next_h = rem;
        next_clipped = 1;
      }
      if (next_h != h) next_c6 = next_h / 6.0;
      if (lane == 0) {
        sh.bad_m = 0;                                // (the previous step's flag was read before stage 1)
        sh.done = tn >= t_end;
      }
    }
    if (ST == 4) {
      const bool ba = __any(mode && !(isfinite(as.r) && isfinite(as.i)));
      if (lane == 0) {
        sh.bad_a = ba;
        sh.h = next_h;
        sh.h6 = (float)next_c6;
      }
    }
    __syncthreads();
  };
  // one pass past the last step forms what needs m^- of the last state
  for (int it = 0;; ++it) {
    const bool last = it == steps || done;
    if (!split && it > 0) {
      mm = gather(0);
      k0 = rhs(t, a, mm);
      sample();
    }
    if (last) break;
    stage(std::integral_constant<int, 1>{}, it);
    stage(std::integral_constant<int, 2>{}, it);
    stage(std::integral_constant<int, 3>{}, it);
    stage(std::integral_constant<int, 4>{}, it);
    bad = sh.bad_m || sh.bad_a;
    if (bad) break;
    ran = it + 1;
    done = sh.done;
    a = as;
    t = clipped ? t_end : t + h;
    accepted += 1;
    hmin = fmin(hmin, h);
    hmax = fmax(hmax, h);
    if (!done) {
      h = next_h;
      c6 = next_c6;
      clipped = next_clipped;
    }
    if (split) {
      mm = gather(0);
      sample();
      if (!done) {
        // the cavity's own RK4 step with m^- held feeds every LLG stage of the next step
        Cplx f = k0 = rhs(t, a, mm);
        ksum = k0;
#pragma unroll 1
        for (int s = 1; s <= 3; ++s) {
          const double c = (s == 3) ? h : 0.5 * h;
          as = {a.r + c * f.r, a.i + c * f.i};
          f = rhs(t + c, as, mm);
          const double w = s == 3 ? 1.0 : 2.0;
          ksum.r += w * f.r;
          ksum.i += w * f.i;
        }
        as = {a.r + c6 * ksum.r, a.i + c6 * ksum.i};
        publish(0, as);
        publish(1, as);
      }
      __syncthreads();
    }
  }
  if (bad || !split) as = a;
  if (mode) {
    C0->a[n][0] = a.r;
    C0->a[n][1] = a.i;
    C0->as[n][0] = as.r;
    C0->as[n][1] = as.i;
    C0->ka[0][n][0] = k0.r;
    C0->ka[0][n][1] = k0.i;
    C0->mm1[n][0] = mm.r;
    C0->mm1[n][1] = mm.i;
  }
  if (lane == 0) {
    C0->t = t;
    C0->h = h;
    C0->clipped = clipped;
    C0->accepted = accepted;
    C0->dt_min_seen = hmin;
    C0->dt_max_seen = hmax;
    C0->cur = cur0 ^ (ran & 1);
    C0->trace_n = trace_n;
    C0->trace_steps = trace_steps;
    if (rec) C0->rec_index = ri0 + ran;
    if (bad) C0->status = -6;
    C0->done = (bad || done) ? 1 : 0;
  }
}

// S sublattices, up to C cells per cell thread; PROF: the instances with mode
// profiles (the others of the list are left alone).  One workgroup per entry of
// `list` (instance indices); blockDim.x = cell threads + 64.  The two roles
// meet at the same number of barriers: one at the start, four per step, a
// fifth per step in the operator-split scheme.
template <int S, int C, bool PROF>
__global__ __launch_bounds__(SM_T) void k_small_rk4(const InstDesc* __restrict__ descs,
                                                    const int* __restrict__ list, int steps) {
  __shared__ SmallShared<C> sh;
  extern __shared__ float4 sm[];                   // [2][S][512 C] stage inputs, then [N][ncell] profiles
  const InstDesc& D = descs[list[blockIdx.x]];
  const InstCtl* const C0 = D.ctl;
  if (C0->done || (D.profiled != 0) != PROF) return;
  const int ri0 = C0->rec_index, cur0 = C0->cur;
  for (int e = threadIdx.x; e < (int)(sizeof(sh.sum) / sizeof(double)); e += blockDim.x) (&sh.sum[0][0][0][0])[e] = 0.0;
  __syncthreads();                                 // (also: every wavefront has read the control block)
  const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (role == (int)(blockDim.x >> 6) - 1) __builtin_amdgcn_s_setprio(3);   // the cells wait for it
  if (role == (int)(blockDim.x >> 6) - 1) small_cavity<S, C, PROF>(D, sh, steps, ri0, cur0);
  else small_cells<S, C, PROF>(D, sh, sm, steps, ri0, cur0);
}

}  // namespace mmk

hipError_t mmk_launch_small_rk4(int S, int ncell, bool profiled, int nblocks, size_t lds, const InstDesc* d, const int* list, int steps,
                                hipStream_t s) {
  const int threads = (ncell < mmk::SM_CELLS_T ? (ncell + 63) / 64 * 64 : mmk::SM_CELLS_T) + 64;
#define MM_SMALL(A, B)                                                                                     \
  do {                                                                                                     \
    if (profiled)                                                                                          \
      MM_LAUNCH((mmk::k_small_rk4<A, B, true>), dim3(nblocks), dim3(threads), lds, s, d, list, steps);     \
    else                                                                                                   \
      MM_LAUNCH((mmk::k_small_rk4<A, B, false>), dim3(nblocks), dim3(threads), lds, s, d, list, steps);    \
  } while (0)
  const int per = (ncell + mmk::SM_CELLS_T - 1) / mmk::SM_CELLS_T;
  if (per < 1 || per > 4 || ncell > MMI_SMALL_CELLS) return hipErrorInvalidValue;
  if (S == 1) {
    if (per == 1) MM_SMALL(1, 1);
    else if (per == 2) MM_SMALL(1, 2);
    else MM_SMALL(1, 4);
  } else {
    if (per == 1) MM_SMALL(2, 1);
    else if (per == 2) MM_SMALL(2, 2);
    else MM_SMALL(2, 4);
  }
#undef MM_SMALL
  return hipGetLastError();
}

hipError_t mmk_set_small_lds_limits() {
  hipError_t e = hipSuccess;
#define MM_SMALL_ATTR(A, B)                                                                              \
  if (e == hipSuccess)                                                                                   \
    e = hipFuncSetAttribute((const void*)mmk::k_small_rk4<A, B, false>,                                   \
                            hipFuncAttributeMaxDynamicSharedMemorySize, MMI_SMALL_LDS);                    \
  if (e == hipSuccess)                                                                                   \
    e = hipFuncSetAttribute((const void*)mmk::k_small_rk4<A, B, true>,                                    \
                            hipFuncAttributeMaxDynamicSharedMemorySize, MMI_SMALL_LDS);
  MM_SMALL_ATTR(1, 1) MM_SMALL_ATTR(1, 2) MM_SMALL_ATTR(1, 4)
  MM_SMALL_ATTR(2, 1) MM_SMALL_ATTR(2, 2) MM_SMALL_ATTR(2, 4)
#undef MM_SMALL_ATTR
  return e;
}
