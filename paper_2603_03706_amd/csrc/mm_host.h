// Host-side helpers of the library (setup and launch wrappers).
#pragma once
#include <hip/hip_runtime.h>
#include <mutex>
#include <vector>

#include "mm_internal.h"

namespace mmh {
void demag_tensor(double X, double Y, double Z, double dx, double dy, double dz, double* out6);
int padded(int n);
void kernel_spectrum(int nx, int ny, int nz, double dx, double dy, double dz, std::vector<float>& out);
}  // namespace mmh

// Parameters of a run, applied to an instance's control block at its start.
struct MmRunArgs {
  InstCtl* ctl;
  double T, t_end_abs, tol, dt_fixed, dt_min, dt_max;   // t_end = t_end_abs if finite, t + T if T > 0, else unbounded
  int rec_index, sampling, trace_on, pad;               // sampling: the trace settings below are new
  double trace_dt;
  long long trace_max, trace_stride;
};
// What a run leaves for the instance's statistics.
struct MmRunStats {
  long long accepted, rejected;
  double t, dt, dt_fixed, dt_min_seen, dt_max_seen;
  int status;
};
__host__ __device__ inline void mm_apply_run(InstCtl& h, const MmRunArgs& r) {
  h.t_end = r.t_end_abs - r.t_end_abs == 0.0 ? r.t_end_abs : r.T > 0 ? h.t + r.T : 1e300;
  h.tol = r.tol;
  h.dt_fixed = r.dt_fixed;
  h.dt_min = r.dt_min;
  h.dt_max = r.dt_max;
  h.done = 0;
  h.idle = 0;
  h.status = 0;
  // the run-start stage kernel evaluates the feedback from the stage
  // amplitude: it must be the amplitude of the state the run starts from
  // (a previous run leaves the next stage input there, mm_set_a and
  // mm_set_state set a alone)
  for (int n = 0; n < MMI_MAX_MODES; ++n) {
    h.as[n][0] = h.a[n][0];
    h.as[n][1] = h.a[n][1];
  }
  h.rec_index = r.rec_index;
  if (r.sampling) {
    h.trace_on = r.trace_on;
    h.trace_started = 0;
    h.trace_n = 0;
    h.trace_steps = 0;
    h.trace_max = r.trace_max;
    h.trace_dt = r.trace_dt;
    h.trace_stride = r.trace_stride;
  }
}
// exchanges with the host through pinned memory, on the null stream (kernels_io.hip)
hipError_t mmk_launch_state_out(const InstCtl* c, const float* y0, const float* y1, int n, char* dst);
hipError_t mmk_launch_state_in(InstCtl* c, float* y0, int n, const char* src);
hipError_t mmk_launch_trace_out(const InstCtl* c, const double* trace, long long cap, int N, long long most, double* dst);
hipError_t mmk_launch_run_begin(const MmRunArgs* args, int count);
hipError_t mmk_launch_run_stats(InstCtl* const* ctl, MmRunStats* out, int count);
hipError_t mmk_launch_to_float(const double* src, float* dst, size_t n);

hipError_t mmk_launch_xfwd_cells(int method, int stage, int nblocks, const InstDesc* descs, const int* wg,
                                 const float2* tw, size_t lds, hipStream_t s);
hipError_t mmk_launch_stage(int method, int stage, bool final_pass, int nblocks, int count,
                            const InstDesc* descs, const int* wg, const float2* tw, size_t lds,
                            hipStream_t stream);
// `steps` whole RK4 steps of nblocks small instances (indices in list), each of S sublattices and at most ncell
// (<= MMI_SMALL_CELLS) cells; profiled: steps those with mode profiles, else those without; lds: dynamic LDS, the largest of the instances'
hipError_t mmk_launch_small_rk4(int S, int ncell, bool profiled, int nblocks, size_t lds, const InstDesc* d, const int* list, int steps,
                                hipStream_t s);
hipError_t mmk_set_small_lds_limits();
// `steps` reverse steps of instance `inst` of S sublattices and ncell <= 1024 cells;
// lds: dynamic LDS, with grad u (g_lds) and the profiles (u_lds) in it where they are kept there
hipError_t mmk_launch_small_adj(int S, int ncell, size_t lds, bool g_lds, bool u_lds, const InstDesc* d, int inst, int steps,
                                hipStream_t s);
hipError_t mmk_set_small_adj_lds_limits();
// x passes with lines in registers: Px = 4 MX, MX in {4, 8, 16, 32}; dir +1 forward (method,
// stage select the stage input), -1 inverse; work items are tiles of 128 rows
hipError_t mmk_launch_fft_xr(int dir, int MX, int nblocks, const InstDesc* d, const WorkItem* w, int method,
                             int stage, const float2* tw, hipStream_t s);
hipError_t mmk_launch_fft_xf(int W, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                             int method, int stage, const float2* tw, hipStream_t s);
hipError_t mmk_launch_fft_xi(int W, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                             const float2* tw, hipStream_t s);
// fused y-z with lines in registers: Py = 4 MY, Pz = 4 MZ, MY in {4,8,16,32}, MZ in {4,8,16}
hipError_t mmk_launch_fft_yzr(int MY, int MZ, int nblocks, size_t lds, const InstDesc* d,
                              const WorkItem* w, const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0,
                              int fstage = 0);
// the same with eight lanes per z column (512 threads): MY in {4,8,16,32}, MZ in {8,16}.
// nfinal > 0 appends that many workgroups that run the finalisation of stage
// fstage of method fmethod for instances 0 .. nfinal - 1.
hipError_t mmk_launch_fft_yz8(int MY, int MZ, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0,
                              int fstage = 0);
hipError_t mmk_launch_fft_yzx(int MY, int MZ, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0,
                              int fstage = 0);
int mmk_yzx_pad();
// k_fft_yzx for padded (py, pz) carries the real planes kx = 0 and Px/2 of an
// instance in one work item (item 0; no item Px/2), with 6 pz float2 more LDS
bool mmk_yzx_pairs(int py, int pz);
// y-z of few z planes: padded z of 4, 8 or 16 with padded y of 8..256, or one z plane with padded y of 8..512;
// mmk_yzs_lds is 0 for other shapes
size_t mmk_yzs_lds(int py, int pz);
hipError_t mmk_launch_fft_yzs(int py, int pz, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0, int fstage = 0);
hipError_t mmk_set_short_lds_limits();
// y-z in two halves of the ky range (2 kx items per instance and the planes 0 and Px/2 in one pair of items):
// padded y of 64..256, padded z of 32 or 64; mmk_yzh_lds is 0 for other shapes
size_t mmk_yzh_lds(int py, int pz);
hipError_t mmk_launch_fft_yzh(int py, int pz, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0, int fstage = 0);
hipError_t mmk_launch_fft_ysx(int dir, int py, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0,
                              int fstage = 0);
int mmk_sx_rows(int py);
hipError_t mmk_launch_fft_yz(int TK, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                             const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0, int fstage = 0);
hipError_t mmk_launch_fft_y(int dir, int W, int nblocks, size_t lds, const InstDesc* d,
                            const WorkItem* w, const float2* tw, hipStream_t s, int nfinal = 0, int fmethod = 0,
                            int fstage = 0);
hipError_t mmk_launch_fft_zc(int TW, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                             const float2* tw, hipStream_t s);
// Whether finalisations ride on a launch of the fused or the register y-z kernel or of the split y forward pass
// (nblocks workgroups, lds bytes each, on a device of cus CUs): where it keeps as many workgroups in flight with them as without
enum { MMK_RIDE_FUSED, MMK_RIDE_REGISTER, MMK_RIDE_Y };
bool mmk_final_rides(int kind, int py, int pz, int nblocks, size_t lds, int cus);
hipError_t mmk_set_lds_limits();
hipError_t mmk_launch_adj(int kind, bool dp, int stage, int nblocks, int count, const InstDesc* d, const int* wg,
                          hipStream_t s, const float2* tw = nullptr, size_t lds = 0);
hipError_t mmk_launch_gather_done(int count, const InstDesc* d, int* out, hipStream_t s);
// the no-allocation run: this device's fixed scratch (address and size), the
// per-device lock that serialises such runs, and a zero-fill kernel
hipError_t mmk_noalloc_scratch(int dev, void** ptr, size_t* bytes);
std::mutex& mmk_noalloc_lock(int dev);
hipError_t mmk_launch_fill_zero(void* p, size_t bytes, hipStream_t s);
