// State, trace and run parameters between the host and small instances.
//
// A fetch of a few kilobytes with hipMemcpy costs about 15 us whatever its
// size, and a state or a trace took two to four of them (the control block
// says which buffer holds the state, and how many samples there are), so a
// sweep of 41 small instances spent 8 of 12.7 ms on them.  Each of these
// kernels does the whole exchange with one pinned buffer of the host, which it
// reads or writes over the bus: one launch and one wait.  Of a transfer of
// more than 256 KB the copy engine's rate counts, and it stays with hipMemcpy.
#include <cstddef>
#include <cstring>

#include "mm_internal.h"
#include "mm_host.h"
#include "launch.h"

namespace {

constexpr int IO_T = 256;
static_assert(sizeof(InstCtl) % 8 == 0 && offsetof(InstCtl, trace_n) % 8 == 0 && offsetof(InstCtl, rec_index) % 8 == 0,
              "the control block is copied in 8-byte words");
constexpr int kCtlWords = sizeof(InstCtl) / 8;

// control block and, with n > 0, the n floats of the current state
__global__ __launch_bounds__(IO_T) void k_state_out(const InstCtl* C, const float* y0, const float* y1, int n, char* dst) {
  const int i0 = blockIdx.x * IO_T + threadIdx.x, step = gridDim.x * IO_T;
  for (int i = i0; i < kCtlWords; i += step) ((long long*)dst)[i] = ((const long long*)C)[i];
  const float* y = C->cur ? y1 : y0;
  for (int i = i0; i < n; i += step) ((float*)(dst + sizeof(InstCtl)))[i] = y[i];
}

// the same into the device, but for the trace settings, which stay
__global__ __launch_bounds__(IO_T) void k_state_in(InstCtl* C, float* y0, int n, const char* src) {
  constexpr int t0 = offsetof(InstCtl, trace_n) / 8, t1 = offsetof(InstCtl, rec_index) / 8;
  const int i0 = blockIdx.x * IO_T + threadIdx.x, step = gridDim.x * IO_T;
  for (int i = i0; i < kCtlWords; i += step)
    if (i < t0 || i >= t1) ((long long*)C)[i] = ((const long long*)src)[i];
  for (int i = i0; i < n; i += step) y0[i] = ((const float*)(src + sizeof(InstCtl)))[i];
}

// sample count, then times, amplitudes and m^- of at most `most` samples, at
// the stride `most`; trace: device arrays of capacity cap, n1 = max(N, 1)
__global__ __launch_bounds__(IO_T) void k_trace_out(const InstCtl* C, const double* trace, long long cap, int N, int n1,
                                                    long long most, double* dst) {
  const long long have = C->trace_n, cnt = have < most ? have : most;
  const long long i0 = (long long)blockIdx.x * IO_T + threadIdx.x, step = (long long)gridDim.x * IO_T;
  if (i0 == 0) dst[0] = (double)cnt;
  const double *a = trace + cap, *m = trace + cap * (1 + 2 * n1);
  double *ot = dst + 1, *oa = ot + most, *om = oa + 2 * N * most;
  for (long long i = i0; i < cnt; i += step) ot[i] = trace[i];
  for (long long i = i0; i < cnt * 2 * N; i += step) {
    oa[i] = a[i];
    om[i] = m[i];
  }
}

__global__ void k_run_begin(const MmRunArgs* args, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) mm_apply_run(*args[i].ctl, args[i]);
}

__global__ void k_run_stats(InstCtl* const* ctl, MmRunStats* out, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const InstCtl* C = ctl[i];
  out[i] = {C->accepted, C->rejected, C->t, C->dt, C->dt_fixed, C->dt_min_seen, C->dt_max_seen, C->status};
}

__global__ __launch_bounds__(IO_T) void k_to_float(const double* src, float* dst, size_t n) {
  const size_t step = (size_t)gridDim.x * IO_T;
  for (size_t i = (size_t)blockIdx.x * IO_T + threadIdx.x; i < n; i += step) dst[i] = (float)src[i];
}

unsigned io_blocks(size_t n, unsigned most) {
  const size_t b = (n + IO_T - 1) / IO_T;
  return (unsigned)(b < 1 ? 1 : b < most ? b : most);
}

}  // namespace

// All on the null stream, as the copies they take the place of; the caller waits.
hipError_t mmk_launch_state_out(const InstCtl* c, const float* y0, const float* y1, int n, char* dst) {
  MM_LAUNCH(k_state_out, dim3(io_blocks(n, 64)), dim3(IO_T), 0, nullptr, c, y0, y1, n, dst);
  return hipGetLastError();
}
hipError_t mmk_launch_state_in(InstCtl* c, float* y0, int n, const char* src) {
  MM_LAUNCH(k_state_in, dim3(io_blocks(n, 64)), dim3(IO_T), 0, nullptr, c, y0, n, src);
  return hipGetLastError();
}
hipError_t mmk_launch_trace_out(const InstCtl* c, const double* trace, long long cap, int N, long long most, double* dst) {
  const int n1 = N > 1 ? N : 1;
  MM_LAUNCH(k_trace_out, dim3(io_blocks(most * n1 * 2, 64)), dim3(IO_T), 0, nullptr, c, trace, cap, N, n1, most, dst);
  return hipGetLastError();
}
hipError_t mmk_launch_run_begin(const MmRunArgs* args, int count) {
  MM_LAUNCH(k_run_begin, dim3((count + 63) / 64), dim3(64), 0, nullptr, args, count);
  return hipGetLastError();
}
hipError_t mmk_launch_run_stats(InstCtl* const* ctl, MmRunStats* out, int count) {
  MM_LAUNCH(k_run_stats, dim3((count + 63) / 64), dim3(64), 0, nullptr, ctl, out, count);
  return hipGetLastError();
}
hipError_t mmk_launch_to_float(const double* src, float* dst, size_t n) {
  MM_LAUNCH(k_to_float, dim3(io_blocks(n, 2048)), dim3(IO_T), 0, nullptr, src, dst, n);
  return hipGetLastError();
}
