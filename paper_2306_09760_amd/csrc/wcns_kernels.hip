// Time-step and elementwise kernels of the WCNS-FE library on gfx950 (the
// directional sweeps are in wcns_sweep.hip).
//
//  cfl      sum_d (|u_d| + c)/h_d, its maximum and dt = cfl / max: one block for
//           a small grid, else per-block maxima and one block that turns them
//           into dt (both deterministic).
#include <hip/hip_runtime.h>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

// --------------------------------------------------------------------- CFL --
// Maximum of a block of WAVES wavefronts; valid in every thread (bit patterns:
// a NaN reaches dt from any lane, see wave_max_bits).
template <int WAVES>
__device__ __forceinline__ unsigned long long block_max_bits(unsigned long long m) {
  __shared__ unsigned long long red[WAVES];
  m = wave_max_bits(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) m = umax64(m, red[w]);
  return m;
}

// Maximum wave rate over the nodes first, first + step, ..
template <int NV>
__device__ __forceinline__ unsigned long long rate_max(const double* __restrict__ U, int64_t npts,
                                                       double gamma, const double (&ih)[3],
                                                       double adv_rate, int64_t first, int64_t step) {
  unsigned long long m = 0;
  if constexpr (NV == 1) {
    m = __builtin_bit_cast(unsigned long long, adv_rate);
  } else {
#pragma unroll 4
    for (int64_t i = first; i < npts; i += step) {
      double u[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) u[v] = U[v * npts + i];
      m = umax64(m, __builtin_bit_cast(unsigned long long, wave_rate<NV - 2>(u, gamma, ih)));
    }
  }
  return m;
}

// ONE: a single block, which writes dt to `out`; else each block its maximum.
template <int NV, bool ONE>
__global__ void __launch_bounds__(ONE ? 1024 : 256)
    cfl_kernel(const double* __restrict__ U, int64_t npts, double gamma, double ih0, double ih1,
               double ih2, double adv_rate, double cfl, double* __restrict__ out) {
  constexpr int NT = ONE ? 1024 : 256;
  const double ih[3] = {ih0, ih1, ih2};
  const unsigned long long m = block_max_bits<NT / 64>(
      rate_max<NV>(U, npts, gamma, ih, adv_rate, (int64_t)blockIdx.x * NT + threadIdx.x,
                   (int64_t)gridDim.x * NT));
  const double r = __builtin_bit_cast(double, m);
  if (threadIdx.x == 0) out[blockIdx.x] = ONE ? cfl / r : r;
}

__global__ void __launch_bounds__(256) cfl_final_kernel(const double* __restrict__ partial,
                                                        int n, double cfl,
                                                        double* __restrict__ dt) {
  unsigned long long m = 0;
  for (int i = threadIdx.x; i < n; i += 256)
    m = umax64(m, __builtin_bit_cast(unsigned long long, partial[i]));
  m = block_max_bits<4>(m);
  if (threadIdx.x == 0) dt[0] = cfl / __builtin_bit_cast(double, m);
}

// The batch maxima use wave_max_bits (wcns_device.hpp).
__device__ __forceinline__ void batch_dt_store(const BatchArgs& b, int p, const BatchDt& d,
                                               double* t, int32_t* status) {
  b.dtp[p] = d.dt;
  t[p] = d.tn;
  if (d.bad && status) atomicOr(status, 1);
}

// One block per problem: the maximum wave rate of its nodes, then batch_dt.
// wmax, when given, is cleared for the fused maximum of the step's last stage.
// The time goes from t to t_out (the same array, or another).
__global__ void __launch_bounds__(256) batch_cfl_kernel(const double* __restrict__ U,
                                                        int64_t total, BatchArgs b,
                                                        double gamma, const double* t,
                                                        double* t_out, double t_end, double cfl,
                                                        unsigned long long* wmax,
                                                        int32_t* status, int32_t* nlive) {
  __shared__ unsigned long long red[4];
  const int p = blockIdx.x;
  if (nlive && p == 0 && threadIdx.x == 0) *nlive = 0;
  if (wmax && threadIdx.x == 0) wmax[p] = 0;
  if (!(t[p] < t_end)) {  // uniform: the whole block leaves
    if (threadIdx.x == 0) {
      b.dtp[p] = 0.0;
      t_out[p] = t[p];
    }
    return;
  }
  const int64_t o0 = b.offset[p], o1 = b.offset[p + 1];
  const double ih[1] = {b.ih[p]};
  unsigned long long m = 0;
  // (four nodes' loads in flight: a problem's maximum is a chain of trips to memory)
#pragma unroll 4
  for (int64_t i = o0 + threadIdx.x; i < o1; i += 256) {
    double u[3] = {U[i], U[total + i], U[2 * total + i]};
    const unsigned long long r = __builtin_bit_cast(unsigned long long, wave_rate<1>(u, gamma, ih));
    m = r > m ? r : m;
  }
  m = wave_max_bits(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) m = red[w] > m ? red[w] : m;  // m = red[0] here
    batch_dt_store(b, p, batch_dt(__builtin_bit_cast(double, m), t[p], t_end, cfl), t_out, status);
  }
}

// The same dt from the maxima that the previous step's last stage took as it
// wrote the state (sweep kernel, SweepArgs::wmax); clears them for this
// step's.  One thread per problem.
__global__ void __launch_bounds__(256) batch_dt_kernel(BatchArgs b, double* __restrict__ t,
                                                       double t_end, double cfl,
                                                       unsigned long long* __restrict__ wmax,
                                                       int32_t* status, int32_t* nlive) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (nlive && p == 0) *nlive = 0;
  if (p >= b.nprob) return;
  const double m = __builtin_bit_cast(double, wmax[p]);
  wmax[p] = 0;
  batch_dt_store(b, p, batch_dt(m, t[p], t_end, cfl), t, status);
}

// The live-tile list: lane k tests tile k (live if one of its problems has
// dt > 0); each wavefront appends its live tiles in order with one atomic,
// so the list holds runs of up to 64 consecutive tiles.
__global__ void __launch_bounds__(256) batch_live_kernel(BatchArgs b, int32_t* __restrict__ live,
                                                         int32_t* __restrict__ nlive) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  bool on = false;
  if (k < b.ntiles) {
    const int p1 = b.tile_p1[k];
    for (int p = b.tile_p0[k]; p <= p1 && !on; ++p) on = b.dtp[p] != 0.0;
  }
  const unsigned long long mask = __ballot(on);
  if (mask == 0) return;  // uniform across the wavefront
  const int lane = threadIdx.x & 63;
  int base = 0;
  if (lane == 0) base = atomicAdd(nlive, __popcll(mask));
  base = __shfl(base, 0, 64);
  if (on) live[base + __popcll(mask & ((1ull << lane) - 1ull))] = k;
}

// ------------------------------------------------------------ elementwise --
__global__ void lincomb_kernel(double* __restrict__ out, const double* __restrict__ x, double ax,
                               const double* __restrict__ y, double ay,
                               const double* __restrict__ dt, double ydt, int64_t n) {
  // out = ax*x + (ay + ydt*dt)*y
  const double cy = ay + (dt ? ydt * dt[0] : 0.0);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double r = cy * y[i];
    if (x) r = __builtin_fma(ax, x[i], r);
    out[i] = r;
  }
}

// (-u + u1 + 2 u2) / 3 in one pass (1D 15000 nodes, a four-stage step with a given
// dt: with the sweep's gains 30.0 -> 24.4 us), as lincomb of u and u1 and then of that and u2 round it.
__global__ void rk4_sum_kernel(double* __restrict__ out, const double* __restrict__ u,
                               const double* __restrict__ u1, const double* __restrict__ u2,
                               int64_t n) {
#pragma clang fp contract(off)
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = __builtin_fma(1.0, __builtin_fma(-1.0 / 3.0, u[i], 1.0 / 3.0 * u1[i]), 2.0 / 3.0 * u2[i]);
}

// --------------------------------------------------------------- launchers --
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int cfl_blocks(int64_t npts) {
  int64_t b = ceil_div(npts, 256 * 8);
  if (b < 1) b = 1;
  if (b > 2048) b = 2048;
  return (int)b;
}

// One block where its chain of loads is shorter than a second launch: microseconds,
// two launches -> one block: 1000 nodes 4.3 -> 2.2, 60^2 4.8 -> 3.8, 5000 4.4 -> 3.6,
// 15000 4.5 -> 6.9.  (Advection's rate is a number of the plan's.)
template <int NV>
static hipError_t cfl_go(const double* U, int64_t npts, double gamma, const double (&ih)[3],
                         double adv_rate, double cfl, double* partial, int nblocks, double* dt_out,
                         hipStream_t stream) {
  if (NV == 1 || npts <= 4096) {
    hipLaunchKernelGGL((cfl_kernel<NV, true>), dim3(1), dim3(1024), 0, stream, U, npts, gamma, ih[0],
                       ih[1], ih[2], adv_rate, cfl, dt_out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((cfl_kernel<NV, false>), dim3(nblocks), dim3(256), 0, stream, U, npts, gamma,
                     ih[0], ih[1], ih[2], adv_rate, cfl, partial);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cfl_final_kernel, dim3(1), dim3(256), 0, stream, partial, nblocks, cfl,
                     dt_out);
  return hipGetLastError();
}

hipError_t launch_cfl(int nv, int ndim, const double* U, int64_t npts, double gamma,
                      const double* ih, const double* adv, double cfl, double* partial,
                      int nblocks, double* dt_out, hipStream_t stream) {
  double adv_rate = 0.0;
  for (int d = 0; d < ndim; ++d) adv_rate += (adv[d] < 0 ? -adv[d] : adv[d]) * ih[d];
  const double h[3] = {ih[0], ndim > 1 ? ih[1] : 0.0, ndim > 2 ? ih[2] : 0.0};
#define WCNS_C(NVV) \
  case NVV: return cfl_go<NVV>(U, npts, gamma, h, adv_rate, cfl, partial, nblocks, dt_out, stream);
  switch (nv) {
    WCNS_C(1) WCNS_C(3) WCNS_C(4) WCNS_C(5)
    default: return hipErrorInvalidValue;
  }
#undef WCNS_C
}

hipError_t launch_batch_cfl(const double* U, int64_t total, const BatchArgs& b, double gamma,
                            const double* t, double* t_out, double t_end, double cfl,
                            unsigned long long* wmax, int32_t* status, int32_t* nlive,
                            hipStream_t stream) {
  hipLaunchKernelGGL(batch_cfl_kernel, dim3(b.nprob), dim3(256), 0, stream, U, total, b, gamma,
                     t, t_out, t_end, cfl, wmax, status, nlive);
  return hipGetLastError();
}

hipError_t launch_batch_dt(const BatchArgs& b, double* t, double t_end, double cfl,
                           unsigned long long* wmax, int32_t* status, int32_t* nlive,
                           hipStream_t stream) {
  hipLaunchKernelGGL(batch_dt_kernel, dim3((unsigned)ceil_div(b.nprob, 256)), dim3(256), 0,
                     stream, b, t, t_end, cfl, wmax, status, nlive);
  return hipGetLastError();
}

hipError_t launch_batch_live(const BatchArgs& b, int32_t* live, int32_t* nlive,
                             hipStream_t stream) {
  hipLaunchKernelGGL(batch_live_kernel, dim3((unsigned)ceil_div(b.ntiles, 256)), dim3(256), 0,
                     stream, b, live, nlive);
  return hipGetLastError();
}

static inline int elem_grid(int64_t n) {
  int64_t g = ceil_div(n, 256 * 4);
  if (g < 1) g = 1;
  if (g > 16384) g = 16384;
  return (int)g;
}

hipError_t launch_lincomb(double* out, const double* x, double ax, const double* y, double ay,
                          const double* dt, double ydt, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(lincomb_kernel, dim3(elem_grid(n)), dim3(256), 0, stream, out, x, ax, y, ay,
                     dt, ydt, n);
  return hipGetLastError();
}

hipError_t launch_rk4_sum(double* out, const double* u, const double* u1, const double* u2,
                          int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(rk4_sum_kernel, dim3(elem_grid(n)), dim3(256), 0, stream, out, u, u1, u2, n);
  return hipGetLastError();
}

}  // namespace wcns
