// An SSP-RK3 step of a small 2D or 3D WCNS-Euler problem with one launch per
// stage.
//
// A small problem's step was bound by its launches: two for dt and ndim per
// stage, each about 5.5 us long however small the grid (the launch, the load
// from the other XCDs' results, one tile's chain of phases), with one or two
// tiles per CU.  The sweeps of a stage are only tied by their sum R, so here the
// tiles of all directions run side by side in one launch, each direction's
// residual goes to an array of its own, and the next stage's load phase adds
// them up and combines the stage state as it reads (in emit's order and
// rounding: bitwise the sweeps' step).  The x tiles, whose outputs cover each
// node once, keep U1 and check it, and take U^n's maximum wave rate in stage 1,
// which every tile of stage 2 reduces to dt by itself; U2 is made again
// pointwise in the last kernel.  Four launches instead of eight (2D) or eleven
// (3D), for (ndim + 1) more array reads per loaded node, which the caches hold.
// Microseconds per CFL-limited step, sweeps -> here (FE, one box): 2D 64^2 39.3
// -> 21.6, 128^2 40.0 -> 25.4, 256^2 57.2 -> 44.4; 3D 16^3 66.6 -> 24.7, 32^3
// 85.7 -> 51.6, 48^3 135 -> 109.  At 256^2 a CU has 4.4 tiles at once, in step
// with each other: the vector units issue in half of their slots, and neither
// more waves per SIMD nor fewer change the time.
#include <hip/hip_runtime.h>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"
#include "wcns_sweep_tile.hpp"

namespace wcns {

constexpr int kStageTmX = 128;

constexpr int stage_waves(int spec) {
  return spec == SPEC_GENERIC ? 1 : spec == SPEC_FE_SAT ? 4 : 5;
}

template <int ND, int SPEC, int TM, int W>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(stage_waves(SPEC))))
    stage_kernel(StageKernArgs<ND> k) {
  extern __shared__ double smem[];
  constexpr int NV = ND + 2;
  const BatchArgs b{};
  int w = blockIdx.x;
  if (w < k.nb[0]) {
    if (w >= k.g[0].ntiles) return;
    sweep_tile<NV, 0, false, SPEC, kStageTmX, 1, true>(k.a[0], b, k.g[0], 0,
                                                       xcd_tile(w, k.g[0].ntiles), smem);
    return;
  }
  w -= k.nb[0];
  if (ND == 2 || w < k.nb[1]) {
    if (w >= k.g[1].ntiles) return;
    sweep_tile<NV, 1, false, SPEC, TM, W, true>(
        k.a[1], b, k.g[1], 0, xcd_tile(w, k.g[1].ntiles), smem);
    return;
  }
  if constexpr (ND == 3) {
    w -= k.nb[1];
    if (w >= k.g[2].ntiles) return;
    sweep_tile<NV, 2, false, SPEC, TM, W, true>(
        k.a[2], b, k.g[2], 0, xcd_tile(w, k.g[2].ntiles), smem);
  }
}

// U^(n+1) = 1/3 U^n + 2/3 (U2 + dt R3), U2 = 3/4 U^n + 1/4 (U1 + dt R2) made
// again from what stage 3 read (and kept in U2 when given).
template <int ND>
__global__ void __launch_bounds__(256)
    stage_final_kernel(double* __restrict__ U, const double* __restrict__ U1, double* U2,
                       const double* __restrict__ R2, const double* __restrict__ R3,
                       int64_t rstride, int64_t npts, const double* __restrict__ dtp, double gamma,
                       int32_t* status) {
  constexpr int NV = ND + 2;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npts) return;
  const double dt = *dtp;
  double u2[NV], y[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int64_t e = v * npts + i;
    double r2 = R2[e], r3 = R3[e];
#pragma unroll
    for (int d = 1; d < ND; ++d) {
      r2 += R2[d * rstride + e];
      r3 += R3[d * rstride + e];
    }
    const double u0 = U[e];
    u2[v] = stage_value(0.75, 0.25, u0, U1[e], dt, r2);
    y[v] = stage_value(1.0 / 3.0, 2.0 / 3.0, u0, u2[v], dt, r3);
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if (U2) U2[v * npts + i] = u2[v];
    U[v * npts + i] = y[v];
  }
  if (!physical<NV>(u2, gamma) || !physical<NV>(y, gamma)) flag_status(status);
}

int64_t stage_partials(const int64_t n[3], int diff) {
  return make_geom(0, n, diff, kStageTmX, 1).ntiles;
}

// Up to the sizes at which the extra reads cost what the launches did: measured,
// sweeps (as autotuned) -> here, with a given dt and CFL-limited: 2D 362^2 FE 67.1
// -> 65.2, 74.6 -> 66.8 us, Z 53.9 -> 54.4, 61.2 -> 57.8; 440^2 Z 65.0 -> 69.6,
// 72.5 -> 74.6; 512^2 FE 112 -> 118 (CFL); 3D 64^3 FE 219 -> 212, 225 -> 225, Z
// 165 -> 158, 172 -> 172; 72^3 FE 291 -> 304, 299 -> 325.
bool stage_step_ok(int ndim, int nv, const int64_t n[3]) {
  return ndim > 1 && nv == ndim + 2 && n[0] * n[1] * n[2] <= (int64_t(1) << (ndim == 2 ? 17 : 18));
}

template <int ND, int SPEC, int TM, int W>
static hipError_t stage_go(const StageStep& p, hipStream_t s) {
  constexpr int NV = ND + 2;
  StageKernArgs<ND> k{};
  int64_t blocks = 0;
  for (int d = 0; d < ND; ++d) {
    k.a[d] = p.a[d];
    k.g[d] = d == 0 ? make_geom(0, p.a[0].n, p.a[0].diff, kStageTmX, 1)
                    : make_geom(d, p.a[d].n, p.a[d].diff, TM, W);
    if (k.g[d].ntiles > (int64_t(1) << 28)) return hipErrorInvalidConfiguration;
    k.nb[d] = (int)((k.g[d].ntiles + 7) & ~int64_t(7));
    blocks += k.nb[d];
  }
  k.in.U0 = p.U;
  k.in.U1 = p.U1;
  k.in.rstride = p.rstride;
  k.in.dt_out = p.dt_out;
  k.in.partial = p.partial;
  k.in.npartial = (int32_t)k.g[0].ntiles;
  k.in.status = p.status;
  k.in.cfl = p.cfl;
  for (int d = 0; d < ND; ++d) k.in.ih[d] = p.a[d].ih;
  constexpr size_t lx = SweepLayout<NV, kStageTmX, 1>::lds_doubles;
  constexpr size_t ly = SweepLayout<NV, TM, W>::lds_doubles;
  const size_t lds = sizeof(double) * (lx > ly ? lx : ly);
  for (int st = 1; st <= 3; ++st) {
    k.in.st = st;
    k.in.dt = p.dt ? p.dt : st == 3 ? p.dt_out : nullptr;
    k.in.R = st == 2 ? p.RA : p.RB;
    k.in.Rout = st == 2 ? p.RB : p.RA;
    hipLaunchKernelGGL((stage_kernel<ND, SPEC, TM, W>), dim3((unsigned)blocks), dim3(256), lds, s, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int64_t npts = p.a[0].npts;
  hipLaunchKernelGGL(stage_final_kernel<ND>, dim3((unsigned)ceil_div64(npts, 256)), dim3(256), 0, s,
                     p.U, p.U1, p.U2, p.RB, p.RA, p.rstride, npts, p.dt ? p.dt : p.dt_out,
                     p.a[0].pp.gamma, p.status);
  return hipGetLastError();
}

template <int ND, int TM, int W>
static hipError_t stage_spec(const StageStep& p, hipStream_t s) {
  switch (spec_of(p.a[0].ip)) {
    case SPEC_FE: return stage_go<ND, SPEC_FE, TM, W>(p, s);
    case SPEC_FE_SAT: return stage_go<ND, SPEC_FE_SAT, TM, W>(p, s);
    case SPEC_JS: return stage_go<ND, SPEC_JS, TM, W>(p, s);
    case SPEC_Z: return stage_go<ND, SPEC_Z, TM, W>(p, s);
    case SPEC_PFE: return stage_go<ND, SPEC_PFE, TM, W>(p, s);
    default: return stage_go<ND, SPEC_GENERIC, TM, W>(p, s);
  }
}

// Tiles of the y and z sweeps with segments of tm midpoints by w columns.
static int64_t yz_tiles(int ndim, const SweepArgs* a, int tm, int w) {
  int64_t t = 0;
  for (int d = 1; d < ndim; ++d) t += make_geom(d, a[d].n, a[d].diff, tm, w).ntiles;
  return t;
}

// Segments of 16 midpoints by 8 columns where that takes no more tiles than 32 by
// 4: lines a little longer than a multiple of 29 nodes leave most of their last
// tile empty (32^3, CFL-limited: 1.6 times the tiles, 59.9 -> 51.5 us; 64^3 247 ->
// 221), and at equal counts it is a little faster (128^2 26.3 -> 25.9).
hipError_t launch_stage_step(int ndim, const StageStep& p, hipStream_t s) {
  const bool t16 = yz_tiles(ndim, p.a, 16, 8) <= yz_tiles(ndim, p.a, 32, 4);
  if (ndim == 2) return t16 ? stage_spec<2, 16, 8>(p, s) : stage_spec<2, 32, 4>(p, s);
  return t16 ? stage_spec<3, 16, 8>(p, s) : stage_spec<3, 32, 4>(p, s);
}

}  // namespace wcns
