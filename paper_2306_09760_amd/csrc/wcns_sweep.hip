// The sweep kernel and its launchers: one launch per direction (see
// wcns_sweep_tile.hpp for a tile).
#include <hip/hip_runtime.h>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"
#include "wcns_sweep_tile.hpp"

namespace wcns {

// The sweep kernel: one tile per workgroup, in XCD-aware order.  A batch
// launch with a live list (BatchArgs::live) maps workgroup b to list
// position xcd_tile(b, nlive) (each XCD a contiguous range of the list, so
// neighbouring tiles, which share halo lines, run on one L2 at about the same
// time) and workgroups b >= nlive leave after reading the count: the list is
// read on the device, so the host launches the same grid whatever the number
// of live tiles.
template <int NV, int DIR, bool BATCH, int SPEC, int TM, int W>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(sweep_waves(NV, TM * W, SPEC))))
    sweep_kernel(SweepKernArgs k) {
  extern __shared__ double smem[];
  const SweepArgs& a = k.a;
  const BatchArgs& b = k.b;
  const TileGeom& g = k.g;
  const int mode = k.mode;
  int64_t tile;
  if (BATCH && b.live) {
    const int n = *b.nlive;
    // a launch capped below the list's length leaves tiles out: say so
    if (n > (int)gridDim.x && blockIdx.x == 0 && threadIdx.x == 0 && a.status)
      atomicOr(a.status, 2);
    if ((int)blockIdx.x >= n) return;
    tile = b.live[xcd_tile(blockIdx.x, n)];
  } else {
    if ((int64_t)blockIdx.x >= g.ntiles) return;
    tile = xcd_tile(blockIdx.x, g.ntiles);
  }
  sweep_tile<NV, DIR, BATCH, SPEC, TM, W>(a, b, g, mode, tile, smem);
}

// --------------------------------------------------------------- launchers --
// Compiled tile shapes: x direction and batch tm in {128, 256}; y/z (tm, w)
// in {(16, 8), (32, 4), (32, 8), (64, 4), (128, 2), (256, 1)}.
bool sweep_shape_ok(int nv, int dir, int tm, int w) {
  if (dir == 0) return w == 1 && (tm == 128 || tm == 256);
  const bool known = (tm == 16 && w == 8) || (tm == 32 && w == 4) || (tm == 32 && w == 8) ||
                     (tm == 64 && w == 4) || (tm == 128 && w == 2) || (tm == 256 && w == 1);
  if (!known) return false;
  return sizeof(double) * sweep_lds_doubles(nv, tm, w) <= 64 * 1024;
}

template <int NV, int DIR, bool BATCH, int SPEC, int TM, int W>
static hipError_t sweep_launch(const SweepArgs& a, const BatchArgs& b, const TileGeom& g,
                               int mode, size_t lds, hipStream_t s) {
  const SweepKernArgs k{a, b, g, mode};
  hipLaunchKernelGGL((sweep_kernel<NV, DIR, BATCH, SPEC, TM, W>),
                     dim3((unsigned)(g.grid > 0 ? g.grid : g.ntiles)), dim3(256), lds, s, k);
  return hipGetLastError();
}

template <int NV, int DIR, bool BATCH, int TM, int W>
static hipError_t sweep_go(const SweepArgs& a, const BatchArgs& b, const TileGeom& g, int mode,
                           hipStream_t s) {
  const size_t lds = sizeof(double) * SweepLayout<NV, TM, W>::lds_doubles;
  const int spec = sweep_spec_of(a.ip);
  if constexpr (!BATCH) {
    if (spec == SPEC_PLAIN_FE)
      return sweep_launch<NV, DIR, BATCH, SPEC_PLAIN_FE, TM, W>(a, b, g, mode, lds, s);
    if (spec == SPEC_PLAIN)
      return sweep_launch<NV, DIR, BATCH, SPEC_PLAIN, TM, W>(a, b, g, mode, lds, s);
  }
  switch (spec) {
    case SPEC_FE: return sweep_launch<NV, DIR, BATCH, SPEC_FE, TM, W>(a, b, g, mode, lds, s);
    case SPEC_FE_SAT: return sweep_launch<NV, DIR, BATCH, SPEC_FE_SAT, TM, W>(a, b, g, mode, lds, s);
    case SPEC_JS: return sweep_launch<NV, DIR, BATCH, SPEC_JS, TM, W>(a, b, g, mode, lds, s);
    case SPEC_Z: return sweep_launch<NV, DIR, BATCH, SPEC_Z, TM, W>(a, b, g, mode, lds, s);
    case SPEC_PFE: return sweep_launch<NV, DIR, BATCH, SPEC_PFE, TM, W>(a, b, g, mode, lds, s);
    default: return sweep_launch<NV, DIR, BATCH, SPEC_GENERIC, TM, W>(a, b, g, mode, lds, s);
  }
}

template <int NV, int DIR, bool BATCH>
static hipError_t sweep_shape(const SweepArgs& a, const BatchArgs& b, const TileGeom& g, int mode,
                              hipStream_t s) {
  if constexpr (DIR == 0) {
    if (g.tm == 128) return sweep_go<NV, DIR, BATCH, 128, 1>(a, b, g, mode, s);
    return sweep_go<NV, DIR, BATCH, 256, 1>(a, b, g, mode, s);
  } else {
    if (g.tm == 16) return sweep_go<NV, DIR, BATCH, 16, 8>(a, b, g, mode, s);
    if (g.w == 4 && g.tm == 32) return sweep_go<NV, DIR, BATCH, 32, 4>(a, b, g, mode, s);
    if (g.tm == 32) return sweep_go<NV, DIR, BATCH, 32, 8>(a, b, g, mode, s);
    if (g.tm == 128) return sweep_go<NV, DIR, BATCH, 128, 2>(a, b, g, mode, s);
    if (g.tm == 256) return sweep_go<NV, DIR, BATCH, 256, 1>(a, b, g, mode, s);
    return sweep_go<NV, DIR, BATCH, 64, 4>(a, b, g, mode, s);
  }
}

hipError_t launch_sweep(int nv, int dir, const SweepArgs& a, int mode, int tm, int w,
                        hipStream_t stream) {
  if (!sweep_shape_ok(nv, dir, tm, w)) return hipErrorInvalidConfiguration;
  const TileGeom g = make_geom(dir, a.n, a.diff, tm, w);
  if (g.ntiles > 0x7fffffff) return hipErrorInvalidConfiguration;
  BatchArgs b{};
#define WCNS_S(NVV, DD) \
  if (nv == NVV && dir == DD) return sweep_shape<NVV, DD, false>(a, b, g, mode, stream);
  WCNS_S(1, 0) WCNS_S(1, 1) WCNS_S(1, 2)
  WCNS_S(3, 0)
  WCNS_S(4, 0) WCNS_S(4, 1)
  WCNS_S(5, 0) WCNS_S(5, 1) WCNS_S(5, 2)
#undef WCNS_S
  return hipErrorInvalidValue;
}

hipError_t launch_batch_sweep(const SweepArgs& a, const BatchArgs& b, int mode, int tm,
                              hipStream_t stream, int32_t cap) {
  if (!sweep_shape_ok(3, 0, tm, 1)) return hipErrorInvalidConfiguration;
  TileGeom g{};
  g.tm = tm;
  g.w = 1;
  g.lw = 0;
  g.ltmw = 0;
  g.tl = tm - (a.diff ? 5 : 3);
  g.segs = 1;
  g.xgroups = 1;
  g.ntiles = b.ntiles;
  g.lines = 0;
  g.inv_line = 0.0;
  g.grid = (cap > 0 && b.live && cap < b.ntiles) ? cap : 0;
  return sweep_shape<3, 0, true>(a, b, g, mode, stream);
}

}  // namespace wcns
