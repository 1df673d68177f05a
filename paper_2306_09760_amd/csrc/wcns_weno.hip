// Directional sweep of the filtered embedded WENO scheme of App. B on gfx950:
// finite-difference WENO5 with Lax-Friedrichs flux splitting and a
// conservative difference, on the tiles of the WCNS sweep.
//
// A workgroup of 128 GR lanes owns TM midpoints (TM W = 128) of W adjacent columns,
// one midpoint per lane (GR = 2, for small grids: two lanes per midpoint, every
// other field each), and writes the TL = TM - 1 nodes between them.
// Along x the lines are packed end to end (TileGeom::lines, 3 ghost slots per
// side).  Phases:
//   load     the TM+5 nodes of every column, ghosts applied; each lane takes
//            the physical flux and the wave speed |u_n| + c of the nodes it has
//            loaded, and node, flux (but for the density's, a momentum row) and
//            speed go to LDS;
//   mid      the lane's Roe state of nodes m, m+1 (in registers) and splitting
//            speed alpha, the largest wave speed of the six stencil nodes;
//   recon    per field: its projections of F and U at the six nodes, the split
//            fluxes F + alpha U and F - alpha U (twice those of the splitting:
//            the half goes into the difference, eps is taken four times), and
//            the WENO5 reconstruction of the first from the left-biased, of the
//            second from the mirrored stencil;
//   flux     2 F~ = R (f+^ + f-^), the lane's own values;
//   diff     -(F~_{i+1/2} - F~_{i-1/2}) / h, written as R, R+= or a stage.
// Bound by FP64 VALU issue.  One lane reconstructs both sides from projections
// of F and U, 12 NV products per field where a task per side, field and
// midpoint took 30 NV; load | mid and flux | diff are the only barriers.
// Against 256 lanes on 128 midpoints with two tasks per field and midpoint in
// five phases: residual 2D 512^2 0.0598 -> 0.0445 ms, 1024^2 0.179 -> 0.127,
// 2048^2 0.635 -> 0.436, 3D 128^3 0.892 -> 0.497 ms.  256 lanes on 256
// midpoints are 1 % faster from 1024^2 on, and 13 % slower in 3D.
// The weights have the kernels of the WCNS sweep (spec_of): with the run-time ones
// for all but FE, residual 2D 1000 x 993 PFE 0.161 -> 0.101 ms, Z 0.153 -> 0.093, JS
// 0.148 -> 0.088, FE at xi = 1e6 0.187 -> 0.116; 3D 64^3 PFE 0.222 -> 0.103 ms (each
// against the five phases).
// LDS (doubles): sU[NV][TM+5][W] | sF[NV-1][TM+5][W] | sL[TM+5][W] |
// sW[NV][128] | the exp table.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

template <int NV, int TM, int W>
struct WenoLayout {
  static constexpr int ND = NV > 1 ? NV - 2 : 1;
  static constexpr int TN = TM + 5;
  static constexpr int TMW = TM * W;
  static constexpr int SV = TN * W;
  static constexpr int LW = W == 1 ? 0 : W == 2 ? 1 : W == 4 ? 2 : 3;
  static constexpr size_t lds_doubles =
      (size_t)(NV > 1 ? 2 * NV : 1) * SV + (size_t)NV * TMW + 64;
  static_assert(TMW == 128, "one midpoint per lane");
};

// Register budget: the specialisations fit five waves per SIMD, the staircase maps
// four, the run-time weights three (at four they spill).
constexpr int weno_waves(int spec) { return spec == SPEC_GENERIC ? 3 : spec == SPEC_FE_SAT ? 4 : 5; }

template <int NV, int DIR, int SPEC, int TM, int W, int GR>
__global__ void __launch_bounds__(128 * GR) __attribute__((amdgpu_waves_per_eu(weno_waves(SPEC))))
    weno_sweep_kernel(SweepArgs a, TileGeom g, int mode) {
  using L = WenoLayout<NV, TM, W>;
  constexpr int ND = L::ND, TMW = L::TMW, SV = L::SV, LW = L::LW;
  constexpr int NT = TMW * GR;
  constexpr int TL = TM - 1;
  constexpr int G = 3;  // ghosts on each side
  extern __shared__ double smem[];
  double* sU = smem;
  double* sF = sU + NV * SV;                   // rows 1 .. NV-1 of the flux
  double* sL = sF + (NV - 1) * SV;
  double* sW = NV > 1 ? sL + SV : sU + SV;
  double* sX = sW + NV * TMW;  // exp2_tab_entry
  const int tid = threadIdx.x;
  const int mid = tid & (TMW - 1);                                    // the lane's midpoint
  const int grp = GR > 1 ? __builtin_amdgcn_readfirstlane(tid >> 7) : 0;  // and its fields'

  if ((int64_t)blockIdx.x >= g.ntiles) return;
  const int64_t tile = xcd_tile(blockIdx.x, g.ntiles);
  int64_t base = 0, N, stride = 1, i0;
  int ncol = 1;
  BatchTile bt{};
  bool near = true;  // the tile spans at most two lines
  if constexpr (DIR == 0) {
    N = a.n[0];
    i0 = tile * TL;
    bt = line_tile(i0, N, g.lines, G, TL, g.inv_line);
    near = bt.p1 <= bt.p0 + 1;
  } else {
    // column groups fastest: adjacent groups split the same cache lines
    // tile < 2^31 (checked at launch): multiply-shift divisions
    const uint32_t t32 = (uint32_t)tile;
    const uint32_t r32 = g.dxg.div(t32);
    const uint32_t o32 = g.dseg.div(r32);
    const int64_t xg = t32 - r32 * (uint32_t)g.xgroups;
    const int64_t seg = r32 - o32 * (uint32_t)g.segs;
    const int64_t other = o32;
    i0 = seg * TL;
    const int64_t x0 = xg * W;
    ncol = (int)((a.n[0] - x0) < W ? (a.n[0] - x0) : W);
    if constexpr (DIR == 1) {
      N = a.n[1];
      stride = a.n[0];
      base = x0 + other * a.n[0] * a.n[1];
    } else {
      N = a.n[2];
      stride = a.n[0] * a.n[1];
      base = x0 + other * a.n[0];
    }
  }
  const double dt = (mode >= MODE_STAGE) ? *a.dt : 0.0;
  const int64_t nb = i0 - 3;  // position of LDS node 0; midpoint t is m = i0 - 1 + t

  // load: every global read issued before the first LDS write
  constexpr int NIT = (SV + NT - 1) / NT;
  static_assert(NIT <= 2, "a tile holds at most two nodes per lane");
  double buf[NIT][NV];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int idx = tid + it * NT;
    if (idx < SV) {
      const int k = idx >> LW, c = idx & (W - 1);
      const int cc = c < ncol ? c : ncol - 1;
      int64_t gi;
      if constexpr (DIR == 0) {
        const BatchSlot sl =
            near ? batch_slot_near(bt, k - G) : line_slot(nb + k, N, g.lines, G, g.inv_line);
        // slots outside every line load a ghost; no output node uses them
        const int j = sl.j < -G ? -G : (sl.j >= sl.n + G ? sl.n + G - 1 : sl.j);
        gi = sl.o + bc_index_near(j, sl.n, a.bc);
      } else {
        gi = base + bc_index(nb + k, N, a.bc) * stride + cc;
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) buf[it][v] = a.U[v * a.npts + gi];
    }
  }
  // the lane's output node in a tile of packed lines (-1: none or a ghost slot)
  int64_t onode = -1;
  if constexpr (DIR == 0) {
    if (tid < TL) {
      const BatchSlot sl =
          near ? batch_slot_near(bt, tid) : line_slot(i0 + tid, N, g.lines, G, g.inv_line);
      if (sl.j >= 0 && sl.j < sl.n) onode = sl.o + sl.j;
    }
  }
  if constexpr (spec_table(SPEC)) {
    if (tid < 64) sX[tid] = exp2_tab_entry(tid, a.ip.xsh);
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int idx = tid + it * NT;
    if (idx < SV) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sU[v * SV + idx] = buf[it][v];
      if constexpr (NV > 1) {
        const double* U = buf[it];
        const Prim<ND> q = primitives<ND>(U, a.pp.gamma);
        const double vn = q.vel[DIR];
#pragma unroll
        for (int k = 0; k < ND; ++k)
          sF[k * SV + idx] = k == DIR ? __builtin_fma(U[1 + k], vn, q.p) : U[1 + k] * vn;
        sF[ND * SV + idx] = q.ep * vn;
        sL[idx] = __builtin_fabs(vn) + sqrt_pos(a.pp.gamma * q.p * q.ir);
      }
    }
  }
  __syncthreads();

  const bool proj = (NV > 1) && a.pp.charproj;
  const double eps4 = 4.0 * a.ip.eps;
  RoeState<ND> rsq{};
  double al = 0.0;
  if constexpr (NV > 1) {
    al = sL[mid];
#pragma unroll
    for (int j = 1; j < 6; ++j) al = __builtin_fmax(al, sL[mid + j * W]);
    if (proj) {
      const double* u = sU + mid + 2 * W;
      double UA[NV], UB[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        UA[v] = u[v * SV];
        UB[v] = u[v * SV + W];
      }
      rsq = roe_average<ND>(UA, UB, a.pp.gamma);
    }
  }

  // reconstruction of field v at the lane's midpoint, f+^ + f-^ (wide: std::true_type
  // for wide_weights)
  auto recon = [&](int v, auto wide) {
    constexpr bool WIDE = decltype(wide)::value;
    double wp[5], wm[5];  // F + alpha U of nodes 0 .. 4, F - alpha U of nodes 5 .. 1
    if constexpr (NV == 1) {
      const double sp = a.pp.adv + __builtin_fabs(a.pp.adv);
      const double sm = a.pp.adv - __builtin_fabs(a.pp.adv);
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        wp[j] = sp * sU[mid + j * W];
        wm[j] = sm * sU[mid + (5 - j) * W];
      }
    } else {
      double wu[6], wf[6];
      const double* u = sU + mid;
      const double* fr = sU + (1 + DIR) * SV + mid;  // the density's flux
      const double* f = sF + mid;                    // row e - 1: component e
      if (proj) {
        if (v >= 2 && v < NV - 1) {  // shear field: X_ax - vel_ax X_rho
          const int ax = tangential_axis<ND, DIR>(v - 2);
          // (from a copy: a choice among members behind a reference is taken as one of
          // their addresses, and the Roe state then goes to scratch)
          const RoeState<ND> rz = rsq;
          double va = rz.vel[0];
#pragma unroll
          for (int k = 1; k < ND; ++k) va = (ax == k) ? rz.vel[k] : va;
#pragma unroll
          for (int j = 0; j < 6; ++j) {
            wu[j] = __builtin_fma(-va, u[j * W], u[(1 + ax) * SV + j * W]);
            wf[j] = __builtin_fma(-va, fr[j * W], f[ax * SV + j * W]);
          }
        } else {
          RoeState<ND> rs;
          // recomputed per field from vel and ic (the empty asm hides that
          // they are loop-invariant)
#pragma unroll
          for (int k = 0; k < ND; ++k) {
            rs.vel[k] = rsq.vel[k];
            asm volatile("" : "+v"(rs.vel[k]));
          }
          rs.ic = rsq.ic;
          asm volatile("" : "+v"(rs.ic));
          roe_derived<ND>(rs, a.pp.gamma);
          double l[NV];
          field_row<ND, DIR>(rs, v, l);
          project_stencil<NV, SV, W>(u, l, wu);
#pragma unroll
          for (int j = 0; j < 6; ++j) wf[j] = l[0] * fr[j * W];
#pragma unroll
          for (int e = 1; e < NV; ++e) {
            const lds_cptr fe = lds_row(f + (e - 1) * SV);
#pragma unroll
            for (int j = 0; j < 6; ++j) wf[j] = __builtin_fma(l[e], fe[j * W], wf[j]);
          }
        }
      } else {
        const double* fv = v == 0 ? fr : f + (v - 1) * SV;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          wu[j] = u[v * SV + j * W];
          wf[j] = fv[j * W];
        }
      }
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        wp[j] = __builtin_fma(al, wu[j], wf[j]);
        wm[j] = __builtin_fma(-al, wu[5 - j], wf[5 - j]);
      }
    }
    if constexpr (SPEC != SPEC_GENERIC)
      return weno5_spec<SPEC, WIDE>(a.ip, eps4, wp[0], wp[1], wp[2], wp[3], wp[4], sX) +
             weno5_spec<SPEC, WIDE>(a.ip, eps4, wm[0], wm[1], wm[2], wm[3], wm[4], sX);
    else
      return weno5(a.ip, eps4, wp[0], wp[1], wp[2], wp[3], wp[4]) +
             weno5(a.ip, eps4, wm[0], wm[1], wm[2], wm[3], wm[4]);
  };
#pragma unroll 1
  for (int v = grp; v < NV; v += GR) sW[v * TMW + mid] = recon(v, std::false_type{});

  // twice the midpoint flux, 2 F~ = R (f+^ + f-^), of the lane's own midpoint
  if constexpr (GR > 1) __syncthreads();
  if constexpr (spec_narrow(SPEC)) {
    if (grp == 0) {
      double s = sW[mid];
#pragma unroll
      for (int v = 1; v < NV; ++v) s += sW[v * TMW + mid];
      if (overflown(s)) {
#pragma unroll 1
        for (int v = 0; v < NV; ++v) sW[v * TMW + mid] = recon(v, std::true_type{});
      }
    }
  }
  if constexpr (NV > 1) {
    if (proj && grp == 0) {
      double Gv[NV], F[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Gv[v] = sW[v * TMW + mid];
      unproject<ND, DIR>(rsq, Gv, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[v * TMW + mid] = F[v];
    }
  }
  __syncthreads();

  // conservative difference
  if (tid >= TL * W) return;
  const int t = tid >> LW, c = tid & (W - 1);
  int64_t i = i0 + t;
  if constexpr (DIR == 0) {
    if (onode < 0) return;
    base = onode;
    i = 0;
  } else {
    if (i >= N || c >= ncol) return;
  }
  double res[NV], Un[NV];
  const double hih = -0.5 * a.ih;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double* fv = sW + v * TMW + tid;  // 2 F~ of midpoint t at fv[0], t + 1 at fv[W]
    res[v] = hih * (fv[W] - fv[0]);
    Un[v] = sU[v * SV + tid + 3 * W];
  }
  emit_rt<NV>(mode, a, base + i * stride + c, a.npts, res, Un, dt);
}

// --------------------------------------------------------------- launchers --
template <int NV, int DIR, int TM, int W>
static hipError_t weno_go(const SweepArgs& a, int mode, hipStream_t s) {
  using L = WenoLayout<NV, TM, W>;
  static_assert(L::lds_doubles * sizeof(double) <= 64 * 1024, "WENO tile exceeds 64 KB of LDS");
  TileGeom g{};
  g.tm = TM;
  g.w = W;
  g.lw = L::LW;
  g.ltmw = 7;
  g.tl = TM - 1;
  g.segs = (a.n[DIR] + g.tl - 1) / g.tl;
  g.xgroups = DIR == 0 ? 1 : (a.n[0] + W - 1) / W;
  // (both below 2^31 whenever the tile count is, which the launch checks)
  g.dxg = fast_div((uint32_t)g.xgroups);
  g.dseg = fast_div((uint32_t)g.segs);
  const int64_t others = DIR == 0 ? a.n[1] * a.n[2] : (DIR == 1 ? a.n[2] : a.n[1]);
  g.ntiles = g.segs * g.xgroups * others;
  if (DIR == 0) {  // packed x-lines, 3 ghost slots per side
    const int64_t len = a.n[0] + 6;
    g.lines = others;
    g.inv_line = 1.0 / (double)len;
    g.ntiles = (others * len + g.tl - 1) / g.tl;
  }
  if (g.ntiles > 0x7fffffff) return hipErrorInvalidConfiguration;
  // Two lanes per midpoint while a CU has five or six tiles at most: such a sweep is
  // the length of one tile's chain of fields.  One lane -> two, residuals: 2D 60 x 53
  // FE 17.2 -> 14.9 us, PFE 18.7 -> 14.4, 400 x 393 FE 33.9 -> 31.0, JS 24.3 -> 23.5
  // (1300 tiles); 460^2 (1700) FE 39.2 -> 38.4, JS 26.4 -> 27.3; 1000^2 FE 127 -> 134.
  const bool split = NV > 1 && g.ntiles <= 1408;
#define WCNS_W(SP)                                                                              \
  case SP:                                                                                      \
    if (split)                                                                                  \
      hipLaunchKernelGGL((weno_sweep_kernel<NV, DIR, SP, TM, W, NV == 1 ? 1 : 2>),              \
                         dim3((unsigned)g.ntiles), dim3(2 * L::TMW),                            \
                         sizeof(double) * L::lds_doubles, s, a, g, mode);                       \
    else                                                                                        \
      hipLaunchKernelGGL((weno_sweep_kernel<NV, DIR, SP, TM, W, 1>), dim3((unsigned)g.ntiles),  \
                         dim3(L::TMW), sizeof(double) * L::lds_doubles, s, a, g, mode);         \
    break;
  switch (spec_of(a.ip)) {
    WCNS_W(SPEC_FE) WCNS_W(SPEC_FE_SAT) WCNS_W(SPEC_JS) WCNS_W(SPEC_Z) WCNS_W(SPEC_PFE)
    default:
    WCNS_W(SPEC_GENERIC)
  }
#undef WCNS_W
  return hipGetLastError();
}

hipError_t launch_weno_sweep(int nv, int dir, const SweepArgs& a, int mode, hipStream_t stream) {
#define WCNS_W(NVV, DD, TMM, WW) \
  if (nv == NVV && dir == DD) return weno_go<NVV, DD, TMM, WW>(a, mode, stream);
  WCNS_W(1, 0, 128, 1) WCNS_W(1, 1, 32, 4) WCNS_W(1, 2, 32, 4)
  WCNS_W(3, 0, 128, 1)
  WCNS_W(4, 0, 128, 1) WCNS_W(4, 1, 32, 4)
  WCNS_W(5, 0, 128, 1) WCNS_W(5, 1, 32, 4) WCNS_W(5, 2, 32, 4)
#undef WCNS_W
  return hipErrorInvalidValue;
}

}  // namespace wcns
