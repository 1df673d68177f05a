// Adjoint (vector-Jacobian product) of the WCNS-FE residual on gfx950, one
// direction per launch: Ubar += s (dL/dU)^T Rbar, or, for the first direction
// of a step's stage, Ubar = ca A + cb B + cc C + s (dL/dU)^T Rbar (s = scale,
// times *dt when given; see AdjArgs).
//
// A workgroup of one wavefront per field (64 midpoints each; four wavefronts
// for the five fields of the 3D system) owns the nodes i0 .. i0+TL-1 (TL = TM
// - 5) of W adjacent lines, TM W = 64, and recomputes the TM midpoints i0-3 ..
// i0+TL+1 whose fluxes read them, so every node's cotangent is completed
// inside one tile (no atomics: the result is deterministic and independent
// of the launch shape's scheduling).  Phases, separated by barriers:
//   load     the TM+5 nodes of every column into LDS, ghosts applied;
//   roe      Roe average per midpoint (one wavefront);
//   interp   wavefront v interpolates field v at the 64 midpoints, both
//            sides, with the gradients (interp5_grad), which stay in the
//            lane's registers;
//   flux     flux cotangent from Rbar (transpose of the MND6 / MD6
//            difference), local Lax-Friedrichs VJP and back-projection VJP:
//            the left state's on one wavefront, the right state's on another
//            -> cotangents of the interpolated characteristic values and of
//            the Roe quantities;
//   interp^T wavefront v: the cotangents of field v's six stencil values
//            (gradients times the values' cotangents) and their moments with
//            the stencil nodes' states;
//   proj^T   one wavefront: the Roe-average VJP, from the moments and the two
//            sides' cotangents; the others: the projection VJP of the six
//            stencil nodes (in place in LDS), the nodes dealt in turn;
//   gather   wavefront v, component v of every node: the six midpoint
//            contributions, ghost positions folded onto the boundary node
//            (transmissive), the node-flux term of MND6, and the epilogue
//            above.
// The fifth field of the 3D system goes to two of the four wavefronts first, a
// side each, its gradients kept in LDS rows that are free until one of the two
// writes them; that and the other roles turn with the tile, so that no SIMD
// carries the same one for every tile.  (Five wavefronts per workgroup
// leave a CU two workgroups: the first SIMD takes two wavefronts of each.
// 36 % slower than four.)
// What bounds it: FP64 VALU issue and the serial length of a tile.  The SIMDs issue
// in 72-75 % of the slots of the cycles their CU is busy in the 2D kernels and 66 %
// in the 3D ones (SQ_INSTS_VALU / SQ_BUSY_CU_CYCLES; 1024^2: 59-60 % of the slots of
// 2.4 GHz, at an engine clock of 2.12-2.15 GHz).  With 256 lanes for every system and
// every per-midpoint phase on the first of four wavefronts, that wavefront issued
// about 1700 vector instructions per tile and the others 700, and the share was 55 %.
// Measured (one box, both sides in turn): residual adjoint 60 x 72 x 81 0.317
// -> 0.248 ms; 2D 1024^2, x and y sweep 0.206 and 0.198 -> 0.165 and 0.168 ms,
// two differentiable steps with their reverse 3.00 -> 2.51 ms (2.84 with the
// forward's gain alone).  Taking the nodes' MND6 terms once, on a wavefront
// the flux VJP leaves idle, instead of in every wavefront of the gather gave
// 5 % of the 2D kernels.
// LDS (doubles): sU[NV][TM+5][W] | sR[NR][64] | sWB[6 NV][64] | sM[NM][64] |
// sRB[NV][TM+5][W] | sI[TM+5][W] (64-bit integers) | the exp table | sF.  Slot s of
// task (field v, midpoint q) is sWB[(s NV + v) 64 + q]: slots 0, 1 hold the
// left and right interpolated values, then their cotangents; the
// interpolation VJP overwrites slots 0-5 with the cotangents of the six
// stencil values (each task reads its own slots first).  sM holds the two
// sides' Roe cotangents and the moments, whose rows the Roe-average VJP then
// overwrites with the cotangents of the two centre nodes.  sRB holds Rbar of
// the tile's nodes for the flux VJP, sI where the tile's own nodes lie, sF[NV][64]
// (1D and 2D systems) their MND6 terms.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wcns_adjoint_device.hpp"
#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

// Wavefronts of a workgroup (see above).
constexpr int adj_wavefronts(int nv) { return nv == 5 ? 4 : nv; }

template <int NV, int TM, int W>
struct AdjLayout {
  static constexpr int ND = NV > 1 ? NV - 2 : 1;
  // rows of sR: vel[ND], H, c, ic, and q2h, b1, b2 where a CU still holds four
  // workgroups with them (recomputed where they are read in the 3D system)
  static constexpr bool DER = NV == 3 || NV == 4;
  static constexpr int NR = NV > 1 ? NV - 2 + (DER ? 6 : 3) : 0;
  static constexpr int TN = TM + 5;
  static constexpr int TMW = TM * W;
  static constexpr int NW = adj_wavefronts(NV);
  static constexpr int NT = 64 * NW;
  static constexpr int SV = TN * W;
  static constexpr int LW = W == 1 ? 0 : W == 2 ? 1 : W == 4 ? 2 : W == 8 ? 3 : 4;
  static constexpr int NS = 6;  // LDS slots per (field, midpoint) task
  // rows of sM: the two sides' Roe cotangents (vel, H, c, q2h), then the
  // moments: NV per acoustic or entropy field, one per shear field
  static constexpr int NSB = NV > 1 ? ND + 3 : 0;
  static constexpr int NM = NV > 1 ? 2 * NSB + 3 * NV + (NV - 3) : 0;
  // rows of the tile's nodes' MND6 term, taken on a wavefront that the flux
  // VJP leaves idle (in the 3D system each wavefront of the gather takes it)
  static constexpr int NF = DER ? NV : 0;
  static constexpr size_t lds_doubles =
      (2 * (size_t)NV + 1) * SV + (size_t)(NR + NS * NV + NM + NF) * TMW + 64;
  static_assert(TMW == 64, "a tile holds one wavefront of midpoints");
  static_assert(NV == 1 || 3 * NV + (NV - 3) >= 2 * NV, "centre nodes' rows in the moments'");
  static_assert((1 << LW) == W, "W must be a power of two up to 16");
};

// Waves per SIMD the register budget is set for: four where they fit 128
// registers (the fast FE weights; LDS holds four workgroups of four
// wavefronts), three for the run-time choices, which need about 140.
constexpr int adj_waves(int spec) { return spec == SPEC_FE ? 4 : 3; }

template <int NV, int DIR, int SPEC, int TM, int W>
__global__ void __launch_bounds__(64 * adj_wavefronts(NV))
    __attribute__((amdgpu_waves_per_eu(adj_waves(SPEC))))
    adj_sweep_kernel(AdjArgs a, TileGeom g) {
  using L = AdjLayout<NV, TM, W>;
  constexpr int ND = L::ND, NR = L::NR, TMW = L::TMW, SV = L::SV, NT = L::NT;
  constexpr int LW = L::LW, NS = L::NS, NSB = L::NSB, NM = L::NM, NW = L::NW;
  constexpr bool XF = NV > NW;  // one field more than wavefronts
  constexpr int TL = TM - 5;
  extern __shared__ double smem[];
  double* sU = smem;
  double* sR = sU + NV * SV;
  double* sWB = sR + NR * TMW;
  // Interpolated values and their cotangents: left field v in row v, right in
  // row NV + v (slots 0 and 1).
  double* sW = sWB;
  double* sM = sWB + NS * NV * TMW;
  double* sMM = sM + 2 * NSB * TMW;  // the moments, then the centre nodes' cotangents
  double* sRB = sM + NM * TMW;       // Rbar of the tile's nodes
  int64_t* sI = (int64_t*)(sRB + NV * SV);
  double* sX = sRB + (NV + 1) * SV;  // exp2_tab_entry
  double* sF = sX + 64;              // the nodes' MND6 term
  const int tid = threadIdx.x;
  const int q = tid & 63;                                      // the lane's midpoint
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);     // its wavefront

  if ((int64_t)blockIdx.x >= g.ntiles) return;
  const int64_t tile = xcd_tile(blockIdx.x, g.ntiles);
  // the wavefront's role: 0 and NW - 1 take the odd field (XF), 1 and 2 the
  // flux VJP's sides, NW - 1 the Roe-average VJP
    const int role = XF ? (wv - (int)tile) & (NW - 1) : wv;

  // load: all global reads of the tile issued before the first LDS write
  constexpr int P = 5;  // ghosts on each side
  constexpr int NIT = (SV + NT - 1) / NT;
  static_assert(NIT <= 2, "a tile holds at most two nodes per lane");
  // Rbar of the same nodes (the transposed difference of the flux VJP reads
  // nodes m-2 .. m+3 of every midpoint m) goes to sRB.  sI: the index of a
  // node of the tile's own and whether it ends its line, as 4 index + (first)
  // + 2 (last), or -1.  Only the wavefronts that load map the tile to nodes.
  double buf[NIT][NV], rbuf[NIT][NV];
  int64_t info[NIT];
  if (wv * 64 < SV) {
    // Along x the lines are packed end to end with 5 ghost slots on each side
    // (TileGeom::lines, L = n[0] + 10): every position a node's cotangent
    // gathers from (nodes j-5 .. j+5) then lies in its own line's slots.
    int64_t base = 0, N, stride = 1, i0;
    int ncol = 1;
    BatchTile bt{};
    bool near = true;  // the tile spans at most two lines
    if constexpr (DIR == 0) {
      N = a.n[0];
      i0 = tile * TL;
      bt = line_tile(i0, N, g.lines, P, TL, g.inv_line);
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
    const int64_t nb = i0 - P;  // position of LDS node 0
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int idx = tid + it * NT;
      if (idx < SV) {
        const int k = idx >> LW, c = idx & (W - 1);
        const int cc = c < ncol ? c : ncol - 1;
        int64_t gi;
        bool ghost, own, first, last;
        if constexpr (DIR == 0) {
          const BatchSlot sl =
              near ? batch_slot_near(bt, k - P) : line_slot(nb + k, N, g.lines, P, g.inv_line);
          // slots before the first line or after the last load a ghost (no
          // node gathers from them)
          const int j = sl.j < -P ? -P : (sl.j >= sl.n + P ? sl.n + P - 1 : sl.j);
          gi = sl.o + bc_index_near(j, sl.n, a.bc);
          ghost = j < 0 || j >= sl.n;
          own = !ghost;
          first = j == 0;
          last = j == sl.n - 1;
        } else {
          const int64_t j = nb + k;
          gi = base + bc_index(j, N, a.bc) * stride + cc;
          ghost = j < 0 || j >= N;
          own = !ghost && c < ncol;
          first = j == 0;
          last = j == N - 1;
        }
        info[it] = own ? 4 * gi + (first ? 1 : 0) + (last ? 2 : 0) : -1;
        const bool zero = ghost && a.bc != 0;  // Rbar: zero at a transmissive ghost
#pragma unroll
        for (int v = 0; v < NV; ++v) buf[it][v] = a.U[v * a.npts + gi];
#pragma unroll
        for (int v = 0; v < NV; ++v) rbuf[it][v] = zero ? 0.0 : a.Rbar[v * a.npts + gi];
      }
    }
  }
  double xv = 0.0;
  if constexpr (SPEC == SPEC_FE) {
    if (tid < 64) xv = exp2_tab_entry(tid, a.ip.xsh);
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int idx = tid + it * NT;
    if (idx < SV) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        sU[v * SV + idx] = buf[it][v];
        sRB[v * SV + idx] = rbuf[it][v];
      }
      sI[idx] = info[it];
    }
  }
  if constexpr (SPEC == SPEC_FE) {
    if (tid < 64) sX[tid] = xv;
  }
  __syncthreads();

  const bool proj = (NV > 1) && a.pp.charproj;
  if constexpr (NV > 1) {
    if (proj) {
      if (role == 0) {
        const double* u = sU + q + 2 * W;  // nodes m, m+1 of midpoint q
        double UA[NV], UB[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          UA[v] = u[v * SV];
          UB[v] = u[v * SV + W];
        }
        const RoeState<ND> rs = roe_average<ND>(UA, UB, a.pp.gamma);
        double* rr = sR + q;
#pragma unroll
        for (int k = 0; k < ND; ++k) rr[k * TMW] = rs.vel[k];
        rr[(ND + 0) * TMW] = rs.H;
        rr[(ND + 1) * TMW] = rs.c;
        rr[(ND + 2) * TMW] = rs.ic;
        if constexpr (L::DER) {
          rr[(ND + 3) * TMW] = rs.q2h;
          rr[(ND + 4) * TMW] = rs.b1;
          rr[(ND + 5) * TMW] = rs.b2;
        }
      }
      __syncthreads();
    }
  }

  auto load_roe = [&]() {
    RoeState<ND> rs;
    const double* rr = sR + q;
#pragma unroll
    for (int k = 0; k < ND; ++k) rs.vel[k] = rr[k * TMW];
    rs.H = rr[(ND + 0) * TMW];
    rs.c = rr[(ND + 1) * TMW];
    rs.ic = rr[(ND + 2) * TMW];
    if constexpr (L::DER) {
      rs.q2h = rr[(ND + 3) * TMW];
      rs.b1 = rr[(ND + 4) * TMW];
      rs.b2 = rr[(ND + 5) * TMW];
    } else {
      roe_derived<ND>(rs, a.pp.gamma);
    }
    return rs;
  };

  // rows for the moments of field f: acoustic 0, entropy, acoustic NV-1 (NV
  // each), shear (one each)
  auto moments = [&](int f) {
    return sMM + (f >= 2 && f < NV - 1 ? 3 * NV + f - 2 : (f < 2 ? f : 2) * NV) * TMW + q;
  };

  // the odd field (an acoustic one): its left interpolation on the wavefront
  // of role 0, the right one on the last; the gradients go to its slots 2-5
  // and to the rows of its moments
  if constexpr (XF) {
    if (role == 0 || role == NW - 1) {
      const int step = role == 0 ? W : -W;
      const double* u = sU + q + (role == 0 ? 0 : 5 * W);
      double w[5], G[4];
      if (proj) {
        const RoeState<ND> rs = load_roe();
        double l[NV];
        field_row<ND, DIR>(rs, NW, l);
#pragma unroll
        for (int s = 0; s < 5; ++s) {
          double acc = l[0] * u[s * step];
#pragma unroll
          for (int e = 1; e < NV; ++e) acc = __builtin_fma(l[e], u[e * SV + s * step], acc);
          w[s] = acc;
        }
      } else {
#pragma unroll
        for (int s = 0; s < 5; ++s) w[s] = u[NW * SV + s * step];
      }
      const double y = interp5_grad_one<SPEC>(a.ip, w, G, sX);
      sW[((role == 0 ? 0 : NV) + NW) * TMW + q] = y;
      double* gr = role == 0 ? sWB + (2 * NV + NW) * TMW + q : moments(NW);
      const int gs = (role == 0 ? NV : 1) * TMW;
#pragma unroll
      for (int j = 0; j < 4; ++j) gr[j * gs] = G[j];
    }
  }

  // forward interpolation of field wv at midpoint q, both sides
  double GL[4], GR[4];
  {
    double w[6];
    const double* u = sU + q;
    if (proj) {
      if constexpr (NV > 1) {
        const double* rr = sR + q;
        if (wv >= 2 && wv < NV - 1) {  // shear field: m_ax - vel_ax rho
          const int ax = tangential_axis<ND, DIR>(wv - 2);
          const double va = rr[ax * TMW];
#pragma unroll
          for (int s = 0; s < 6; ++s) w[s] = __builtin_fma(-va, u[s * W], u[(1 + ax) * SV + s * W]);
        } else {
          const RoeState<ND> rs = load_roe();
          double l[NV];
          field_row<ND, DIR>(rs, wv, l);
#pragma unroll
          for (int s = 0; s < 6; ++s) {
            double acc = l[0] * u[s * W];
#pragma unroll
            for (int e = 1; e < NV; ++e) acc = __builtin_fma(l[e], u[e * SV + s * W], acc);
            w[s] = acc;
          }
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < 6; ++s) w[s] = u[wv * SV + s * W];
    }
    double yl, yr;
    interp5_grad<SPEC>(a.ip, w, &yl, &yr, GL, GR, sX);
    sW[wv * TMW + q] = yl;
    sW[(NV + wv) * TMW + q] = yr;
  }
  __syncthreads();

  // flux VJP of midpoint q: sW <- cotangents of the interpolated values
  auto flux_cotangent = [&](double (&Fb)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      // Rbar at node m + d (m = i0 - 3 + t, q = t W + c) is staged at LDS
      // node t + 2 + d
      const double* Rb = sRB + v * SV + q;
      const double r0 = Rb[2 * W], r1 = Rb[3 * W], rm1 = Rb[W], r2 = Rb[4 * W];
      double d;
      if (a.diff == 0) {
        d = 1.5 * (r0 - r1) + (1.0 / 30.0) * (rm1 - r2);
      } else {
        const double rm2 = Rb[0], r3 = Rb[5 * W];
        d = (75.0 / 64.0) * (r0 - r1) + (-25.0 / 384.0) * (rm1 - r2) + (3.0 / 640.0) * (rm2 - r3);
      }
      Fb[v] = -a.ih * d;
    }
  };
  // the cotangent of node idx's physical flux, and its state: F_i enters
  // D_{i+1} with -3/10 and D_{i-1} with +3/10; Rbar of nodes i - 1 .. i + 1
  // from the tile's copy (sRB: the line's ghosts applied, zero beyond a
  // transmissive end, whose ghost node carries the end node's state)
  auto node_cotangent = [&](int idx, int64_t own, double (&Fb)[NV], double (&U)[NV]) {
    const bool first = a.bc != 0 && (own & 1), last = a.bc != 0 && (own & 2);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double* Rb = sRB + v * SV + idx;
      double f = Rb[W] - Rb[-W];
      if (first) f += Rb[0];
      if (last) f -= Rb[0];
      Fb[v] = -0.3 * a.ih * f;
      U[v] = sU[v * SV + idx];
    }
  };
  if constexpr (NV == 1) {
    double Fb[1];
    flux_cotangent(Fb);
    sW[q] = 0.5 * (a.pp.adv + __builtin_fabs(a.pp.adv)) * Fb[0];
    sW[TMW + q] = 0.5 * (a.pp.adv - __builtin_fabs(a.pp.adv)) * Fb[0];
  } else {
    // one side (0 left, 1 right) on its own wavefront; both read both states,
    // so the cotangents wait for the barrier
    double Wb[NV];
    auto side = [&](auto sc) {
      constexpr int SIDE = decltype(sc)::value;
      double Fb[NV], WL[NV], WR[NV], Ub[NV];
      flux_cotangent(Fb);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        WL[v] = sW[v * TMW + q];
        WR[v] = sW[(NV + v) * TMW + q];
      }
      if (proj) {
        const RoeState<ND> rs = load_roe();
        double UL[NV], UR[NV];
        unproject<ND, DIR>(rs, WL, UL);
        unproject<ND, DIR>(rs, WR, UR);
        llf_vjp<ND, DIR, SIDE>(UL, UR, a.pp.gamma, Fb, Ub);
        RoeSideBar<ND> rb;
        unproject_vjp<ND, DIR>(rs, SIDE == 0 ? WL : WR, Ub, Wb, rb);
        double* mb = sM + SIDE * NSB * TMW + q;
#pragma unroll
        for (int k = 0; k < ND; ++k) mb[k * TMW] = rb.vel[k];
        mb[(ND + 0) * TMW] = rb.H;
        mb[(ND + 1) * TMW] = rb.c;
        mb[(ND + 2) * TMW] = rb.q2h;
      } else {
        llf_vjp<ND, DIR, SIDE>(WL, WR, a.pp.gamma, Fb, Ub);
#pragma unroll
        for (int v = 0; v < NV; ++v) Wb[v] = Ub[v];
      }
    };
    if constexpr (L::NF > 0) {
      if (role == 0 && a.diff == 0 && q < TL * W) {
        double Fb[NV], U[NV], Ub[NV];
        node_cotangent(q + 5 * W, sI[q + 5 * W], Fb, U);
#pragma unroll
        for (int v = 0; v < NV; ++v) Ub[v] = 0.0;
        flux_speed_vjp<ND, DIR>(U, primitives<ND>(U, a.pp.gamma), a.pp.gamma, 0.0, Fb, 0.0, Ub);
#pragma unroll
        for (int v = 0; v < NV; ++v) sF[v * TMW + q] = Ub[v];
      }
    }
    if (role == 1)
      side(std::integral_constant<int, 0>{});
    else if (role == 2)
      side(std::integral_constant<int, 1>{});
    __syncthreads();
    if (role == 1 || role == 2) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[((role - 1) * NV + v) * TMW + q] = Wb[v];
    }
  }
  __syncthreads();

  // interpolation VJP of field f: slot j <- cotangent of stencil value j of
  // the field, from the task's own slots (the other wavefronts write the
  // other fields' rows), and its moments with the stencil nodes' states
  auto stencil_vjp = [&](int f, const double (&gl)[4], const double (&gr)[4]) {
    double wb[6];
    interp5_vjp(sW[f * TMW + q], sW[(NV + f) * TMW + q], gl, gr, wb);
#pragma unroll
    for (int j = 0; j < 6; ++j) sWB[(j * NV + f) * TMW + q] = wb[j];
    if constexpr (NV > 1) {
      if (proj) {
        const double* u = sU + q;
        double* mm = moments(f);
#pragma unroll
        for (int e = 0; e < NV; ++e) {
          if (e > 0 && f >= 2 && f < NV - 1) break;  // (a shear field: rho only)
          double t = wb[0] * u[e * SV];
#pragma unroll
          for (int j = 1; j < 6; ++j) t = __builtin_fma(wb[j], u[e * SV + j * W], t);
          mm[e * TMW] = t;
        }
      }
    }
  };
  stencil_vjp(wv, GL, GR);
  if constexpr (XF) {
    if (role == 0) {
      const double* mm = moments(NW);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        GL[j] = sWB[((2 + j) * NV + NW) * TMW + q];
        GR[j] = mm[j * TMW];
      }
      stencil_vjp(NW, GL, GR);
    }
  }
  __syncthreads();

  // Roe-average VJP on one wavefront, the projection VJP of the six
  // stencil nodes on the others (in place: slot j's NV rows)
  if constexpr (NV > 1) {
    if (proj) {
      const RoeState<ND> rs = load_roe();
      if (role == NW - 1) {
        const double *ml = sM + q, *mr = sM + NSB * TMW + q;
        RoeBar<ND> rb;
#pragma unroll
        for (int k = 0; k < ND; ++k) rb.vel[k] = ml[k * TMW] + mr[k * TMW];
        rb.H = ml[(ND + 0) * TMW] + mr[(ND + 0) * TMW];
        rb.c = ml[(ND + 1) * TMW] + mr[(ND + 1) * TMW];
        rb.q2h = ml[(ND + 2) * TMW] + mr[(ND + 2) * TMW];
        rb.ic = rb.b1 = rb.b2 = 0.0;
        double* mm = sMM + q;
        double T[NV], S[ND];
#pragma unroll
        for (int e = 0; e < NV; ++e)
          T[e] = 0.5 * (mm[e * TMW] + mm[(2 * NV + e) * TMW]) - mm[(NV + e) * TMW];
        const double A0 = 0.5 * (mm[0] - mm[2 * NV * TMW]);
        const double An = 0.5 * (mm[(1 + DIR) * TMW] - mm[(2 * NV + 1 + DIR) * TMW]);
#pragma unroll
        for (int k = 0; k < ND - 1; ++k) S[k] = mm[(3 * NV + k) * TMW];
        project_roe_bar<ND, DIR>(rs, T, A0, An, S, rb);
        const double* u = sU + q;
        double UA[NV], UB[NV], UbA[NV], UbB[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          UA[v] = u[v * SV + 2 * W];
          UB[v] = u[v * SV + 3 * W];
        }
        roe_vjp<ND>(UA, UB, a.pp.gamma, rs, rb, UbA, UbB);
        // (the moments of midpoint q have been read by this lane alone)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          mm[v * TMW] = UbA[v];
          mm[(NV + v) * TMW] = UbB[v];
        }
      } else {
#pragma unroll 1
        for (int j = role; j < 6; j += NW - 1) {
          double Wb[NV], Ub[NV];
          double* sl = sWB + j * NV * TMW + q;
#pragma unroll
          for (int v = 0; v < NV; ++v) Wb[v] = sl[v * TMW];
          project_vjp<ND, DIR>(rs, Wb, Ub);
#pragma unroll
          for (int v = 0; v < NV; ++v) sl[v * TMW] = Ub[v];
        }
      }
      __syncthreads();
    }
  }

  // gather component f of the tile's own nodes: component wv, and the odd one
  // on the wavefront that did the Roe-average VJP
#pragma unroll 1
  for (int f = wv; f < NV; f += (XF && role == NW - 1 && f < NW) ? NW - wv : NV) {
    if (q >= TL * W) break;
    const int t = q >> LW, c = q & (W - 1);
    const int k = t + 5;  // LDS node index of node i0 + t
    const int64_t own = sI[q + 5 * W];
    if (own >= 0) {
      const int64_t e = f * a.npts + (own >> 2);
      // the epilogue's inputs, read while the contributions are summed
      double y;
      if (a.A) {
        y = a.ca * a.A[e];
        if (a.B) y = __builtin_fma(a.cb, a.B[e], y);
        if (a.C) y = __builtin_fma(a.cc, a.C[e], y);
      } else {
        y = a.Ubar[e];
      }
      double acc = 0.0;
      // contributions at LDS position kk: midpoints kk - j, j = 0..5, inside the tile
      auto add_position = [&](int kk) {
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          const int tm = kk - j;
          if (tm >= 0 && tm < TM) {
            acc += sWB[(j * NV + f) * TMW + tm * W + c];
            if constexpr (NV > 1) {
              if ((j == 2 || j == 3) && proj)
                acc += sMM[((j == 2 ? 0 : NV) + f) * TMW + tm * W + c];
            }
          }
        }
      };
      add_position(k);
      const int G = a.diff ? 5 : 4;
      const bool first = a.bc != 0 && (own & 1), last = a.bc != 0 && (own & 2);
      if (first)
        for (int gg = 1; gg <= G; ++gg) add_position(k - gg);
      if (last)
        for (int gg = 1; gg <= G; ++gg) add_position(k + gg);
      if (a.diff == 0) {
        if constexpr (L::NF > 0) {
          acc += sF[f * TMW + q];
        } else {
          double Fb[NV], U[NV];
          node_cotangent(q + 5 * W, own, Fb, U);
          acc += node_flux_vjp<NV, DIR>(a.pp, U, Fb, f);
        }
      }
      const double sc = a.dt ? a.scale * *a.dt : a.scale;
      a.Ubar[e] = __builtin_fma(sc, acc, y);
    }
  }
}

// --------------------------------------------------------------- launchers --
static inline int64_t ceil_div64(int64_t x, int64_t y) { return (x + y - 1) / y; }

// One wavefront of midpoints per tile.  y and z tiles are two columns wide: a
// taller tile recomputes fewer overlap rows (5 of 32 instead of 5 of 16 with
// four columns), and the XCD-aware order keeps the column pairs that share a
// cache line on one L2.
template <int DIR>
struct AdjShape {
  static constexpr int W = DIR == 0 ? 1 : 2;
  static constexpr int TM = 64 / W;
};

template <int NV, int DIR>
static hipError_t adj_go(const AdjArgs& a, hipStream_t s) {
  constexpr int TM = AdjShape<DIR>::TM, W = AdjShape<DIR>::W;
  using L = AdjLayout<NV, TM, W>;
  static_assert(L::lds_doubles * sizeof(double) <= 64 * 1024, "adjoint tile exceeds 64 KB of LDS");
  TileGeom g{};
  g.tm = TM;
  g.w = W;
  g.lw = L::LW;
  g.ltmw = 6;
  g.tl = TM - 5;
  g.segs = ceil_div64(a.n[DIR], g.tl);
  g.xgroups = DIR == 0 ? 1 : ceil_div64(a.n[0], W);
  // (both below 2^31 whenever the tile count is, which the launch checks)
  g.dxg = fast_div((uint32_t)g.xgroups);
  g.dseg = fast_div((uint32_t)g.segs);
  const int64_t others = DIR == 0 ? a.n[1] * a.n[2] : (DIR == 1 ? a.n[2] : a.n[1]);
  g.ntiles = g.segs * g.xgroups * others;
  g.lines = 0;
  g.inv_line = 0.0;
  if (DIR == 0) {  // packed x-lines, 5 ghost slots per side
    const int64_t L = a.n[0] + 10;
    g.lines = others;
    g.inv_line = 1.0 / (double)L;
    g.ntiles = ceil_div64(others * L, g.tl);
  }
  if (g.ntiles > 0x7fffffff) return hipErrorInvalidConfiguration;
  const size_t lds = sizeof(double) * L::lds_doubles;
  if (spec_of(a.ip) == SPEC_FE)
    hipLaunchKernelGGL((adj_sweep_kernel<NV, DIR, SPEC_FE, TM, W>), dim3((unsigned)g.ntiles),
                       dim3(L::NT), lds, s, a, g);
  else
    hipLaunchKernelGGL((adj_sweep_kernel<NV, DIR, SPEC_GENERIC, TM, W>), dim3((unsigned)g.ntiles),
                       dim3(L::NT), lds, s, a, g);
  return hipGetLastError();
}

hipError_t launch_adjoint_dir(int nv, int dir, const AdjArgs& a, hipStream_t stream) {
#define WCNS_A(NVV, DD) \
  if (nv == NVV && dir == DD) return adj_go<NVV, DD>(a, stream);
  WCNS_A(1, 0) WCNS_A(1, 1) WCNS_A(1, 2)
  WCNS_A(3, 0)
  WCNS_A(4, 0) WCNS_A(4, 1)
  WCNS_A(5, 0) WCNS_A(5, 1) WCNS_A(5, 2)
#undef WCNS_A
  return hipErrorInvalidValue;
}

}  // namespace wcns
