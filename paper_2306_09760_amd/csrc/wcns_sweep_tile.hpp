// Directional sweep of the WCNS-FE residual on gfx950 (all directions and
// the ragged batch).
//
// A workgroup of 256 lanes owns one tile: TM midpoints along the sweep
// direction by W adjacent x-columns (W = 1 for the x direction; for y and z
// the columns make the global loads coalesced rows).  TM*W is 128 or 256 and
// both are compile-time, so every LDS address is a lane base plus an
// immediate offset.  Phases, with every lane looping over the phase's tasks
// (no wavefront idles through a short phase):
//   load    the TM+5 nodes of every column into LDS, ghosts applied (all
//           global reads issued before the first LDS write);
//   roe     Roe average of the two nodes around each midpoint;
//   interp  one task = one field of one midpoint: its six stencil values
//           projected on the fly from the LDS nodes, then the left-biased
//           and the mirrored right-biased nonlinear interpolation
//           (interp5_pair).  TM*W is a multiple of 64, so the field is
//           uniform across a wavefront;
//   flux    back-projection of the two interpolated states and (twice) the
//           local Lax-Friedrichs flux;
//   diff    MND6 or MD6 flux difference of TL = TM-3 (TM-5) nodes per
//           column, written as R, R+= or the fused SSP-RK3 stage combine.
// The ragged batch packs its tiles across problem ends (BatchArgs): a tile's
// slots may belong to two or more problems, each slot mapped to its problem,
// node or ghost in the load phase.
// Barriers separate load | roe | interp | flux | diff; with TM*W = 256 every
// lane owns one midpoint column through roe, interp and flux, and only
// load | roe and flux | diff are synchronised.
// LDS (doubles): sU[NV][TM+5][W] | sR[NR][TM*W] | sW[2 NV][TM*W] | the
// 64-entry exp table; the flux overwrites sW rows 0..NV-1 (each task reads
// its midpoint's two states before writing that midpoint's flux), and with
// MND6 rows NV..2NV-1 with the physical flux of node m + 2.  On the
// register path (sweep_reg: 4 and 5 variables, TM*W = 256) each lane keeps
// its midpoint's Roe state in registers and sR is left out.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "wcns_internal.hpp"
#include "wcns_plain_device.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

#ifndef WCNS_REG_MIN_NV  // fewest variables of a register-path tile
#define WCNS_REG_MIN_NV 4
#endif

// With TM W = 256 every lane owns one midpoint column through the Roe,
// interpolation and flux phases.  From WCNS_REG_MIN_NV variables on, that
// lane keeps its Roe state in registers instead of LDS: the 5-variable tile
// then needs 31 KB of LDS instead of 43 KB (five workgroups per CU instead of
// three), the 4-variable one 25 KB instead of 35 KB.
constexpr bool sweep_reg(int nv, int tmw) { return tmw == 256 && nv > 1 && nv >= WCNS_REG_MIN_NV; }

// The 5-variable y and z tiles of four and eight columns keep the last field's
// two states in registers between the interpolation and the flux, and the node
// fluxes of their last two variables in the tile's own nodes, which nobody reads
// by then (one more barrier): two rows of sW less let a CU's LDS hold five of
// them instead of four (a 32 x 8 tile 28.7 instead of 32.8 KB; the 64 x 4 one of
// 32.0 KB, too, took the room of four).  Residual 256^3, Z 2.300 -> 2.219 ms, FE
// 3.135 -> 3.105; 200 x 190 x 180, FE 1.375 -> 1.350.
constexpr bool sweep_trim(int nv, int tm, int w) {
  return nv == 5 && sweep_reg(nv, tm * w) && w >= 4;
}

// LDS doubles of a tile: nodes sU[NV][TM+5][W] | Roe states sR[NR][TM W]
// (none on the register path) | interpolated states sW[2 NV][TM W] | the
// 64-entry exp table.
constexpr size_t sweep_lds_doubles(int nv, int tm, int w) {
  const size_t nr = (nv > 1 && !sweep_reg(nv, tm * w)) ? (size_t)nv + 1 : 0;
  const size_t rows = nr + 2 * (size_t)nv - (sweep_trim(nv, tm, w) ? 2 : 0);
  return (size_t)nv * (tm + 5) * w + rows * ((size_t)tm * w) + 64;
}

template <int NV, int TM, int W>
struct SweepLayout {
  static constexpr int ND = NV > 1 ? NV - 2 : 1;
  static constexpr bool REG = sweep_reg(NV, TM * W);
  static constexpr bool TRIM = sweep_trim(NV, TM, W);
  static constexpr int NS = 2 * NV - (TRIM ? 2 : 0);   // rows of sW
  static constexpr int NR = (NV > 1 && !REG) ? NV - 2 + 3 : 0;  // vel[ND], H, c, ic
  static constexpr int TN = TM + 5;                    // nodes per column
  static constexpr int TMW = TM * W;                   // midpoints per tile
  static constexpr int SV = TN * W;                    // LDS stride between variables
  static constexpr int LW = W == 1 ? 0 : W == 2 ? 1 : W == 4 ? 2 : W == 8 ? 3 : 4;
  static constexpr int LTMW = TMW == 128 ? 7 : 8;
  static constexpr size_t lds_doubles = sweep_lds_doubles(NV, TM, W);
  static_assert(lds_doubles == (size_t)NV * SV + (size_t)(NR + NS) * TMW + 64, "LDS layout");
  static_assert(TMW == 128 || TMW == 256, "tile must hold 128 or 256 midpoints");
  static_assert((1 << LW) == W, "W must be a power of two up to 16");
};

// The sweep kernel's arguments, one struct so that its layout in the kernel
// argument segment is the struct's.
struct SweepKernArgs {
  SweepArgs a;
  BatchArgs b;
  TileGeom g;
  int mode;
};
using SweepKernArgsPtr = const __attribute__((address_space(4))) SweepKernArgs*;

// The kernel's arguments for a late phase.  Values held in scalar registers
// from the kernel's start through the interpolation spill to VGPR lanes
// (every reload a VALU instruction per lane) once the FE constants fill the
// scalar file; the empty asm hides that the segment does not change, so the
// late phase reads what it needs with scalar loads at that point instead.
__device__ __forceinline__ SweepKernArgsPtr sweep_kernargs_late() {
  unsigned long long p = reinterpret_cast<unsigned long long>(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("" : "+s"(p));
  return reinterpret_cast<SweepKernArgsPtr>(p);
}

// What a tile of a one-launch stage (wcns_stage.hip) reads and writes instead
// of SweepArgs' state, residual and output.  The state under stage st + 1 is
// combined in the load phase from what stage st left: U^n, U1 and the
// directional residuals of the last stage (direction d at R + d rstride).
struct StageIn {
  int st;                // 1, 2, 3
  const double* U0;      // U^n
  double* U1;            // U1, written by stage 2's x tiles (own nodes), read by stage 3
  const double* R;       // directional residuals of the previous stage (st > 1)
  double* Rout;          // of this stage
  int64_t rstride;
  const double* dt;      // step size, or null: cfl / max partial, left in *dt_out
  double* dt_out;
  double* partial;       // maxima (bit patterns) of the wave rate per x tile, by stage 1
  int32_t npartial;
  int32_t* status;
  double cfl;
  double ih[3];
};

// The kernel's arguments: stage_kernel reads them through a pointer to its
// argument segment (as sweep_kernargs_late, for the same reason).
template <int ND>
struct StageKernArgs {
  StageIn in;
  SweepArgs a[ND];
  TileGeom g[ND];
  int nb[ND];  // workgroups of each direction's tiles: a multiple of the 8 XCDs
};
template <int ND>
using StageKernArgsPtr = const __attribute__((address_space(4))) StageKernArgs<ND>*;
template <int ND>
__device__ __forceinline__ StageKernArgsPtr<ND> stage_kernargs() {
  unsigned long long p = reinterpret_cast<unsigned long long>(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("" : "+s"(p));
  return reinterpret_cast<StageKernArgsPtr<ND>>(p);
}
template <class T>
__device__ __forceinline__ StageIn stage_in(const T& k) {
  StageIn in;
  in.st = k.st;
  in.U0 = k.U0;
  in.U1 = k.U1;
  in.R = k.R;
  in.Rout = k.Rout;
  in.rstride = k.rstride;
  in.dt = k.dt;
  in.dt_out = k.dt_out;
  in.partial = k.partial;
  in.npartial = k.npartial;
  in.status = k.status;
  in.cfl = k.cfl;
#pragma unroll
  for (int d = 0; d < 3; ++d) in.ih[d] = k.ih[d];
  return in;
}

// *(p + off bytes): a uniform base and a 32-bit lane offset, which the memory
// instructions add themselves (a one-launch stage's arrays are small).
template <class T>
__device__ __forceinline__ T& at_bytes(T* p, uint32_t off) {
  using C = std::conditional_t<std::is_const_v<T>, const char, char>;
  return *reinterpret_cast<T*>(reinterpret_cast<C*>(p) + off);
}

// One tile (logical index `tile`) of a sweep; every lane of the workgroup
// calls it from sweep_kernel (its late phases re-read the kernel arguments).
// STEP: a tile of a one-launch stage, with its state from StageIn and its
// direction's residual to Rout (mode unused).
template <int NV, int DIR, bool BATCH, int SPEC, int TM, int W, bool STEP = false>
__device__ __forceinline__ void sweep_tile(const SweepArgs& a, const BatchArgs& b,
                                           const TileGeom& g, int mode, int64_t tile,
                                           double* smem) {
  static_assert(!(STEP && BATCH), "a one-launch stage is of one problem");
  constexpr bool PLAIN = spec_plain(SPEC);
  using L = SweepLayout<NV, TM, W>;
  constexpr int ND = L::ND, NR = L::NR, TN = L::TN, TMW = L::TMW, SV = L::SV;
  constexpr int LW = L::LW, LTMW = L::LTMW;
  constexpr bool REG = L::REG;
  constexpr int NT = 256;
  double* sU = smem;
  double* sR = sU + NV * SV;
  double* sW = sR + NR * TMW;
  double* sX = sW + L::NS * TMW;  // exp2_tab_entry
  constexpr bool TRIM = L::TRIM;
  constexpr int RO = TRIM ? NV - 1 : NV;  // the right states' first row of sW
  const int tid = threadIdx.x;
  const int G = a.diff ? 5 : 4;
  const int TL = TM - (a.diff ? 5 : 3);

  int64_t base = 0, N = 0, stride = 1, i0;
  int ncol = 1;
  double ih = a.ih, dt = 0.0;
  // Along x (and in the batch) the lines are packed end to end: i0 is a slot
  // of the packed index space (BatchArgs, TileGeom::lines).
  constexpr bool LINES = BATCH || DIR == 0;
  BatchTile bt{};
  bool near = true;  // the tile spans at most two lines or problems
  if constexpr (BATCH) {
    i0 = tile * TL;
    bt = batch_tile(b, tile, i0, G);
    near = bt.p1 <= bt.p0 + 1;
    if (mode == MODE_STAGE) {
      bool live = false;  // uniform across the block
      for (int p = bt.p0; p <= bt.p1; ++p) live |= (b.dtp[p] != 0.0);
      if (!live) return;  // every problem of the tile has finished
    }
  } else if constexpr (DIR == 0) {
    i0 = tile * TL;
    N = a.n[0];
    bt = line_tile(i0, N, g.lines, G, TL, g.inv_line);
    near = bt.p1 <= bt.p0 + 1;
    if (!STEP && mode >= MODE_STAGE) dt = *a.dt;
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
    if (!STEP && mode >= MODE_STAGE) dt = *a.dt;
  }
  const int64_t nb = i0 - G;

  // load: every global read of the tile (at most two nodes per lane, and the
  // exp table) is issued before the first LDS write, so their latencies
  // overlap
  constexpr int NIT = (SV + NT - 1) / NT;
  static_assert(NIT <= 2, "a tile holds at most two nodes per lane");
  double buf[NIT][NV];
  static_assert(!STEP || NIT == 1, "one node per lane");
  StageIn in{};
  if constexpr (STEP) in = stage_in(stage_kernargs<ND>()->in);
  double b1[STEP ? NV : 1], br[STEP ? NV : 1][STEP ? ND : 1];  // U1 and R of the lane's node
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int idx = tid + it * NT;
    if (idx < SV) {
      const int k = idx >> LW, c = idx & (W - 1);
      const int cc = c < ncol ? c : ncol - 1;
      int64_t gi;
      if constexpr (LINES) {
        BatchSlot sl;
        if (near)
          sl = batch_slot_near(bt, k - G);
        else if constexpr (BATCH)
          sl = batch_slot(b, bt.p0, bt.p1, G, nb + k);
        else
          sl = line_slot(nb + k, N, g.lines, G, g.inv_line);
        // slots outside every problem's range (before the first, after the
        // last) load a ghost; no output node uses them
        const int j = sl.j < -G ? -G : (sl.j >= sl.n + G ? sl.n + G - 1 : sl.j);
        gi = sl.o + bc_index_near(j, sl.n, a.bc);
      } else {
        gi = base + bc_index(nb + k, N, a.bc) * stride + cc;
      }
      if constexpr (STEP) {
        const uint32_t off = (uint32_t)gi * 8;
#pragma unroll
        for (int v = 0; v < NV; ++v) buf[it][v] = at_bytes(in.U0 + v * a.npts, off);
        if (in.st == 3) {
#pragma unroll
          for (int v = 0; v < NV; ++v) b1[v] = at_bytes(in.U1 + v * a.npts, off);
        }
        if (in.st > 1) {
#pragma unroll
          for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int d = 0; d < ND; ++d)
              br[v][d] = at_bytes(in.R + d * in.rstride + v * a.npts, off);
        }
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) buf[it][v] = a.U[v * a.npts + gi];
      }
    }
  }
  // the lane's output node in a tile of packed lines (-1: none, or a ghost
  // slot)
  int64_t onode = -1;
  int oprob = 0;
  if constexpr (LINES) {
    static_assert(W == 1 && TM <= NT, "one output node per lane");
    if (tid < TL) {
      BatchSlot sl;
      if (near)
        sl = batch_slot_near(bt, tid);
      else if constexpr (BATCH)
        sl = batch_slot(b, bt.p0, bt.p1, G, i0 + tid);
      else
        sl = line_slot(i0 + tid, N, g.lines, G, g.inv_line);
      if (sl.j >= 0 && sl.j < sl.n) {
        onode = sl.o + sl.j;
        oprob = sl.p;
      }
    }
  }
  double xv = 0.0;
  if constexpr (spec_table(SPEC)) {
    if (tid < 64) xv = exp2_tab_entry(tid, a.ip.xsh);
  } else if constexpr (SPEC == SPEC_PLAIN_FE) {
    if (tid < 64) xv = kExp2Tab64[tid];
  }
  if constexpr (STEP) {
    if (in.st > 1) {
      if (in.dt) {
        dt = *in.dt;
      } else {
        // every tile of stage 2 takes the maximum itself
        unsigned long long m = 0;
        const unsigned long long* part = reinterpret_cast<const unsigned long long*>(in.partial);
        for (int i = tid; i < in.npartial; i += NT) m = umax64(m, part[i]);
        m = wave_max_bits(m);
        unsigned long long* sM = reinterpret_cast<unsigned long long*>(sW);
        if ((tid & 63) == 0) sM[tid >> 6] = m;
        __syncthreads();  // (sW is written again only after the next barrier)
        m = umax64(umax64(sM[0], sM[1]), umax64(sM[2], sM[3]));
        dt = in.cfl / __builtin_bit_cast(double, m);
        if (DIR == 0 && tile == 0 && tid == 0) *in.dt_out = dt;
      }
      if (tid < SV) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
          for (int d = 1; d < ND; ++d) br[v][0] += br[v][d];
        }
        if (in.st == 3) {
#pragma unroll
          for (int v = 0; v < NV; ++v)
            buf[0][v] = stage_value(0.75, 0.25, buf[0][v], b1[v], dt, br[v][0]);
        } else {  // (ca = 0: its term adds +0)
#pragma unroll
          for (int v = 0; v < NV; ++v)
            buf[0][v] = stage_value(0.0, 1.0, 0.0, buf[0][v], dt, br[v][0]);
        }
      }
    }
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int idx = tid + it * NT;
    if (idx < SV) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sU[v * SV + idx] = buf[it][v];
    }
  }
  if constexpr (spec_table(SPEC) || SPEC == SPEC_PLAIN_FE) {
    if (tid < 64) sX[tid] = xv;
  }
  __syncthreads();

  // the functions below in the specialisation's arithmetic
  auto roe = [&](const double* UA, const double* UB) {
    if constexpr (PLAIN) return plain::roe_average<ND>(UA, UB, a.pp.gamma);
    else return roe_average<ND>(UA, UB, a.pp.gamma);
  };
  auto interp = [&](const double (&w)[6], double* l, double* r) {
    if constexpr (PLAIN) plain::interp5_pair<SPEC == SPEC_PLAIN_FE>(a.ip, w, l, r, sX);
    else interp5_pair<SPEC>(a.ip, w, l, r, sX);
  };
  // With one midpoint column per lane (TM W = 256), lane q computes the Roe
  // state, all interpolations and the flux of midpoint column q itself, so
  // the Roe, interpolation and flux phases need no barrier between them.
  constexpr bool OWN = (TMW == NT);
  const bool proj = (NV > 1) && a.pp.charproj;
  RoeState<ND> rsq{};  // the register path: Roe state of the lane's midpoint column
  if constexpr (REG) {
    if (proj) {
      const double* u = sU + tid + 2 * W;
      double UA[NV], UB[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        UA[v] = u[v * SV];
        UB[v] = u[v * SV + W];
      }
      rsq = roe(UA, UB);
    }
  } else if constexpr (NV > 1) {
    if (proj) {
#pragma unroll 1
      for (int q = tid; q < TMW; q += NT) {
        // node m+2 of column c sits at LDS index q + 2W (q = m W + c)
        const double* u = sU + q + 2 * W;
        double UA[NV], UB[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          UA[v] = u[v * SV];
          UB[v] = u[v * SV + W];
        }
        const RoeState<ND> rs = roe(UA, UB);
        double* r = sR + q;
#pragma unroll
        for (int k = 0; k < ND; ++k) r[k * TMW] = rs.vel[k];
        r[(ND + 0) * TMW] = rs.H;
        r[(ND + 1) * TMW] = rs.c;
        r[(ND + 2) * TMW] = rs.ic;
      }
      if constexpr (!OWN) __syncthreads();
    }
  }

  // the six values of field v around midpoint rem = m W + c
  auto stencil = [&](int v, int rem, double (&w)[6]) {
    const double* u = sU + rem;  // node m of column c; node m + j at u[j W]
    if (proj) {
      if constexpr (NV > 1) {
        const double* r = sR + rem;
        if (v >= 2 && v < NV - 1) {  // shear field: m_ax - vel_ax rho
          const int ax = tangential_axis<ND, DIR>(v - 2);
          double va;
          if constexpr (REG) {
            // (from a copy: a choice among members behind a reference is taken as one of
            // their addresses, and the Roe state then goes to scratch)
            const RoeState<ND> rz = rsq;
            va = rz.vel[0];
#pragma unroll
            for (int k = 1; k < ND; ++k) va = (ax == k) ? rz.vel[k] : va;
          } else {
            va = r[ax * TMW];
          }
          const double* um = u + (1 + ax) * SV;
#pragma unroll
          for (int j = 0; j < 6; ++j) w[j] = __builtin_fma(-va, u[j * W], um[j * W]);
        } else {
          RoeState<ND> rs;
          if constexpr (REG) {
            // recomputed per field from vel and ic, which are all the loop
            // keeps of the Roe state besides H and c (the empty asm hides
            // that they are loop-invariant)
#pragma unroll
            for (int k = 0; k < ND; ++k) {
              rs.vel[k] = rsq.vel[k];
              asm volatile("" : "+v"(rs.vel[k]));
            }
            rs.ic = rsq.ic;
            asm volatile("" : "+v"(rs.ic));
          } else {
#pragma unroll
            for (int k = 0; k < ND; ++k) rs.vel[k] = r[k * TMW];
            rs.ic = r[(ND + 2) * TMW];
          }
          roe_derived<ND>(rs, a.pp.gamma);
          double l[NV];
          if constexpr (PLAIN) plain::field_row<ND, DIR>(rs, v, l);
          else field_row<ND, DIR>(rs, v, l);
          project_stencil<NV, SV, W>(u, l, w);
        }
      }
    } else {
      const double* uv = u + v * SV;
#pragma unroll
      for (int j = 0; j < 6; ++j) w[j] = uv[j * W];
    }
  };

  double wl = 0.0, wr = 0.0;  // TRIM: the last field's states
  // one field of one midpoint per task: its left- and right-biased
  // interpolations share the six projected stencil values
#pragma unroll 1
  for (int q = tid; q < NV * TMW; q += NT) {
    const int v = q >> LTMW;
    double w[6];
    stencil(v, q & (TMW - 1), w);
    if constexpr (TRIM) {
      interp(w, &wl, &wr);
      if (v < NV - 1) {
        sW[q] = wl;
        sW[RO * TMW + q] = wr;
      }
    } else {
      interp(w, sW + q, sW + NV * TMW + q);
    }
  }
  if constexpr (!OWN) __syncthreads();

  // A batch tile has at most one output node per lane (TL < 256): the lane
  // locates it during the load phase and reads its problem's 1/h and dt
  // here, so that these reads overlap the flux phase rather than the
  // epilogue.
  double oih = 0.0, odt = 0.0;
  if constexpr (BATCH) {
    if (onode >= 0) {
      const SweepKernArgsPtr k = sweep_kernargs_late();
      oih = k->b.ih[oprob];
      if (mode == MODE_STAGE) odt = k->b.dtp[oprob];
    }
  }

  // TRIM: the lane's output node's last two variables, and the node fluxes of
  // those on their way into sU
  double Ut[2] = {}, Ft[2] = {};
  if constexpr (TRIM) {
    if (tid < TL * W) {
#pragma unroll
      for (int t = 0; t < 2; ++t) Ut[t] = sU[(NV - 2 + t) * SV + tid + G * W];
    }
  }
  // midpoint flux (overwrites sW rows 0..NV-1 of the same midpoint)
#pragma unroll 1
  for (int q = tid; q < TMW; q += NT) {
    double F[NV];
#pragma unroll
    for (int pass = 0; pass < (spec_narrow(SPEC) ? 2 : 1); ++pass) {
      if constexpr (NV == 1) {
        // (twice the upwind flux, as llf_flux2)
        const double uL = sW[q], uR = sW[TMW + q];
        if constexpr (PLAIN)
          F[0] = plain::advection_flux(a.pp.adv, uL, uR);
        else
          F[0] = __builtin_fma(a.pp.adv, uL + uR, -__builtin_fabs(a.pp.adv) * (uR - uL));
      } else {
        double WL[NV], WR[NV], UL[NV], UR[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          WL[v] = TRIM && v == NV - 1 ? wl : sW[v * TMW + q];
          WR[v] = TRIM && v == NV - 1 ? wr : sW[(RO + v) * TMW + q];
        }
        if (proj) {
          RoeState<ND> rs = rsq;
          if constexpr (!REG) {
            const double* r = sR + q;
#pragma unroll
            for (int k = 0; k < ND; ++k) rs.vel[k] = r[k * TMW];
            rs.H = r[(ND + 0) * TMW];
            rs.c = r[(ND + 1) * TMW];
            rs.ic = r[(ND + 2) * TMW];
            roe_derived<ND>(rs, a.pp.gamma);
          }
          if constexpr (PLAIN) {
            plain::unproject<ND, DIR>(rs, WL, UL);
            plain::unproject<ND, DIR>(rs, WR, UR);
          } else {
            unproject<ND, DIR>(rs, WL, UL);
            unproject<ND, DIR>(rs, WR, UR);
          }
        } else {
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            UL[v] = WL[v];
            UR[v] = WR[v];
          }
        }
        if constexpr (PLAIN) plain::llf_flux<ND, DIR>(UL, UR, a.pp.gamma, F);
        else llf_flux2<ND, DIR>(UL, UR, a.pp.gamma, F);
      }
      // (the last component depends on every field)
      if (!spec_narrow(SPEC) || pass > 0 || !overflown(F[NV - 1])) break;
      if constexpr (spec_narrow(SPEC)) {
#pragma unroll 1
        for (int v = 0; v < NV; ++v) {
          double w[6], l, r;
          stencil(v, q, w);
          interp5_pair<SPEC, true>(a.ip, w, &l, &r, sX);
          if (TRIM && v == NV - 1) {
            wl = l;
            wr = r;
          } else {
            sW[v * TMW + q] = l;
            sW[(RO + v) * TMW + q] = r;
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) sW[v * TMW + q] = F[v];
    if (a.diff == 0) {
      // the physical flux of node m + 2 (q = m W + c) for the MND6
      // difference, into the right-state rows this lane has just read: each
      // node's flux is computed once instead of by both its neighbours
      double Uc[NV], Fc[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Uc[v] = sU[v * SV + q + 2 * W];
      if constexpr (PLAIN) plain::node_flux<NV, DIR>(a.pp, Uc, Fc);
      else node_flux<NV, DIR>(a.pp, Uc, Fc);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        if (TRIM && v >= NV - 2)
          Ft[v - (NV - 2)] = Fc[v];
        else
          sW[(NV + v) * TMW + q] = Fc[v];
      }
    }
  }
  if constexpr (TRIM) {
    if (a.diff == 0) {
      __syncthreads();  // the last reads of sU
#pragma unroll
      for (int t = 0; t < 2; ++t) sU[(NV - 2 + t) * SV + tid + 2 * W] = Ft[t];
    }
  }
  __syncthreads();

  // flux difference and output
  EmitArgs ea{};
  int64_t npts = 0;
  if constexpr (STEP) {
    const StageKernArgsPtr<ND> k = stage_kernargs<ND>();
    in = stage_in(k->in);
    npts = k->a[DIR].npts;
    ih = k->a[DIR].ih;
  } else {
    ea = emit_args(sweep_kernargs_late()->a);
    npts = a.npts;
  }
  // a batch stage has no residual of earlier sweeps (one direction):
  // known here, its reads and selects drop out of the epilogue
  if constexpr (BATCH) ea.Rin = nullptr;
  unsigned long long rbits = 0;  // wave rate of the lane's written node (SweepArgs::wmax)
#pragma unroll 1
  for (int q = tid; q < TL * W; q += NT) {
    const int t = q >> LW, c = q & (W - 1);
    int64_t i = i0 + t;
    if constexpr (LINES) {
      // q == tid here (one output node per lane)
      if (onode < 0) continue;  // a ghost slot
      if constexpr (BATCH) {
        dt = odt;
        if (mode == MODE_STAGE && dt == 0.0) continue;  // finished problem
        ih = oih;
      }
      base = onode;
      i = 0;
    } else {
      if (i >= N || c >= ncol) continue;
    }
    const double* f = sW + q;        // 2 F~ of midpoint t + k of column c at f[k W]
    const double* u = sU + q;        // node t + k of column c at u[k W]
    double res[NV], Un[NV];
    if (a.diff == 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const bool tv = TRIM && v >= NV - 2;
        Un[v] = tv ? Ut[v - (NV - 2)] : u[v * SV + 4 * W];
        const lds_cptr fv = lds_row(f + v * TMW);
        // F of node t + k + 2 at nf[k W]: nodes t + 3 and t + 5 around t + 4
        const lds_cptr nf = lds_row(tv ? u + v * SV + 2 * W : f + (NV + v) * TMW);
        double d;
        if constexpr (PLAIN)
          d = plain::diff_mnd6<W>(fv, nf);
        else
          d = __builtin_fma(
              0.75, fv[2 * W] - fv[W],
              __builtin_fma(-0.3, nf[3 * W] - nf[W], (1.0 / 60.0) * (fv[3 * W] - fv[0])));
        res[v] = -ih * d;
      }
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        Un[v] = u[v * SV + 5 * W];
        const lds_cptr fv = lds_row(f + v * TMW);
        double d;
        if constexpr (PLAIN)
          d = plain::diff_md6<W>(fv);
        else
          d = __builtin_fma(
              75.0 / 128.0, fv[3 * W] - fv[2 * W],
              __builtin_fma(-25.0 / 768.0, fv[4 * W] - fv[W], (3.0 / 1280.0) * (fv[5 * W] - fv[0])));
        res[v] = -ih * d;
      }
    }
    if constexpr (BATCH) {
      double y[NV];
      emit_rt<NV>(mode, ea, base + i * stride + c, npts, res, Un, dt, y);
      if (a.wmax && mode == MODE_STAGE) {
        const double ihv[1] = {ih};
        rbits = __builtin_bit_cast(unsigned long long, wave_rate<1>(y, a.pp.gamma, ihv));
      }
    } else if constexpr (STEP) {
      const int64_t gi = base + i * stride + c;
      const uint32_t off = (uint32_t)gi * 8;
#pragma unroll
      for (int v = 0; v < NV; ++v) at_bytes(in.Rout + DIR * in.rstride + v * npts, off) = res[v];
      if constexpr (DIR == 0) {
        // the x tiles, which hold each node once, keep U1 and check it, and
        // take U^n's wave rate for dt
        if (in.st == 2) {
#pragma unroll
          for (int v = 0; v < NV; ++v) at_bytes(in.U1 + v * npts, off) = Un[v];
          if (!physical<NV>(Un, a.pp.gamma)) flag_status(in.status);
        } else if (in.st == 1 && !in.dt) {
          rbits = __builtin_bit_cast(unsigned long long, wave_rate<ND>(Un, a.pp.gamma, in.ih));
        }
      }
    } else {
      emit_rt<NV>(mode, ea, base + i * stride + c, npts, res, Un, dt);
    }
  }
  if constexpr (STEP && DIR == 0) {
    if (in.st == 1 && !in.dt) {  // uniform
      const unsigned long long m = wave_max_bits(rbits);
      __syncthreads();  // the last reads of sU are done
      unsigned long long* sM = reinterpret_cast<unsigned long long*>(sU);
      if ((tid & 63) == 0) sM[tid >> 6] = m;
      __syncthreads();
      if (tid == 0)
        reinterpret_cast<unsigned long long*>(in.partial)[tile] =
            umax64(umax64(sM[0], sM[1]), umax64(sM[2], sM[3]));
    }
  }
  // The batch's last stage of a step also takes each problem's maximum wave
  // rate of the state it writes (uniform branch; every lane reaches it).
  if constexpr (BATCH) {
    if (a.wmax && mode == MODE_STAGE) {
      batch_rate_max(a.wmax, bt, near, oprob, rbits);
    }
  }
}

// Waves per SIMD that the compiler must leave room for, by specialisation (vector
// registers of the Euler kernels; the register path is that of 256-midpoint tiles with
// 4 and 5 variables):
//   FE, PFE, PLAIN_FE  six off the register path (FE 70-80, PFE 65-78); the 16x8 and
//            32x4 y and z tiles of 5 variables spill two registers there in FE and
//            PLAIN_FE.  Five on it (FE 87-95, PFE 75-91, no spill): at six the Roe state
//            spills, and the LDS of 5-variable tiles holds five workgroups on a CU.
//   JS, Z    six throughout (56-80); the 5-variable register path spills up to 16
//            registers for it, which costs what a wave fewer does (128^3 residual, six
//            and five waves: Z 0.331 and 0.334 ms, JS 0.305 and 0.306).
//   FE_SAT   five off the register path (90-96; 4 spilled in the 16x8 and 32x4 z tiles),
//            four on it (98-116).
//   run-time weights, PLAIN  unconstrained: 106-128, four waves (capped at 80 they spill).
#ifndef WCNS_REG_WAVES
#define WCNS_REG_WAVES 5
#endif
constexpr int sweep_waves(int nv, int tmw, int spec) {
  return spec == SPEC_GENERIC || spec == SPEC_PLAIN ? 1
         : spec == SPEC_JS || spec == SPEC_Z ? 6
         : spec == SPEC_FE_SAT               ? (sweep_reg(nv, tmw) ? 4 : 5)
         : sweep_reg(nv, tmw)                ? WCNS_REG_WAVES
                                             : 6;
}

inline int64_t ceil_div64(int64_t x, int64_t y) { return (x + y - 1) / y; }

inline TileGeom make_geom(int dir, const int64_t n[3], int diff, int tm, int w) {
  TileGeom g{};
  g.tm = tm;
  g.w = w;
  g.lw = 0;
  g.ltmw = 0;
  g.tl = tm - (diff ? 5 : 3);
  g.segs = ceil_div64(n[dir], g.tl);
  g.xgroups = dir == 0 ? 1 : ceil_div64(n[0], w);
  // (both below 2^31 whenever the tile count is, which the launch checks)
  g.dxg = fast_div((uint32_t)g.xgroups);
  g.dseg = fast_div((uint32_t)g.segs);
  const int64_t others = dir == 0 ? n[1] * n[2] : (dir == 1 ? n[2] : n[1]);
  g.ntiles = g.segs * g.xgroups * others;
  g.lines = 0;
  g.inv_line = 0.0;
  g.grid = 0;
  if (dir == 0) {  // packed x-lines
    const int64_t L = n[0] + 2 * (diff ? 5 : 4);
    g.lines = others;
    g.inv_line = 1.0 / (double)L;
    g.ntiles = ceil_div64(others * L, g.tl);
  }
  return g;
}

}  // namespace wcns
