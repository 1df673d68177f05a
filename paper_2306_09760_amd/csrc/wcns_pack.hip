// A whole SSP-RK3 step of a small ragged batch of 1D Euler problems in one launch.
//
// A small batch's step was a dt kernel and three stage launches of a few tiles per
// CU each, every one of them a trip to memory and back and about 5 us long however
// small the batch.  Here a workgroup keeps its window of the packed slots (see
// BatchArgs) in LDS through all three stages, each as in the sweep kernel (the
// same device functions in the same order and rounding: bitwise the sweeps' step).
// A stage reaches G nodes to each side, so a window of 133 slots steps 125 in the
// first stage, 117 in the second and completes 109 (MND6; 103 with MD6), and a
// problem has 3 G ghost slots on each side: periodic ones are stepped like the
// nodes they copy, of which they hold all that is needed; a transmissive one is
// stepped as its end node, from that node's fluxes, which lie in the window
// wherever an output needs the ghost.  A neighbour may read the state a window
// completes, so a step goes from one array to another.
// dt comes from the maxima of the step before: every window takes its problems'
// by itself, and the window with a problem's first node keeps it.
// 256 lanes: Roe averages on two wavefronts beside the nodes' fluxes on the other
// two, then one wavefront per 64 (field, midpoint) tasks, the two that do not take
// the midpoint fluxes afterwards with two of the six each.  (384 lanes, a task
// per wavefront, leave a CU three workgroups instead of six: 64 tubes of 2176
// nodes 40.2 against 32.8 us per step.)  What a lane knows of its slot waits in LDS
// and the kernel's arguments in their segment, which keeps FE within the 80
// registers of six waves per SIMD and free of spills (32.1 -> 30.8).
// Bound by FP64 issue from about five windows per CU on (3.4 us each for the three
// stages), below that by the chain of the phases.  Microseconds per step in calls
// of four, sweeps -> here (FE; one box): one tube of 500 nodes 22.1 -> 14.4, 32 of
// 2000 30.5 -> 21.1, 64 of 2176 37.8 -> 30.3, 96 45.0 -> 37.8.
#include <hip/hip_runtime.h>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

constexpr int kPackTM = 128, kPackTN = kPackTM + 5;
constexpr int kPackLanes = 256;

struct PackArgs {
  const double* U;
  double* out;
  int64_t npts;
  int bc, diff;
  int32_t* status;
  unsigned long long* wmax;
  PackDt d;
  BatchArgs b;  // tile_p0, tile_p1 and ntiles of these tiles
  InterpParams ip;
  PhysParams pp;
};

// The kernel's arguments, to be read from the argument segment where a phase
// needs them: held in scalar registers through the stages they spill to lanes of
// vector registers.
__device__ __forceinline__ const PackArgs& pack_args() {
  unsigned long long p = reinterpret_cast<unsigned long long>(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("" : "+s"(p));
  return *(const PackArgs*)reinterpret_cast<const __attribute__((address_space(4))) PackArgs*>(p);
}

constexpr int pack_waves(int spec) {
  return spec == SPEC_GENERIC ? 1 : spec == SPEC_FE_SAT ? 4 : 6;
}

template <int SPEC>
__global__ void __launch_bounds__(kPackLanes) __attribute__((amdgpu_waves_per_eu(pack_waves(SPEC))))
    pack_step_kernel(PackArgs) {
  constexpr int NV = 3, ND = 1, TM = kPackTM, TN = kPackTN;
  __shared__ double sU[NV * TN], sR[4 * TM], sW[2 * NV * TM], sF[NV * TM];
  __shared__ double sU0[NV * TN];  // U^n (a lane reads its own slot)
  __shared__ double sX[64];  // exp2_tab_entry
  // what a lane knows of its slot, out of its registers until the stages' ends:
  // 1/h and dt of the slot's problem, the problem, where the node that the slot
  // copies lies in the tile (-1: not to be stepped here) and its index where it
  // is an output of the tile (-1: none)
  __shared__ double sIh[TN], sDt[TN];
  __shared__ int sProb[TN], sPos[TN];
  __shared__ int64_t sNode[TN];
  const PackArgs& a = pack_args();
  if ((int)blockIdx.x >= a.b.ntiles) return;
  const int64_t tile = xcd_tile(blockIdx.x, a.b.ntiles);
  const int tid = threadIdx.x;
  if (a.d.nlive && tile == 0 && tid == 0) *a.d.nlive = 0;
  const int G = a.diff ? 5 : 4, R = 3 * G, TL = TN - 2 * R;
  const int64_t i0 = tile * TL;
  const BatchTile bt = batch_tile(a.b, tile, i0, R);
  const bool near = bt.p1 <= bt.p0 + 1;
  bool live = false;  // uniform across the block
  auto problem_dt = [&](int p) {
    if (!a.d.wmax) return BatchDt{a.b.dtp[p], 0.0, false};
    return batch_dt(__builtin_bit_cast(double, a.d.wmax[p]), a.d.t_in[p], a.d.t_end, a.d.cfl);
  };
  for (int p = bt.p0; p <= bt.p1; ++p) live |= problem_dt(p).dt != 0.0;

  // the lane's slot, r relative to i0
  if (tid < TN) {
    const int r = tid - R;
    const BatchSlot sl = near ? batch_slot_near(bt, r) : batch_slot(a.b, bt.p0, bt.p1, R, i0 + r);
    const int j = sl.j < -R ? -R : (sl.j >= sl.n + R ? sl.n + R - 1 : sl.j);
    const int64_t gi = sl.o + bc_index(j, sl.n, a.bc);
    double u0[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) u0[v] = a.U[v * a.npts + gi];
    sIh[tid] = a.b.ih[sl.p];
    const BatchDt d = problem_dt(sl.p);
    sDt[tid] = d.dt;
    sProb[tid] = sl.p;
    const int64_t onode = sl.j >= 0 && sl.j < sl.n && r >= 0 && r < TL ? gi : -1;
    if (onode >= 0 && sl.j == 0) {  // the problem's first node: its one lane
      if (a.d.clear) a.d.clear[sl.p] = 0;
      if (a.d.wmax) {
        a.b.dtp[sl.p] = d.dt;
        a.d.t_out[sl.p] = d.tn;
        if (d.bad) flag_status(a.status);
      }
    }
    sNode[tid] = onode;
    int pos = tid;
    if (a.bc != 0) pos += j < 0 ? -j : j >= sl.n ? sl.n - 1 - j : 0;
    if (pos < G || pos >= TN - G || sl.j != j) pos = -1;
    sPos[tid] = pos;
    if (!live) {
      if (onode >= 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) a.out[v * a.npts + onode] = u0[v];
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      sU0[v * TN + tid] = u0[v];
      sU[v * TN + tid] = u0[v];
    }
  }
  if (!live) return;
  if constexpr (spec_table(SPEC)) {
    const int x = tid - (kPackLanes - 64);  // (the wavefront with no node)
    if (x >= 0) sX[x] = exp2_tab_entry(x, a.ip.xsh);
  }
  __syncthreads();

  bool bad = false;
#pragma unroll 1
  for (int st = 0; st < 3; ++st) {
    const PackArgs& a = pack_args();
    const bool proj = a.pp.charproj;
    const int G = a.diff ? 5 : 4;
    // Roe averages on the first two wavefronts, the nodes' fluxes (MND6) on the
    // next two
    if (tid < TM) {
      if (proj) {
        const double* u = sU + tid + 2;
        double UA[NV], UB[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          UA[v] = u[v * TN];
          UB[v] = u[v * TN + 1];
        }
        const RoeState<ND> rs = roe_average<ND>(UA, UB, a.pp.gamma);
        sR[tid] = rs.vel[0];
        sR[TM + tid] = rs.H;
        sR[2 * TM + tid] = rs.c;
        sR[3 * TM + tid] = rs.ic;
      }
    } else if (tid < 2 * TM && a.diff == 0) {
      const int q = tid - TM;
      double Uc[NV], Fc[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Uc[v] = sU[v * TN + q + 2];
      node_flux<NV, 0>(a.pp, Uc, Fc);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[v * TM + q] = Fc[v];
    }
    __syncthreads();
    // the six values of field v around midpoint q
    auto stencil = [&](int v, int q, double (&w)[6]) {
      const double* u = sU + q;
      if (proj) {
        RoeState<ND> rs;
        rs.vel[0] = sR[q];
        rs.ic = sR[3 * TM + q];
        roe_derived<ND>(rs, a.pp.gamma);
        double l[NV];
        field_row<ND, 0>(rs, v, l);
        project_stencil<NV, TN, 1>(u, l, w);
      } else {
#pragma unroll
        for (int j = 0; j < 6; ++j) w[j] = u[v * TN + j];
      }
    };
    // one field of one midpoint per task, as in the sweeps
#pragma unroll 1
    for (int k = tid; k < NV * TM; k += tid < TM ? NV * TM : TM) {
      const int v = __builtin_amdgcn_readfirstlane(k >> 7), q = k & (TM - 1);
      double w[6];
      stencil(v, q, w);
      interp5_pair<SPEC>(a.ip, w, sW + v * TM + q, sW + (NV + v) * TM + q, sX);
    }
    __syncthreads();
    if (tid < TM) {  // twice the midpoint flux
      double F[NV];
#pragma unroll
      for (int pass = 0; pass < (spec_narrow(SPEC) ? 2 : 1); ++pass) {  // (as in sweep_tile)
        double WL[NV], WR[NV], UL[NV], UR[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          UL[v] = WL[v] = sW[v * TM + tid];
          UR[v] = WR[v] = sW[(NV + v) * TM + tid];
        }
        if (proj) {
          RoeState<ND> rs;
          rs.vel[0] = sR[tid];
          rs.H = sR[TM + tid];
          rs.c = sR[2 * TM + tid];
          rs.ic = sR[3 * TM + tid];
          roe_derived<ND>(rs, a.pp.gamma);
          unproject<ND, 0>(rs, WL, UL);
          unproject<ND, 0>(rs, WR, UR);
        }
        llf_flux2<ND, 0>(UL, UR, a.pp.gamma, F);
        if (!spec_narrow(SPEC) || pass > 0 || !overflown(F[NV - 1])) break;
        if constexpr (spec_narrow(SPEC)) {
#pragma unroll 1
          for (int v = 0; v < NV; ++v) {
            double w[6];
            stencil(v, tid, w);
            interp5_pair<SPEC, true>(a.ip, w, sW + v * TM + tid, sW + (NV + v) * TM + tid, sX);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[v * TM + tid] = F[v];
    }
    __syncthreads();
    // difference and stage combination at the lane's node
    const int pos = tid < TN ? sPos[tid] : -1;
    if (pos >= 0) {
      double uk[NV];
      const double ih = sIh[tid], dt = sDt[tid];
      const double ca = st == 0 ? 0.0 : st == 1 ? 0.75 : 1.0 / 3.0;
      const double cb = st == 0 ? 1.0 : st == 1 ? 0.25 : 2.0 / 3.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double* f = sW + v * TM + pos - G;
        const double* nf = sF + v * TM + pos - G;
        const double d =
            a.diff == 0
                ? __builtin_fma(0.75, f[2] - f[1],
                                __builtin_fma(-0.3, nf[3] - nf[1], (1.0 / 60.0) * (f[3] - f[0])))
                : __builtin_fma(75.0 / 128.0, f[3] - f[2],
                                __builtin_fma(-25.0 / 768.0, f[4] - f[1],
                                              (3.0 / 1280.0) * (f[5] - f[0])));
        uk[v] = stage_value(ca, cb, st == 0 ? 0.0 : sU0[v * TN + tid], sU[v * TN + tid], dt, -ih * d);
        sU[v * TN + tid] = uk[v];
      }
      if (sNode[tid] >= 0 && dt != 0.0) bad = bad || !physical<NV>(uk, a.pp.gamma);
    }
    __syncthreads();
  }
  const PackArgs& e = pack_args();
  unsigned long long rbits = 0;
  const int64_t onode = tid < TN ? sNode[tid] : -1;
  if (onode >= 0) {
    const bool on = sDt[tid] != 0.0;  // (a finished problem keeps its state)
    double uk[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      uk[v] = (on ? sU : sU0)[v * TN + tid];
      e.out[v * e.npts + onode] = uk[v];
    }
    if (on && e.wmax) {
      const double ihv[1] = {sIh[tid]};
      rbits = __builtin_bit_cast(unsigned long long, wave_rate<1>(uk, e.pp.gamma, ihv));
    }
  }
  if (bad) flag_status(e.status);
  if (e.wmax) batch_rate_max(e.wmax, bt, near, tid < TN ? sProb[tid] : bt.p0, rbits);
}

// --------------------------------------------------------------- launchers --
// Up to twelve windows per CU: a seventh of the midpoints is stepped twice or more,
// which a full chip pays for.  Sweeps -> here, calls of four steps and of one (with
// the copy back): 64 tubes of 2176 nodes (1290 windows) FE 37.8 -> 30.3, 44.9 ->
// 42.5, Z 31.8 -> 23.1, 36.5 -> 33.2; 128 (2600) FE 53.5 -> 47.2, 66.1 -> 64.7; 192
// (3880) FE 69.8 -> 63.8, 82.2 -> 84.7, Z 54.0 -> 48.5, 59.5 -> 63.7; 512 FE 147.6 ->
// 145.6, 165 -> 171.
//
// With FE and PFE maps at run time (116 registers, four wavefronts to a SIMD) up to four
// windows per CU, and three where a single step pays for the copy back (xi = 500,
// sweeps -> here, per call of four steps and of one): 20 tubes of 2000 nodes (367
// windows) FE 148 -> 132, 42.9 -> 41.3; 3000 of 9 (909) 193 -> 186, 52.0 -> 53.6;
// 400 of 200 (823) 182 -> 175, 48.2 -> 51.1, PFE 185 -> 184, 49.2 -> 53.8; 2000 of
// 50 (1358) FE 247 -> 267, 58 -> 71, PFE 248 -> 271, 59 -> 72.
int64_t pack_max_tiles(const InterpParams& ip, int nsteps) {
  return !run_time_maps(ip) ? 3072 : nsteps > 1 ? 1024 : 768;
}
int pack_tile_nodes(int diff) { return kPackTN - 6 * (diff ? 5 : 4); }
int pack_tile_ghosts(int diff) { return 3 * (diff ? 5 : 4); }

hipError_t launch_pack_step(const SweepArgs& s, const BatchArgs& b, const PackDt& d,
                            const double* U, double* out, hipStream_t stream) {
  PackArgs a;
  a.U = U;
  a.out = out;
  a.npts = s.npts;
  a.bc = s.bc;
  a.diff = s.diff;
  a.status = s.status;
  a.wmax = s.wmax;
  a.d = d;
  a.b = b;
  a.ip = s.ip;
  a.pp = s.pp;
#define WCNS_P(SP)                                                                                \
  case SP:                                                                                        \
    hipLaunchKernelGGL((pack_step_kernel<SP>), dim3((unsigned)b.ntiles), dim3(kPackLanes), 0,     \
                       stream, a);                                                                \
    break;
  switch (spec_of(a.ip)) {
    WCNS_P(SPEC_FE) WCNS_P(SPEC_FE_SAT) WCNS_P(SPEC_JS) WCNS_P(SPEC_Z) WCNS_P(SPEC_PFE)
    default:
    WCNS_P(SPEC_GENERIC)
  }
#undef WCNS_P
  return hipGetLastError();
}

}  // namespace wcns
