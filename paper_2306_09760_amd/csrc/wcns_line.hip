// A whole Runge-Kutta step of one short 1D problem in one launch.
//
// A step of a 1D plan was five launches (two for dt, three stages; eight for
// the four-stage scheme), each of a workgroup or two whose few microseconds
// went into the launch, the trip to memory and back and a half-empty CU.  Here
// one workgroup keeps the line in LDS through the step: the wave-rate maximum
// and dt, then the stages, each as in the sweep kernel (load | Roe | interp |
// flux | diff, the same device functions in the same order, so a step is
// bitwise the sweeps' step), with a wavefront per 64 (field, midpoint) tasks
// so that every field is interpolated at the same time.  A lane keeps its
// node's U^n and, in the four-stage scheme, the combination of the earlier
// stages; ghosts are written by the lane of the node they copy.
// Bound by latency: the chain of dependent FP64 operations of the phases and
// four barriers per stage.
// LDS (doubles): sU[NV][N + 2G] | sR[4][NM] (Euler) | sW[2 NV][NM] | the exp
// table | 16 partial maxima, NM = N + 3 (MND6) or N + 5 (MD6) midpoints rounded
// up to a multiple of 64.
#include <hip/hip_runtime.h>

#include "wcns_internal.hpp"
#include "wcns_sweep_common.hpp"

namespace wcns {

struct LineArgs {
  double* U;            // state, in place
  double* U1;           // the first two stage states of the RK3 step (may be null)
  double* U2;
  const double* dt;     // step size, or null: cfl / max rate, left in *dt_out
  double* dt_out;
  int32_t* status;
  double cfl, ih, adv_rate;
  int n, bc, diff;
  int stages;           // 3: SSP-RK3, 4: the scheme of eq. 16
  InterpParams ip;
  PhysParams pp;
};

__host__ __device__ constexpr int line_mids(int n, int diff) {
  return (n + (diff ? 5 : 3) + 63) & ~63;
}
static size_t line_lds(int nv, int n, int diff) {
  const int g = diff ? 5 : 4;
  return sizeof(double) * ((size_t)nv * (n + 2 * g) +
                           ((nv > 1 ? 4 : 0) + 2 * (size_t)nv) * line_mids(n, diff) + 64 + 16);
}

// One stage's result at a node: MODE_STAGE's combination a U0 + b (Uk + dt R)
// or MODE_LIN's a U0 + b Uk + c dt R (see emit).
template <int NV>
__device__ __forceinline__ void line_combine(bool lin, double ca, double cb, double cr, double dt,
                                             const double (&u0)[NV], const double (&uk)[NV],
                                             const double (&r)[NV], double (&y)[NV]) {
  const double crdt = cr * dt;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double s = lin ? __builtin_fma(crdt, r[v], cb * uk[v]) : cb * __builtin_fma(dt, r[v], uk[v]);
    y[v] = __builtin_fma(ca, ca != 0.0 ? u0[v] : 0.0, s);
  }
}

// (-u + u1 + 2 u2) / 3 of the four-stage scheme as rk4_sum_kernel rounds it: with u
// and u1 (st = 0), then with that and u2.
__device__ __forceinline__ double rk4_partial(int st, double a, double y) {
#pragma clang fp contract(off)
  return st == 0 ? __builtin_fma(-1.0 / 3.0, a, 1.0 / 3.0 * y) : a + 2.0 / 3.0 * y;
}

template <int NV, int SPEC>
__global__ void __launch_bounds__(1024) line_step_kernel(LineArgs a) {
  constexpr int ND = NV > 1 ? NV - 2 : 1;
  constexpr int NR = NV > 1 ? 4 : 0;  // vel, H, c, ic
  extern __shared__ double smem[];
  const int N = a.n, G = a.diff ? 5 : 4, SU = N + 2 * G, NM = line_mids(N, a.diff);
  const int mids = N + (a.diff ? 5 : 3);
  double* sU = smem;
  double* sR = sU + NV * SU;
  double* sW = sR + NR * NM;
  double* sX = sW + 2 * NV * NM;  // exp2_tab_entry
  unsigned long long* sM = (unsigned long long*)(sX + 64);
  const int tid = threadIdx.x, lanes = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = lanes >> 6;
  const bool own = tid < N;  // the lane's node

  // the node and the ghosts that copy it
  auto put = [&](const double (&y)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double* u = sU + v * SU + G;
      u[tid] = y[v];
      if (a.bc == 0) {
        if (tid < G) u[N + tid] = y[v];
        if (tid >= N - G) u[tid - N] = y[v];
      } else {
        if (tid == 0)
          for (int k = 1; k <= G; ++k) u[-k] = y[v];
        if (tid == N - 1)
          for (int k = 0; k < G; ++k) u[N + k] = y[v];
      }
    }
  };

  double u0[NV], acc[NV];
  unsigned long long rate = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) u0[v] = acc[v] = 0.0;
  if (own) {
#pragma unroll
    for (int v = 0; v < NV; ++v) u0[v] = a.U[(int64_t)v * N + tid];
    put(u0);
    if constexpr (NV > 1) {
      if (!a.dt) {
        const double ih[1] = {a.ih};
        rate = __builtin_bit_cast(unsigned long long, wave_rate<1>(u0, a.pp.gamma, ih));
      }
    }
  }
  if constexpr (spec_table(SPEC)) {
    if (tid < 64) sX[tid] = exp2_tab_entry(tid, a.ip.xsh);
  }
  if constexpr (NV > 1) {
    if (!a.dt) {
      rate = wave_max_bits(rate);
      if ((tid & 63) == 0) sM[wave] = rate;
    }
  }
  __syncthreads();
  double dt;
  if (a.dt) {
    dt = *a.dt;
  } else {
    double m = a.adv_rate;
    if constexpr (NV > 1) {
      unsigned long long top = sM[0];
      for (int w = 1; w < waves; ++w) top = umax64(top, sM[w]);
      m = __builtin_bit_cast(double, top);
    }
    dt = a.cfl / m;
    if (tid == 0) *a.dt_out = dt;
  }

  const bool proj = (NV > 1) && a.pp.charproj;
  bool bad = false;
#pragma unroll 1
  for (int st = 0; st < a.stages; ++st) {
    if constexpr (NV > 1) {
      if (proj) {
#pragma unroll 1
        for (int q = tid; q < mids; q += lanes) {
          const double* u = sU + q + 2;
          double UA[NV], UB[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            UA[v] = u[v * SU];
            UB[v] = u[v * SU + 1];
          }
          const RoeState<ND> rs = roe_average<ND>(UA, UB, a.pp.gamma);
          double* r = sR + q;
          r[0] = rs.vel[0];
          r[NM] = rs.H;
          r[2 * NM] = rs.c;
          r[3 * NM] = rs.ic;
        }
        __syncthreads();
      }
    }
    // the six values of field v around midpoint q
    auto stencil = [&](int v, int q, double (&w)[6]) {
      const double* u = sU + q;
      if (proj) {
        if constexpr (NV > 1) {
          RoeState<ND> rs;
          rs.vel[0] = sR[q];
          rs.ic = sR[3 * NM + q];
          roe_derived<ND>(rs, a.pp.gamma);
          double l[NV];
          field_row<ND, 0>(rs, v, l);
#pragma unroll
          for (int j = 0; j < 6; ++j) {
            double t = l[0] * u[j];
#pragma unroll
            for (int e = 1; e < NV; ++e) t = __builtin_fma(l[e], u[e * SU + j], t);
            w[j] = t;
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < 6; ++j) w[j] = u[v * SU + j];
      }
    };
    // one task = 64 midpoints of one field
    const int nw = NM >> 6;
#pragma unroll 1
    for (int k = wave; k < NV * nw; k += waves) {
      const int v = NV == 1 ? 0 : (k >= nw) + (k >= 2 * nw);
      const int q = ((k - v * nw) << 6) + (tid & 63);
      if (q < mids) {
        double w[6];
        stencil(v, q, w);
        interp5_pair<SPEC>(a.ip, w, sW + v * NM + q, sW + (NV + v) * NM + q, sX);
      }
    }
    __syncthreads();
    // twice the midpoint flux, and the physical flux of node q + 2 (MND6)
#pragma unroll 1
    for (int q = tid; q < mids; q += lanes) {
      double F[NV];
#pragma unroll
      for (int pass = 0; pass < (spec_narrow(SPEC) ? 2 : 1); ++pass) {  // (as in sweep_tile)
        if constexpr (NV == 1) {
          const double uL = sW[q], uR = sW[NM + q];
          F[0] = __builtin_fma(a.pp.adv, uL + uR, -__builtin_fabs(a.pp.adv) * (uR - uL));
        } else {
          double WL[NV], WR[NV], UL[NV], UR[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            UL[v] = WL[v] = sW[v * NM + q];
            UR[v] = WR[v] = sW[(NV + v) * NM + q];
          }
          if (proj) {
            RoeState<ND> rs;
            rs.vel[0] = sR[q];
            rs.H = sR[NM + q];
            rs.c = sR[2 * NM + q];
            rs.ic = sR[3 * NM + q];
            roe_derived<ND>(rs, a.pp.gamma);
            unproject<ND, 0>(rs, WL, UL);
            unproject<ND, 0>(rs, WR, UR);
          }
          llf_flux2<ND, 0>(UL, UR, a.pp.gamma, F);
        }
        if (!spec_narrow(SPEC) || pass > 0 || !overflown(F[NV - 1])) break;
        if constexpr (spec_narrow(SPEC)) {
#pragma unroll 1
          for (int v = 0; v < NV; ++v) {
            double w[6];
            stencil(v, q, w);
            interp5_pair<SPEC, true>(a.ip, w, sW + v * NM + q, sW + (NV + v) * NM + q, sX);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[v * NM + q] = F[v];
      if (a.diff == 0) {
        double Uc[NV], Fc[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) Uc[v] = sU[v * SU + q + 2];
        node_flux<NV, 0>(a.pp, Uc, Fc);
#pragma unroll
        for (int v = 0; v < NV; ++v) sW[(NV + v) * NM + q] = Fc[v];
      }
    }
    __syncthreads();
    // difference and combination; the lane's node and its ghosts are read by
    // nobody else until the barrier
    if (own) {
      double res[NV], uk[NV], y[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        uk[v] = sU[v * SU + G + tid];
        const double* f = sW + v * NM + tid;
        const double* nf = sW + (NV + v) * NM + tid;
        const double d =
            a.diff == 0
                ? __builtin_fma(0.75, f[2] - f[1],
                                __builtin_fma(-0.3, nf[3] - nf[1], (1.0 / 60.0) * (f[3] - f[0])))
                : __builtin_fma(75.0 / 128.0, f[3] - f[2],
                                __builtin_fma(-25.0 / 768.0, f[4] - f[1],
                                              (3.0 / 1280.0) * (f[5] - f[0])));
        res[v] = -a.ih * d;
      }
      if (a.stages == 3) {
        const double ca = st == 0 ? 0.0 : st == 1 ? 0.75 : 1.0 / 3.0;
        const double cb = st == 0 ? 1.0 : st == 1 ? 0.25 : 2.0 / 3.0;
        line_combine<NV>(false, ca, cb, 0.0, dt, u0, uk, res, y);
        double* out = st == 0 ? a.U1 : st == 1 ? a.U2 : nullptr;
        if (out) {
#pragma unroll
          for (int v = 0; v < NV; ++v) out[(int64_t)v * N + tid] = y[v];
        }
      } else if (st < 3) {
        // u1 = u + dt/2 L(u); u2 = u + dt/2 L(u1); u3 = u + dt L(u2)
        line_combine<NV>(true, st == 0 ? 0.0 : 1.0, st == 0 ? 1.0 : 0.0, st == 2 ? 1.0 : 0.5, dt,
                         u0, uk, res, y);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if (st < 2) acc[v] = rk4_partial(st, st == 0 ? u0[v] : acc[v], y[v]);
        }
      } else {
        // (-u + u1 + 2 u2)/3 + u3/3 + dt/6 L(u3)
        line_combine<NV>(true, 1.0, 1.0 / 3.0, 1.0 / 6.0, dt, acc, uk, res, y);
      }
      bad = bad || !physical<NV>(y, a.pp.gamma);
      if (st + 1 < a.stages) {
        put(y);
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) a.U[(int64_t)v * N + tid] = y[v];
      }
    }
    __syncthreads();
  }
  if (bad) flag_status(a.status);
}

// --------------------------------------------------------------- launchers --
// One node per lane, one workgroup's 64 KB of LDS (Euler: 573 nodes with MND6, 571 with
// MD6, the limit of the four-stage step), and short enough that one CU's latency
// beats the launches it saves.  Microseconds
// per step, launches of the sweeps against one launch (FE, xi = 100; one box):
// Euler SSP-RK3, CFL-limited, 60 nodes 22.3 -> 12.4, 201 21.2 -> 16.2, 300 21.6
// -> 19.4, 400 21.7 -> 22.5; four stages 60 32.0 -> 15.7, 201 32.8 -> 20.2, 400
// 34.6 -> 28.4, 500 34.7 -> 28.6; Z weights 201 21.8 -> 11.6, 500 21.4 -> 15.8;
// advection with a given dt, 200 nodes 13.4 -> 8.4, 1000 13.5 -> 11.8.  The RK3
// line for Euler is drawn where the FE step breaks even.
// FE maps at run time keep three of four wavefronts of a SIMD busy up to 256
// midpoints (xi = 500, RK3 253 nodes 28.9 -> 25.6, four stages 44.2 -> 33.4); the
// fourth costs what the launches do (254 nodes 26.7 -> 30.9, 38.2 -> 40.3; 320 26.6
// -> 36.0, 38.1 -> 47.0; 573 four stages 38.9 -> 59.3).  PFE interpolates most
// midpoints without its maps and gains throughout (320 27.6 -> 27.1, 39.6 -> 35.1; 573
// 40.1 -> 33.9).
bool line_step_ok(int nv, int64_t n, int diff, int stages, const InterpParams& ip) {
  if (nv == 1) return n <= 1024;
  if (nv != 3 || n > 1024) return false;
  if (ip.weights == WFE && run_time_maps(ip) && line_mids((int)n, diff) > 256) return false;
  return (stages == 4 || n <= 320) && line_lds(nv, (int)n, diff) <= 64 * 1024;
}

hipError_t launch_line_step(int nv, const SweepArgs& s, double* U, double* U1, double* U2,
                            const double* dt, double cfl, double adv_rate, double* dt_out,
                            int stages, hipStream_t stream) {
  LineArgs a;
  a.U = U;
  a.U1 = U1;
  a.U2 = U2;
  a.dt = dt;
  a.dt_out = dt_out;
  a.status = s.status;
  a.cfl = cfl;
  a.ih = s.ih;
  a.adv_rate = adv_rate;
  a.n = (int)s.n[0];
  a.bc = s.bc;
  a.diff = s.diff;
  a.stages = stages;
  a.ip = s.ip;
  a.pp = s.pp;
  const int nm = line_mids(a.n, a.diff);
  const int lanes = nv * nm < 1024 ? nv * nm : 1024;
  const size_t lds = line_lds(nv, a.n, a.diff);
#define WCNS_L(NVV, SP)                                                                         \
  if (nv == NVV && spec_of(a.ip) == SP) {                                                       \
    hipLaunchKernelGGL((line_step_kernel<NVV, SP>), dim3(1), dim3((unsigned)lanes), lds, stream, a); \
    return hipGetLastError();                                                                   \
  }
  WCNS_L(1, SPEC_GENERIC) WCNS_L(1, SPEC_FE) WCNS_L(1, SPEC_FE_SAT) WCNS_L(1, SPEC_JS)
  WCNS_L(1, SPEC_Z) WCNS_L(1, SPEC_PFE)
  WCNS_L(3, SPEC_GENERIC) WCNS_L(3, SPEC_FE) WCNS_L(3, SPEC_FE_SAT) WCNS_L(3, SPEC_JS)
  WCNS_L(3, SPEC_Z) WCNS_L(3, SPEC_PFE)
#undef WCNS_L
  return hipErrorInvalidValue;
}

}  // namespace wcns
