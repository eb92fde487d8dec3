// Whole time steps of small systems (every member in the small-member dipole
// layout): forces, gather, second half-kick and the next step's half-kick, drift
// and rotation without a launch between them.
//
// At these sizes a step's arithmetic is a few microseconds and the time goes to
// the launches around it: forces and kick as two kernels took about 5 us each at
// any N up to a few hundred, plus 1.5 us between them. Everything the update of
// a particle needs (its dipole sum, two bonds, contacts) can be had from the
// other particles' positions alone, so a workgroup that owns a few particles does
// all of it and only positions, orientations and moments pass from step to step:
//   k_step:  a workgroup per T particles, one launch per step; the state
//            alternates between two sets of planes, since other workgroups still
//            read the level that this one has finished with;
//   k_steps: a workgroup per member, a launch for many steps; the state stays in
//            LDS, with two barriers per step.
// In both, waves of their own evaluate the bonds while the others sum the
// dipoles (the two chains are about equally long), and the update of the
// particles is lane-parallel in the bond wave.
//
// Measured per step in graphs of 100 (one rod with dipoles, FP64 / mixed): N = 20
// 12.5 -> 3.5 / 3.3 us (k_steps), N = 128 12.6 -> 7.9 / 7.0 us (k_step); 32
// members of 200, mixed: 28 -> 17.5 us. k_steps takes members of up to 32
// particles: its few dipole waves need a round per handful of targets, 4.2 us at
// 32, 7.8 at 48 and 9.9 at 64, where k_step takes 7.0 to 7.6 at any of these.
// Their time grows once every compute unit has a workgroup: two of the five-wave ones
// share a unit (160 to 168 registers, three waves per SIMD), the nine-wave ones and those
// of k_steps (224 registers and more) wait for it. Which systems take them is
// small_form's (rod_api.hip).
#include <type_traits>

#include "rod.h"
#include "small_body.h"
#include "bond_core.h"
#include "particle_body.h"
#include "step_internal.h"

namespace rodmx {

// DAMP: the context has bond damping. A template argument: with both forms of
// bond_one behind a run-time branch the compiler hoists what they share out of
// them, which changes where products and sums contract, and so the last bit.

// Constants of bond k (between particles k and k + 1).
struct BondConst {
  V3<double> rref;
  double r0, K[4], g[4];  // reference vector and length, rod constants, damping factors
};
template <bool DAMP>
__device__ __forceinline__ BondConst bond_const(const Dev& d, long k) {
  const long N = d.n;
  const int rod = d.rod[k];
  BondConst c;
  c.rref = V3<double>{d.bref[k], d.bref[N + k], d.bref[2 * N + k]};
  c.r0 = d.bref[3 * N + k];
  for (int a = 0; a < 4; ++a) {
    c.K[a] = d.rodK[4 * rod + a];
    c.g[a] = DAMP ? d.bdamp[4 * rod + a] : 0.0;
  }
  return c;
}

// Bond k as bond_thread evaluates it; its measures of this level are recorded
// when `record`.
template <class R, bool DAMP>
__device__ __forceinline__ void small_bond(const Dev& d, long k, const BondConst& c, long long L,
                                           V3<double> x1, V3<double> x2, Q4<double> q1,
                                           Q4<double> q2, V3<double> dv, bool record,
                                           V3<double>& F, V3<double>& Ts, V3<double>& Tbt) {
  const long N = d.n;
  if constexpr (DAMP) {
    BondDamp dm;
    dm.gr = c.g[0]; dm.gs = c.g[1]; dm.gt = c.g[2]; dm.gb = c.g[3];
    const double* hprev = d.hist + (long)((L - 1) & 1) * 5 * N;
    for (int a = 0; a < 5; ++a) dm.hprev[a] = hprev[a * N + k];
    dm.rates = L >= d.hist_from;
    dm.dv = dv;
    dm.idt = 1.0 / d.dt;
    bond_one<double, R, true>(x1, x2, q1, q2, c.rref, c.r0, c.K, F, Ts, Tbt, nullptr, &dm);
    if (record && d.hist_write) {
      double* hnow = d.hist + (long)(L & 1) * 5 * N;
      for (int a = 0; a < 5; ++a) hnow[a * N + k] = dm.hnow[a];
    }
  } else {
    bond_one<double, R>(x1, x2, q1, q2, c.rref, c.r0, c.K, F, Ts, Tbt, nullptr);
  }
}

}  // namespace rodmx

#include "integrate_body.h"  // last: contraction within expressions from here on

namespace rodmx {

__device__ __forceinline__ V3<double> shfl3(V3<double> v, int from) {
  return V3<double>{__shfl(v.x, from), __shfl(v.y, from), __shfl(v.z, from)};
}

template <class R> __device__ __forceinline__ const R* moments(const Dev& d);
template <> __device__ __forceinline__ const float* moments(const Dev& d) { return d.muf; }
template <> __device__ __forceinline__ const double* moments(const Dev& d) { return d.mu; }

// One step's forces, closing half-kick and (unless o.last) the next step's
// opening half-kick, drift and rotation, for T particles per workgroup: NW waves
// take the targets in turn, the last wave the T + 1 bonds around them and then
// the update. T = 4 with a wave each up to 2048 particles (512 workgroups cover
// the chip, and a target's chain is as short as it gets); above, T = 16 with two
// targets per wave, which spends one wave's update on four times the particles.
template <class R, bool HM, bool DAMP, int NW, int T>
__global__ __launch_bounds__(64 * (NW + 1)) void k_step(Dev d, StepOut o) {
  __shared__ double sums[T][SMALL_OUT];
  const long N = d.n;
  const int i0 = blockIdx.x * T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const long long L = d.step[d.lc];
  if (wave < NW) {
    for (int t = wave; t < T && i0 + t < N; t += NW) {
      const int i = i0 + t;
      int b = 0, e = (int)N, xlo, xhi;
      if (d.M > 1) {
        const int m = d.mem[i];
        b = d.mrange[2 * m];
        e = d.mrange[2 * m + 1];
      }
      excluded_range(d, i, xlo, xhi);
      const SmallSrc<R> s{d.x, d.v, d.w, moments<R>(d), N, 0};
      small_target<R, HM>(d, s, i, b, e, xlo, xhi, L, sums[t]);
    }
    __syncthreads();
    return;
  }
  // bonds i0 - 1 + lane (lane 0's belongs to the workgroup before), and the
  // particles i0 + lane
  const long kb = i0 - 1 + lane, k = kb < 0 ? 0 : (kb < N ? kb : N - 1), k2 = k + 1 < N ? k + 1 : k;
  V3<double> bF, bTs, bTb;
  if (lane <= T) {
    V3<double> dv{0.0, 0.0, 0.0};
    if constexpr (DAMP) dv = ld3(d.v, N, k2) - ld3(d.v, N, k);
    small_bond<R, DAMP>(d, k, bond_const<DAMP>(d, k), L, ld3(d.x, N, k), ld3(d.x, N, k2), ld4(d.q, N, k), ld4(d.q, N, k2), dv,
                  lane > 0 && kb < N && (d.bflags[k] & 1), bF, bTs, bTb);
  }
  const bool valid = lane < T && i0 + lane < N;
  const long i = valid ? i0 + lane : i0;
  PIn p = load_particle(d, i);
  double fr[12];
  {
    const double* f = field_row(d, L, p.mem);
#pragma unroll
    for (int c = 0; c < 12; ++c) fr[c] = f[c];
  }
  const int nx = lane < 63 ? lane + 1 : lane;
  const Bonds bd{shfl3(bF, nx), shfl3(bTs, nx), shfl3(bTb, nx), bF, bTs, bTb, d.bflags[i]};
  const double mass = d.mass[i], inertia = d.inertia[i];
  if (i0 == 0 && lane == 0) {  // read above by this wave only after every wave began
    if (o.last) d.step[0] = L;
    else d.step[3 - d.lc] = L + 1;
  }
  __syncthreads();
  if (!valid) return;
  V3<double> F, T_, Fd{0.0, 0.0, 0.0}, Bd{0.0, 0.0, 0.0}, cF{0.0, 0.0, 0.0}, cT{0.0, 0.0, 0.0};
  const double* S = sums[lane];
  if (d.dipole_on)
    small_slot<R>(d.C, S, (double)(R)p.m.x, (double)(R)p.m.y, (double)(R)p.m.z, Fd, Bd);
  if (d.contact_on) {
    cF = V3<double>{S[10], S[11], S[12]};
    if constexpr (HM) cT = V3<double>{S[13], S[14], S[15]};
  }
  if (o.Bo) st3(o.Bo, N, i, Bd);
  gather_sum<HM>(d, i, ROD_TERM_ALL, fr, p, bd, mass, inertia, Fd, Bd, cF, cT, F, T_);
  kick(d, i, F, T_, p, o.keep, o.keep || o.last);
  if (o.last) {  // the state of the level, into the caller's planes
    if (o.keep) return;  // (a recorded level's own hold it)
    st3(o.x, N, i, p.x);
    st3(o.v, N, i, p.v);
    st4(o.q, N, i, p.q);
    st3(o.w, N, i, p.w);
    return;
  }
  advance_particle(d, p.b, L + 1, p.x, p.v, p.q, p.w, F, T_, p.minv, p.Iinv);
  st3(o.x, N, i, p.x);
  st3(o.v, N, i, p.v);
  st4(o.q, N, i, p.q);
  st3(o.w, N, i, p.w);
  const V3<double> m = qrot(p.q, p.mb);
  st3(o.mu, N, i, m);
  if (o.muf) st3(o.muf, N, i, V3<float>{(float)m.x, (float)m.y, (float)m.z});
}

// n steps of a member of at most STEPS_MAX particles from the level in d.step[0], by
// one workgroup: lane p < nm of the first wave owns particle p and evaluates its bond
// while the other waves sum the dipoles, 64 / W targets at a time each. Everything
// a particle has lives in LDS and is read where it is used: held in registers
// across the loop, beside the bond's and the update's temporaries, it spilled
// (eight waves leave 256 registers each; with sixteen and 128 the spills cost
// more than the waves gain: N = 20 FP64 6.7 us per step against 3.5). The FP64 forms
// still spill 12 to 28 bytes per lane, the mixed ones nothing.
constexpr int STEPS_THREADS = 512;
struct StepsSmem {
  double x[3 * STEPS_MAX], q[4 * STEPS_MAX], v[3 * STEPS_MAX], w[3 * STEPS_MAX];
  double bond[9 * STEPS_MAX];              // F, tau_s, tau_bt of bond (l, l + 1)
  double bc[12 * STEPS_MAX];               // its constants (BondConst)
  double pc[7 * STEPS_MAX];                // m_body, 1/m, 1/I, m, I
  double sums[STEPS_MAX + 1][SMALL_OUT];   // (the last entry for idle lane groups)
  double field[12];                        // the member's field row of the level
  int xr[STEPS_MAX][2];                    // index range of excluded neighbours
};

// With rec (a recorded run from level lvl0) level lvl0 + s goes to rec + s * rec_stride, in the
// planes of a recorded state followed by the dipole field, and the state read is
// left as it was.
template <class R, bool DAMP, int W>
__global__ __launch_bounds__(STEPS_THREADS) void k_steps(Dev d, long long lvl0, int n, double* rec,
                                                         long rec_stride) {
  constexpr long PM = STEPS_MAX;
  __shared__ StepsSmem S;
  __shared__ R sm[3 * STEPS_MAX];  // moments
  const long N = d.n;
  const int b = d.mrange[2 * blockIdx.x], e = d.mrange[2 * blockIdx.x + 1], nm = e - b;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = STEPS_THREADS / 64;
  if (!rec) lvl0 = d.step[0];
  const bool own = tid < nm;
  const long i = b + (own ? tid : 0);
  const long l = own ? tid : 0;
  const int mem = blockIdx.x;
  const int bcon = d.bc[i];
  const uint8_t flags = d.bflags[i];
  auto publish = [&](const PIn& p) {
    st3(S.x, PM, l, p.x);
    st4(S.q, PM, l, p.q);
    st3(S.v, PM, l, p.v);
    st3(S.w, PM, l, p.w);
    const V3<double> m = qrot(p.q, p.mb);
    sm[l] = (R)m.x; sm[PM + l] = (R)m.y; sm[2 * PM + l] = (R)m.z;
  };
  if (own) {
    PIn p = load_particle(d, i);
    const BondConst c = bond_const<DAMP>(d, i);
    st3(S.bc, PM, l, c.rref);
    S.bc[3 * PM + l] = c.r0;
    for (int a = 0; a < 4; ++a) {
      S.bc[(4 + a) * PM + l] = c.K[a];
      S.bc[(8 + a) * PM + l] = c.g[a];
    }
    st3(S.pc, PM, l, p.mb);
    S.pc[3 * PM + l] = p.minv;
    S.pc[4 * PM + l] = p.Iinv;
    S.pc[5 * PM + l] = d.mass[i];
    S.pc[6 * PM + l] = d.inertia[i];
    excluded_range(d, (int)i, S.xr[l][0], S.xr[l][1]);
    advance_particle(d, p.b, lvl0 + 1, p.x, p.v, p.q, p.w, ld3(d.F, N, i), ld3(d.T, N, i), p.minv,
                     p.Iinv);
    publish(p);
  }
  __syncthreads();
  for (int s = 1; s <= n; ++s) {
    const long long L = lvl0 + s;
    if (wave == 0) {
      if (own && (flags & 1)) {
        BondConst c;
        c.rref = ld3(S.bc, PM, l);
        c.r0 = S.bc[3 * PM + l];
        for (int a = 0; a < 4; ++a) {
          c.K[a] = S.bc[(4 + a) * PM + l];
          if constexpr (DAMP) c.g[a] = S.bc[(8 + a) * PM + l];
        }
        V3<double> bF, bTs, bTb;
        small_bond<R, DAMP>(d, i, c, L, ld3(S.x, PM, l), ld3(S.x, PM, l + 1), ld4(S.q, PM, l),
                      ld4(S.q, PM, l + 1), ld3(S.v, PM, l + 1) - ld3(S.v, PM, l), true, bF, bTs, bTb);
        st3(S.bond, PM, l, bF);
        st3(S.bond + 3 * PM, PM, l, bTs);
        st3(S.bond + 6 * PM, PM, l, bTb);
      }
    } else {
      if (wave == NW - 1 && (tid & 63) < 12) S.field[tid & 63] = field_row(d, L, mem)[tid & 63];
      constexpr int G = 64 / W;  // targets per wave
      for (int t0 = (wave - 1) * G; t0 < nm; t0 += (NW - 1) * G) {
        const int t = t0 + (tid & 63) / W, tv = t < nm ? t : t0;
        const SmallSrc<R> src{S.x, S.v, S.w, sm, PM, b};
        small_target<R, false, W>(d, src, b + tv, b, e, S.xr[tv][0], S.xr[tv][1], L,
                                  S.sums[t < nm ? t : STEPS_MAX]);
      }
    }
    __syncthreads();
    if (own) {
      PIn p;
      p.x = ld3(S.x, PM, l);
      p.v = ld3(S.v, PM, l);
      p.w = ld3(S.w, PM, l);
      p.q = ld4(S.q, PM, l);
      p.mb = ld3(S.pc, PM, l);
      p.m = qrot(p.q, p.mb);
      p.minv = S.pc[3 * PM + l];
      p.Iinv = S.pc[4 * PM + l];
      p.b = bcon;
      const long lm = l > 0 ? l - 1 : 0;
      const Bonds bd{ld3(S.bond, PM, l), ld3(S.bond + 3 * PM, PM, l), ld3(S.bond + 6 * PM, PM, l),
                     ld3(S.bond, PM, lm), ld3(S.bond + 3 * PM, PM, lm),
                     ld3(S.bond + 6 * PM, PM, lm), flags};
      V3<double> F, T, Fd{0.0, 0.0, 0.0}, Bd{0.0, 0.0, 0.0}, cF{0.0, 0.0, 0.0};
      const double* u = S.sums[l];
      if (d.dipole_on)
        small_slot<R>(d.C, u, (double)(R)p.m.x, (double)(R)p.m.y, (double)(R)p.m.z, Fd, Bd);
      if (d.contact_on) cF = V3<double>{u[10], u[11], u[12]};
      gather_sum<false>(d, i, ROD_TERM_ALL, S.field, p, bd, S.pc[5 * PM + l], S.pc[6 * PM + l], Fd, Bd,
                     cF, V3<double>{0.0, 0.0, 0.0}, F, T);
      const bool out = s == n && !rec;
      kick(d, i, F, T, p, out, out);
      if (rec) {
        double* r = rec + s * rec_stride;
        st3(r, N, i, p.x);
        st3(r + 3 * N, N, i, p.v);
        st4(r + 6 * N, N, i, p.q);
        st3(r + 10 * N, N, i, p.w);
        st3(r + 13 * N, N, i, F);
        st3(r + 16 * N, N, i, T);
        st3(r + 19 * N, N, i, Bd);
      }
      if (s < n) {
        advance_particle(d, p.b, L + 1, p.x, p.v, p.q, p.w, F, T, p.minv, p.Iinv);
        publish(p);
      } else if (out) {
        st3(d.x, N, i, p.x);
        st4(d.q, N, i, p.q);
      }
    }
    __syncthreads();
  }
  // the last workgroup to leave, when all have read the level
  if (tid == 0 && !rec && atomicAdd(d.left, 1u) == gridDim.x - 1) {
    *d.left = 0u;
    d.step[0] = lvl0 + n;
  }
}

template <class R, bool HM, bool DAMP>
static void step_variant(const Dev& d, const StepOut& o, hipStream_t s) {
  if (d.n <= 2048)
    hipLaunchKernelGGL((k_step<R, HM, DAMP, 4, 4>), dim3((unsigned)((d.n + 3) / 4)), dim3(64 * 5), 0,
                       s, d, o);
  else
    hipLaunchKernelGGL((k_step<R, HM, DAMP, 8, 16>), dim3((unsigned)((d.n + 15) / 16)), dim3(64 * 9),
                       0, s, d, o);
}
template <class R, bool DAMP>
static void steps_variant(const Dev& d, int max_member, long long lvl0, int n, double* rec,
                          long rec_stride, hipStream_t s) {
  const dim3 g((unsigned)d.M), b(STEPS_THREADS);
  if (max_member <= 16) hipLaunchKernelGGL((k_steps<R, DAMP, 16>), g, b, 0, s, d, lvl0, n, rec, rec_stride);
  else hipLaunchKernelGGL((k_steps<R, DAMP, 32>), g, b, 0, s, d, lvl0, n, rec, rec_stride);
}

template <class F>
static void by_form(const Dev& d, int precision, F&& f) {
  auto with = [&](auto r, auto hm) {
    if (d.bdamp) f(r, hm, std::true_type{});
    else f(r, hm, std::false_type{});
  };
  if (precision == 1) {
    if (d.hm) with(float{}, std::true_type{});
    else with(float{}, std::false_type{});
  } else {
    if (d.hm) with(double{}, std::true_type{});
    else with(double{}, std::false_type{});
  }
}

hipError_t launch_step(const Dev& d, int precision, const StepOut& o, hipStream_t s) {
  by_form(d, precision, [&](auto r, auto hm, auto damp) {
    step_variant<decltype(r), decltype(hm)::value, decltype(damp)::value>(d, o, s);
  });
  return hipGetLastError();
}

hipError_t launch_steps(const Dev& d, int precision, int max_member, long long lvl0, int n,
                        hipStream_t s, double* rec, long rec_stride) {
  by_form(d, precision, [&](auto r, auto, auto damp) {
    steps_variant<decltype(r), decltype(damp)::value>(d, max_member, lvl0, n, rec, rec_stride, s);
  });
  return hipGetLastError();
}

}  // namespace rodmx
