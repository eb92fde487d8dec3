// Per-particle arithmetic of the time step, shared by the particle kernels
// (k_integrate.hip) and the fused step of small systems (k_step.hip): the
// Richardson quaternion update, half-kick and drift, the sum of a particle's
// force terms. Products and sums contract only within one expression
// (contract(on) from here to the end of the file that includes this header,
// after every other header), so that every kernel rounds alike.
#pragma once
#include "rod_internal.h"
#include "rod_math.h"
#include "particle_body.h"

#pragma clang fp contract(on)

namespace rodmx {

// dq/dt = 1/2 (0, w) q for a space-frame angular velocity w.
__device__ __forceinline__ Q4<double> q_rate(Q4<double> q, V3<double> w) {
  return qscale(0.5, qmul(Q4<double>{0.0, w.x, w.y, w.z}, q));
}

// Richardson extrapolation of one full step against two half steps, each
// intermediate renormalised: q(t+dt) = N(2 q2 - q1).
__device__ __forceinline__ Q4<double> richardson(Q4<double> q, V3<double> w, double dt) {
  Q4<double> rq = q_rate(q, w);
  Q4<double> q1 = qnormalize(qadd(q, qscale(dt, rq)));
  Q4<double> qh = qnormalize(qadd(q, qscale(0.5 * dt, rq)));
  Q4<double> q2 = qnormalize(qadd(qh, qscale(0.5 * dt, q_rate(qh, w))));
  return qnormalize(qadd(qscale(2.0, q2), qscale(-1.0, q1)));
}

__device__ __forceinline__ Q4<double> drive_q(const Dev& d, long long lvl) {
  double phi = 2.0 * 3.14159265358979323846 * (double)lvl / (double)d.period;
  double s, c;
  sincos(0.5 * phi, &s, &c);
  return {c, s * d.axis[0], s * d.axis[1], s * d.axis[2]};
}

// State of a free particle advanced from level lvl - 1 to level lvl (in
// registers): half-kick, drift and quaternion update; the imposed rotation of a
// driven one.
__device__ __forceinline__ void advance_particle(const Dev& d, int b, long long lvl, V3<double>& x,
                                                 V3<double>& v, Q4<double>& q, V3<double>& w,
                                                 V3<double> F, V3<double> T, double minv,
                                                 double Iinv) {
  if (b == 0) {
    const double h = 0.5 * d.dt;
    v = v + (h * minv) * F;
    x = x + d.dt * v;
    w = w + (h * Iinv) * T;
    q = richardson(q, w, d.dt);
  } else if (b == 2) {
    q = drive_q(d, lvl);
  }
}

// Advance particle i from its state at level lvl - 1 (in registers) to level
// lvl: half-kick, drift and quaternion update of free particles; the imposed
// rotation of driven ones. The result goes to the planes of d.nx when set,
// else in place; states of particles that do not move are written only when
// `copy_still` is set (out-of-place step). A particle too far from its place at the
// last list build sets rebuild[flag], the entry of the coming force evaluation (unless
// `check` is off: the caller looks itself).
__device__ __forceinline__ void advance(const Dev& d, long i, int b, long long lvl, V3<double>& x,
                                        V3<double>& v, Q4<double>& q, V3<double>& w,
                                        V3<double> F, V3<double> T, double minv, double Iinv,
                                        bool copy_still, int flag, bool check = true) {
  const long N = d.n;
  // output planes: those of the next recorded state, or in place
  double* const xo = d.nx ? d.nx : d.x;
  double* const vo = d.nx ? d.nx + 3 * N : d.v;
  double* const qo = d.nx ? d.nx + 6 * N : d.q;
  double* const wo = d.nx ? d.nx + 10 * N : d.w;
  advance_particle(d, b, lvl, x, v, q, w, F, T, minv, Iinv);
  if (b == 0) {
    if (d.use_lists && check) {  // moved too far since the contact lists were built?
      const V3<double> m = x - ld3(d.xb, N, i);
      const double lim = NBR_MOVE * d.skin;
      const bool far = dot(m, m) > lim * lim;
      const unsigned long long who = __ballot(far);  // one atomic per wave
      if (far && __lane_id() == (unsigned)(__ffsll((long long)who) - 1))
        atomicOr(&d.rebuild[flag], 1u);
    }
    st3(vo, N, i, v);
    st3(xo, N, i, x);
    st3(wo, N, i, w);
    st4(qo, N, i, q);
  } else {
    if (copy_still || b == 2) st4(qo, N, i, q);
    if (copy_still) {
      st3(xo, N, i, x);
      st3(vo, N, i, v);
      st3(wo, N, i, w);
    }
  }
}

__device__ __forceinline__ bool finite3(V3<double> a) {
  return isfinite(a.x) && isfinite(a.y) && isfinite(a.z);
}

// State of one particle as read at the start of a gather: every load that does
// not depend on another is issued before any arithmetic or store.
struct PIn {
  V3<double> x, v, w, m, mb;
  Q4<double> q;
  double minv, Iinv;
  int b, mem, rod;
};
__device__ __forceinline__ PIn load_particle(const Dev& d, long i) {
  const long N = d.n;
  return {ld3(d.x, N, i), ld3(d.v, N, i), ld3(d.w, N, i), ld3(d.mu, N, i), ld3(d.mb, N, i),
          ld4(d.q, N, i), d.minv[i], d.Iinv[i], d.bc[i], d.mem[i], d.rod[i]};
}

// The two bonds of a particle: (i, i+1) and (i-1, i), with the flags saying which
// of them exist.
struct Bonds {
  V3<double> F0, Ts0, Tb0, F1, Ts1, Tb1;
  uint8_t flags;
};

// Field table row of level lvl for a member.
__device__ __forceinline__ const double* field_row(const Dev& d, long long lvl, int mem) {
  const long long L = d.field_len;
  const long long row = ((lvl % L) + L) % L;
  return d.field + (row * d.M + mem) * 12;
}

// Total force and torque on particle i from the terms in `mask` at level lvl
// (bond, dipole, Zeeman, contact, damping, external), with the dipole force Fd
// and field Bd, the contact force cF and torque cT, the particle's two bonds and
// its field row f.
// HM: the contact law is Hertz-Mindlin, whose contacts also exert a torque (a
// template argument, so that the Hookean kernels carry no extra load). FL: the
// immersed-boundary penalty m_p / dt_fluid (U_p - v_p) with the velocity the
// evaluation sees, also stored to d.ibm_f.
template <bool HM, bool FL = false>
__device__ __forceinline__ void gather_sum(const Dev& d, long i, int mask, const double* f,
                                           const PIn& p, const Bonds& bd, double mass,
                                           double inertia, V3<double> Fd, V3<double> Bd,
                                           V3<double> cF, V3<double> cT, V3<double>& F,
                                           V3<double>& T) {
  const long N = d.n;
  F = V3<double>{0.0, 0.0, 0.0};
  T = V3<double>{0.0, 0.0, 0.0};
  if (mask & 1) {  // bonds: +F, tau_s + tau_bt from bond (i, i+1); -F, tau_s - tau_bt from (i-1, i)
    if (bd.flags & 1) {
      F = F + bd.F0;
      T = T + bd.Ts0 + bd.Tb0;
    }
    if (bd.flags & 2) {
      F = F - bd.F1;
      T = T + bd.Ts1 - bd.Tb1;
    }
  }
  const V3<double> m = p.m;
  if ((mask & 2) && d.dipole_on) {  // dipole-dipole: force and torque m x B_dip
    F = F + Fd;
    T = T + cross(m, Bd);
  }
  if (mask & 4) {  // Zeeman: B = B0 + G x, f = G^T m, tau = m x B
    const V3<double> x = p.x;
    V3<double> B{f[0] + f[3] * x.x + f[4] * x.y + f[5] * x.z,
                 f[1] + f[6] * x.x + f[7] * x.y + f[8] * x.z,
                 f[2] + f[9] * x.x + f[10] * x.y + f[11] * x.z};
    F = F + V3<double>{f[3] * m.x + f[6] * m.y + f[9] * m.z,
                       f[4] * m.x + f[7] * m.y + f[10] * m.z,
                       f[5] * m.x + f[8] * m.y + f[11] * m.z};
    T = T + cross(m, B);
  }
  if ((mask & 8) && d.contact_on) {  // contact (Hertz-Mindlin: also its torque)
    F = F + cF;
    if constexpr (HM) T = T + cT;
  }
  if (mask & 16) {  // global viscous damping with the current (half-step) velocities
    F = F - (d.damping * mass) * p.v;
    T = T - (d.damping * inertia) * p.w;
  }
  if constexpr (FL) {
    const V3<double> Fp = (mass * d.ibm_idt) * (ld3(d.ibm_u, N, i) - p.v);
    F = F + Fp;
    st3(d.ibm_f, N, i, Fp);
  }
  if (mask & 32) {
    if (d.extF) F = F + ld3(d.extF, N, i);
    if (d.extT) T = T + ld3(d.extT, N, i);
  }
}

// gather_sum with everything loaded from the work buffers of the separate force
// kernels. Loads are unconditional where the index is valid, so they are all in
// flight together.
template <bool HM, bool FL = false>
__device__ __forceinline__ void gather(const Dev& d, long i, int mask, long long lvl, double* Bo,
                                       const PIn& p, V3<double> Fd, V3<double> Bd, V3<double>& F,
                                       V3<double>& T) {
  const long N = d.n;
  const long im = i > 0 ? i - 1 : 0;
  const Bonds bd{ld3(d.bF, N, i), ld3(d.bTs, N, i), ld3(d.bTbt, N, i),
                 ld3(d.bF, N, im), ld3(d.bTs, N, im), ld3(d.bTbt, N, im), d.bflags[i]};
  const V3<double> cF = d.contact_on ? ld3(d.cF, N, i) : V3<double>{0.0, 0.0, 0.0};
  V3<double> cT{0.0, 0.0, 0.0};  // used only with HM
  if constexpr (HM) cT = ld3(d.cT, N, i);
  if (Bo) st3(Bo, N, i, Bd);
  gather_sum<HM, FL>(d, i, mask, field_row(d, lvl, p.mem), p, bd, d.mass[i], d.inertia[i], Fd, Bd,
                     cF, cT, F, T);
}

// Store the forces of the state (unless a later step of the same launch chain
// overwrites them: store_f) and apply the second half-kick to free
// particles, updating p.v and p.w (stored when `store_vw`; the fused kick
// overwrites them with the next half-kick anyway). Flags non-finite values.
__device__ __forceinline__ void kick(const Dev& d, long i, V3<double> F, V3<double> T, PIn& p,
                                     bool store_vw, bool store_f = true) {
  const long N = d.n;
  if (store_f) {
    st3(d.F, N, i, F);
    st3(d.T, N, i, T);
  }
  if (p.b == 0) {
    const double h = 0.5 * d.dt;
    p.v = p.v + (h * p.minv) * F;
    p.w = p.w + (h * p.Iinv) * T;
    if (store_vw) {
      st3(d.v, N, i, p.v);
      st3(d.w, N, i, p.w);
    }
  }
  if (!finite3(F) || !finite3(T) || !finite3(p.x)) atomicOr(&d.flags[FLAG_NONFINITE], 1u);
}

}  // namespace rodmx
