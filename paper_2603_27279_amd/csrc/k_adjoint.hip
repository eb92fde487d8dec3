// Reverse pass of the time step: gradients of a function of the final state
// with respect to the body dipoles, the field table and the initial state,
// by checkpoint-and-recompute through the recorded steps. All adjoint
// arithmetic is FP64.
//
// One step n -> n+1 of the forward loop (SI "Equations of motion") is
//   v' = v + h F/m, x1 = x + dt v', w' = w + h T/I, q1 = Rich(q, w')   (pre)
//   (F1, T1) = forces(x1, q1, v', w', m_body, field[n+1])             (forces)
//   v1 = v' + h F1/m, w1 = w' + h T1/I                                 (post)
// with h = dt/2, for free particles (clamped ones never move; driven ones
// follow a prescribed rotation). The reverse step takes the cotangent of the
// state at n+1 and returns the one at n:
//   post: v'-bar = v1-bar, F1-bar += h v1-bar / m (likewise for w, T);
//   forces: vector-Jacobian products of every force term (below);
//   pre: the Richardson update differentiated step by step, x-bar passes
//        through, v'-bar += dt x1-bar, F-bar = h v'-bar / m.
// Force terms:
//   bonds   - exact Jacobian columns of the bond function from forward-mode
//             dual numbers (11 inputs: r_f, q1, q2), contracted with the
//             bond's cotangent (F-bar_k - F-bar_{k+1}, T-bar_k + T-bar_{k+1},
//             T-bar_k - T-bar_{k+1});
//   dipoles - closed-form Hessian-vector products of the pair potential
//             U(r, a, b) = (a.b)/r^3 - 3 (a.r)(b.r)/r^5 (force = -dU/dr, field
//             = -dU/da), evaluated once with i as target and once as source;
//   Zeeman, torque m x B, damping, contact, and m = R(q) m_body - by hand.
#include "rod_adjoint.h"
#include "small_body.h"  // (before dual.h, whose sqrt would hide the library's)
#include "bond_core.h"
#include "dual.h"
#include "particle_body.h"
#include "fixsum.h"
#include "step_internal.h"

#include <algorithm>

namespace rodmx {

enum AdjMode { ADJ_STEP = 0, ADJ_PREPARE = 1 };

__device__ __forceinline__ V3<double> ldv(const double* p, long N, long i) { return ld3(p, N, i); }

__device__ __forceinline__ Q4<double> qv(V3<double> v) { return {0.0, v.x, v.y, v.z}; }
__device__ __forceinline__ V3<double> vec(Q4<double> q) { return {q.x, q.y, q.z}; }

// ---------------------------------------------------------------- Richardson VJP
// Cotangent of the normalisation y -> y/|y|: (v - n (n.v)) / |y|.
__device__ __forceinline__ Q4<double> jn(Q4<double> y, Q4<double> v) {
  const double s = 1.0 / ::sqrt(qdot(y, y));
  const Q4<double> n = qscale(s, y);
  return qscale(s, qadd(v, qscale(-qdot(n, v), n)));
}

// Given q, the half-step angular velocity w and the cotangent of the updated
// orientation, add the cotangents of q and w.
__device__ void richardson_vjp(Q4<double> q, V3<double> w, double dt, Q4<double> qbar_new,
                               Q4<double>& qbar, V3<double>& wbar) {
  const Q4<double> p{0.0, w.x, w.y, w.z};
  const Q4<double> pc{0.0, -w.x, -w.y, -w.z};
  auto rate = [&](Q4<double> a) { return qscale(0.5, qmul(p, a)); };
  const Q4<double> y1 = qadd(q, qscale(dt, rate(q)));
  const Q4<double> q1 = qnormalize(y1);
  const Q4<double> yh = qadd(q, qscale(0.5 * dt, rate(q)));
  const Q4<double> qh = qnormalize(yh);
  const Q4<double> y2 = qadd(qh, qscale(0.5 * dt, rate(qh)));
  const Q4<double> q2 = qnormalize(y2);
  const Q4<double> yn = qadd(qscale(2.0, q2), qscale(-1.0, q1));
  const Q4<double> ybn = jn(yn, qbar_new);
  const Q4<double> yb2 = jn(y2, qscale(2.0, ybn));
  const Q4<double> yb1 = jn(y1, qscale(-1.0, ybn));
  // y2 = qh + (dt/2) 1/2 p qh
  const Q4<double> qbh = qadd(yb2, qscale(0.25 * dt, qmul(pc, yb2)));
  V3<double> wb = 0.25 * dt * vec(qmul(yb2, qconj(qh)));
  const Q4<double> ybh = jn(yh, qbh);
  // yh = q + (dt/2) 1/2 p q ;  y1 = q + dt 1/2 p q
  qbar = qadd(qbar, qadd(qadd(ybh, qscale(0.25 * dt, qmul(pc, ybh))),
                         qadd(yb1, qscale(0.5 * dt, qmul(pc, yb1)))));
  wb = wb + 0.25 * dt * vec(qmul(ybh, qconj(q))) + 0.5 * dt * vec(qmul(yb1, qconj(q)));
  wbar = wbar + wb;
}

// ---------------------------------------------------------------- local terms
// Cotangent of one particle's state.
struct Cot {
  V3<double> x, v, w, F, T;
  Q4<double> q;
};

// What the local terms of a particle read besides its cotangent and moment: loaded
// in one go, so that it is all in flight together (and, in the fused step, before
// the barrier).
struct LocalIn {
  int b;
  double minv, Iinv, mass, inertia;
  V3<double> w0, T0, x1, Bd;
  double f[12];  // field row
};
__device__ __forceinline__ LocalIn adj_local_in(const Dev& d, long i, const double* S0,
                                                const double* S1, long long lvl) {
  const long N = d.n;
  LocalIn in{d.bc[i],          d.minv[i],     d.Iinv[i], d.mass[i], d.inertia[i],
             ldv(S0 + 10 * N, N, i), ldv(S0 + 16 * N, N, i), ldv(S1, N, i), ldv(S1 + 19 * N, N, i), {}};
  const long long L = d.field_len;
  const long long row = ((lvl % L) + L) % L;
  const double* f = d.field + (row * d.M + d.mem[i]) * 12;
#pragma unroll
  for (int k = 0; k < 12; ++k) in.f[k] = f[k];
  return in;
}

// Post-kick VJP and the per-particle force terms (Zeeman, dipole torque,
// damping). S1 is the state of the level whose forces are reversed; S0 the
// state one level earlier (ADJ_STEP only).
__device__ __forceinline__ void adj_local_of(const Dev& d, const Adj& a, long i, const LocalIn& in,
                                             V3<double> m, const Cot& c, int mode) {
  const long N = d.n;
  const bool free_p = in.b == 0;
  const double h = 0.5 * d.dt;
  V3<double> Fe{0, 0, 0}, Te{0, 0, 0}, vb{0, 0, 0}, wb{0, 0, 0};
  if (free_p) {
    Fe = c.F;
    Te = c.T;
    vb = c.v;
    wb = c.w;
    if (mode == ADJ_STEP) {
      Fe = Fe + (h * in.minv) * c.v;
      Te = Te + (h * in.Iinv) * c.w;
      // half-step angular velocity of the step, for the Richardson VJP
      st3(a.wh, N, i, in.w0 + (h * in.Iinv) * in.T0);
    }
  }
  // damping: F = -c m v', T = -c I w'
  vb = vb - (d.damping * in.mass) * Fe;
  wb = wb - (d.damping * in.inertia) * Te;
  const V3<double> x1 = in.x1;
  const double* f = in.f;
  const V3<double> Be{f[0] + f[3] * x1.x + f[4] * x1.y + f[5] * x1.z,
                      f[1] + f[6] * x1.x + f[7] * x1.y + f[8] * x1.z,
                      f[2] + f[9] * x1.x + f[10] * x1.y + f[11] * x1.z};
  // torque m x (B_dip + B_ext): m-bar += B x T-bar, B-bar = T-bar x m
  const V3<double> Bt = in.Bd + Be;
  const V3<double> hb = cross(Te, m);
  // Zeeman force G^T m: m-bar += G F-bar
  const V3<double> GF{f[3] * Fe.x + f[4] * Fe.y + f[5] * Fe.z,
                      f[6] * Fe.x + f[7] * Fe.y + f[8] * Fe.z,
                      f[9] * Fe.x + f[10] * Fe.y + f[11] * Fe.z};
  st3(a.mloc, N, i, cross(Bt, Te) + GF);
  // B_ext = B0 + G x1: x-bar += G^T B-bar
  st3(a.xloc, N, i, V3<double>{f[3] * hb.x + f[6] * hb.y + f[9] * hb.z,
                               f[4] * hb.x + f[7] * hb.y + f[10] * hb.z,
                               f[5] * hb.x + f[8] * hb.y + f[11] * hb.z});
  st3(a.h, N, i, hb);
  st3(a.Fe, N, i, Fe);
  st3(a.Te, N, i, Te);
  st3(a.vbar, N, i, vb);
  st3(a.wbar, N, i, wb);
  const double hbv[3] = {hb.x, hb.y, hb.z}, xv[3] = {x1.x, x1.y, x1.z},
               mv[3] = {m.x, m.y, m.z}, Fv[3] = {Fe.x, Fe.y, Fe.z};
  for (int k = 0; k < 3; ++k) a.fieldc[k * N + i] = hbv[k];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) a.fieldc[(3 + 3 * r + c) * N + i] = hbv[r] * xv[c] + mv[r] * Fv[c];
}
__device__ __forceinline__ void adj_local(const Dev& d, const Adj& a, long i, const double* S0,
                                          const double* S1, int koff, int mode) {
  const long N = d.n;
  const Cot c{V3<double>{0, 0, 0}, ldv(a.cv, N, i), ldv(a.cw, N, i), ldv(a.cF, N, i), ldv(a.cT, N, i), {}};
  adj_local_of(d, a, i, adj_local_in(d, i, S0, S1, *a.lbase + koff), ldv(d.mu, N, i), c, mode);
}

// ---------------------------------------------------------------- bonds
// Column `dir` of bond k's Jacobian by a dual-number evaluation: the derivatives of
// F, tau_s and tau_b + tau_t with respect to one of its 11 inputs.
struct BondColumn { V3<double> F, Ts, Tbt; };
__device__ __forceinline__ BondColumn bond_column(const Dev& d, const double* S1, long k, int dir) {
  const long N = d.n;
  const V3<double> x1 = ldv(S1, N, k), x2 = ldv(S1, N, k + 1);
  const Q4<double> q1 = ld4(S1 + 6 * N, N, k), q2 = ld4(S1 + 6 * N, N, k + 1);
  const V3<double> rref{d.bref[k], d.bref[N + k], d.bref[2 * N + k]};
  const double r0 = d.bref[3 * N + k];
  const double* K4 = d.rodK + 4 * d.rod[k];
  auto sd = [&](int c) { return dir == c ? 1.0 : 0.0; };
  V3<DD> X1{DD(x1.x), DD(x1.y), DD(x1.z)};
  V3<DD> X2{DD(x2.x, sd(0)), DD(x2.y, sd(1)), DD(x2.z, sd(2))};
  Q4<DD> Q1{DD(q1.w, sd(3)), DD(q1.x, sd(4)), DD(q1.y, sd(5)), DD(q1.z, sd(6))};
  Q4<DD> Q2{DD(q2.w, sd(7)), DD(q2.x, sd(8)), DD(q2.y, sd(9)), DD(q2.z, sd(10))};
  V3<DD> F, Ts, Tbt;
  bond_one<DD, DD>(X1, X2, Q1, Q2, rref, r0, K4, F, Ts, Tbt, nullptr);
  return {V3<double>{F.x.d, F.y.d, F.z.d}, V3<double>{Ts.x.d, Ts.y.d, Ts.z.d},
          V3<double>{Tbt.x.d, Tbt.y.d, Tbt.z.d}};
}
// The column contracted with the bond's cotangent.
__device__ __forceinline__ double bond_contract(const Dev& d, const Adj& a, long k,
                                                const BondColumn& c) {
  const long N = d.n;
  const V3<double> Fb = ldv(a.Fe, N, k) - ldv(a.Fe, N, k + 1);
  const V3<double> Tsb = ldv(a.Te, N, k) + ldv(a.Te, N, k + 1);
  const V3<double> Tbb = ldv(a.Te, N, k) - ldv(a.Te, N, k + 1);
  return (c.F.x * Fb.x + c.F.y * Fb.y + c.F.z * Fb.z) +
         (c.Ts.x * Tsb.x + c.Ts.y * Tsb.y + c.Ts.z * Tsb.z) +
         (c.Tbt.x * Tbb.x + c.Tbt.y * Tbb.y + c.Tbt.z * Tbb.z);
}
// One thread per (input direction, bond).
__device__ __forceinline__ void adj_bond(const Dev& d, const Adj& a, const double* S1, long t) {
  const long N = d.n;
  if (t >= 11 * N) return;
  const int dir = (int)(t / N);
  const long k = t - (long)dir * N;
  if (!(d.bflags[k] & 1)) return;
  a.bvjp[dir * N + k] = bond_contract(d, a, k, bond_column(d, S1, k, dir));
}

// ---------------------------------------------------------------- dipoles
// Squared distance with explicitly rounded operations: the exact selection of
// the contact search and of the dipole cutoff.
__device__ __forceinline__ double r2x(V3<double> p, V3<double> q) {
  double dx = __dsub_rn(p.x, q.x), dy = __dsub_rn(p.y, q.y), dz = __dsub_rn(p.z, q.z);
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}
// Whether pair (i, j) interacts: every pair of a member, or with a cutoff the
// pairs the forward list walk selects.
__device__ __forceinline__ bool dip_pair_on(const Dev& d, V3<double> xi, V3<double> xj) {
  return d.dcut == 0.0 || r2x(xi, xj) < d.dcut * d.dcut;
}

// Gradients of Phi = grad_r U . g + grad_a U . h with respect to r, a and b.
__device__ void phi_grad(V3<double> r, V3<double> am, V3<double> bm, V3<double> g, V3<double> hv,
                         V3<double>& dr, V3<double>& da, V3<double>& db) {
  const double u = rsqrt_pair(dot(r, r));
  const double u2 = u * u, u3 = u2 * u, u5 = u3 * u2, u7 = u5 * u2, u9 = u7 * u2;
  const double A = dot(am, bm), P = dot(am, r), Q = dot(bm, r), G = dot(r, g);
  const double Ga = dot(am, g), Gb = dot(bm, g), Hb = dot(bm, hv), Hr = dot(r, hv);
  const double cr = 15.0 * A * u7 * G - 105.0 * u9 * P * Q * G + 15.0 * u7 * (Q * Ga + P * Gb) -
                    3.0 * u5 * Hb + 15.0 * u7 * Q * Hr;
  const double ca = 15.0 * u7 * Q * G - 3.0 * u5 * Gb;
  const double cb = 15.0 * u7 * P * G - 3.0 * u5 * Ga - 3.0 * u5 * Hr;
  const double cg = -3.0 * A * u5 + 15.0 * u7 * P * Q;
  const double ch = -3.0 * u5 * Q;
  dr = cr * r + ca * am + cb * bm + cg * g + ch * hv;
  da = ca * r - (3.0 * u5 * G) * bm - (3.0 * u5 * Q) * g;
  db = cb * r - (3.0 * u5 * G) * am - (3.0 * u5 * P) * g + u3 * hv;
}

constexpr int ATJ = 256;

// LDS of the fused reverse force kernel: a dipole tile and its reduction, or
// the field-gradient reduction (different workgroups, one union).
union AdjSmem {
  double sj[12][ATJ];
  double red[4][6][64];
  double fred[12][256];
};

__device__ __forceinline__ void adj_dipole_item(const Dev& d, const Adj& a, const double* S1,
                                                const DipWork& wk, AdjSmem& sm) {
  double(*sj)[ATJ] = sm.sj;
  const long N = d.n;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = wk.i0 + lane;
  const bool act = i < wk.i1;
  V3<double> xi{0, 0, 0}, mi{0, 0, 0}, gi{0, 0, 0}, hi{0, 0, 0};
  if (act) {
    xi = ldv(S1, N, i); mi = ldv(d.mu, N, i); gi = ldv(a.Fe, N, i); hi = ldv(a.h, N, i);
  }
  V3<double> xb{0, 0, 0}, mb{0, 0, 0};
  for (int t0 = wk.j0; t0 < wk.j1; t0 += ATJ) {
    const int jn = min(ATJ, wk.j1 - t0);
    if ((int)threadIdx.x < jn) {
      const int j = t0 + threadIdx.x;
      const double* srcs[4] = {S1, d.mu, a.Fe, a.h};
      for (int s = 0; s < 4; ++s)
        for (int c = 0; c < 3; ++c) sj[3 * s + c][threadIdx.x] = srcs[s][c * N + j];
    }
    __syncthreads();
    const int jb = wave * 64, je = min(jb + 64, jn);
    for (int jj = jb; jj < je; ++jj) {
      if (t0 + jj == i) continue;
      const V3<double> xj{sj[0][jj], sj[1][jj], sj[2][jj]};
      if (!dip_pair_on(d, xi, xj)) continue;
      const V3<double> mj{sj[3][jj], sj[4][jj], sj[5][jj]};
      const V3<double> gj{sj[6][jj], sj[7][jj], sj[8][jj]};
      const V3<double> hj{sj[9][jj], sj[10][jj], sj[11][jj]};
      V3<double> dr, da, db;
      phi_grad(xi - xj, mi, mj, gi, hi, dr, da, db);  // i as target
      xb = xb - dr;
      mb = mb - da;
      phi_grad(xj - xi, mj, mi, gj, hj, dr, da, db);  // i as source
      xb = xb + dr;
      mb = mb - db;
    }
    __syncthreads();
  }
  // (the last tile pass ended with a barrier, so the tile may be overwritten)
  const double v6[6] = {xb.x, xb.y, xb.z, mb.x, mb.y, mb.z};
  for (int k = 0; k < 6; ++k) sm.red[wave][k][lane] = v6[k];
  __syncthreads();
  if (wave == 0 && act) {
    double* p = d.dpart + (long)wk.slot * 6 * N;
    for (int k = 0; k < 6; ++k)
      p[k * N + i] = d.C * (((sm.red[0][k][lane] + sm.red[1][k][lane]) + sm.red[2][k][lane]) +
                            sm.red[3][k][lane]);
  }
}

// Small-member layout (as the forward): one wave per target, lanes striding
// over the member's sources, a fixed xor tree across lanes.
__device__ __forceinline__ void adj_dipole_small_item(const Dev& d, const Adj& a, const double* S1,
                                                      const DipWork& wk) {
  const long N = d.n;
  const int lane = threadIdx.x & 63;
  const int i = wk.i0 + (int)(threadIdx.x >> 6);
  if (i >= wk.i1) return;  // the whole wave
  const V3<double> xi = ldv(S1, N, i), mi = ldv(d.mu, N, i), gi = ldv(a.Fe, N, i),
                   hi = ldv(a.h, N, i);
  V3<double> xb{0, 0, 0}, mb{0, 0, 0};
  for (int jb = wk.j0 + lane; jb < wk.j1; jb += 2 * 64) {
    V3<double> xj[2], mj[2], gj[2], hj[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {  // loads first; out-of-range entries read source j0
      const int j = jb + 64 * u < wk.j1 ? jb + 64 * u : wk.j0;
      xj[u] = ldv(S1, N, j); mj[u] = ldv(d.mu, N, j); gj[u] = ldv(a.Fe, N, j); hj[u] = ldv(a.h, N, j);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = jb + 64 * u;
      if (j >= wk.j1) break;
      if (j == i || !dip_pair_on(d, xi, xj[u])) continue;
      V3<double> dr, da, db;
      phi_grad(xi - xj[u], mi, mj[u], gi, hi, dr, da, db);  // i as target
      xb = xb - dr;
      mb = mb - da;
      phi_grad(xj[u] - xi, mj[u], mi, gj[u], hj[u], dr, da, db);  // i as source
      xb = xb + dr;
      mb = mb - db;
    }
  }
  double v6[6] = {xb.x, xb.y, xb.z, mb.x, mb.y, mb.z};
#pragma unroll
  for (int k = 0; k < 6; ++k)
    for (int o = 32; o > 0; o >>= 1) v6[k] += __shfl_xor(v6[k], o);
  if (lane == 0) {
    double* p = d.dpart + (long)wk.slot * 6 * N;
    for (int k = 0; k < 6; ++k) p[k * N + i] = d.C * v6[k];
  }
}

// ---------------------------------------------------------------- contact

// x-bar_i += J(d) (F-bar_i - F-bar_j) over the contacts j of i, with
// J(d) = k [ (r_c/r - 1) I - r_c d d^T / r^3 ], d = x_i - x_j. Same search
// as the forward contact kernel (27 lanes per particle, exact sums).
__device__ __forceinline__ void adj_contact(const Dev& d, const Adj& a, const double* S1, long blk) {
  const long N = d.n;
  const int lane = threadIdx.x & 31;
  const long i = (blk * blockDim.x + threadIdx.x) >> 5;
  const bool pv = i < N;
  const long ii = pv ? i : 0;
  const V3<double> xi = ldv(S1, N, ii);
  const V3<double> gi = ldv(a.Fe, N, ii);
  const int mem = d.mem[ii], rod = d.rod[ii];
  const int mlo = d.mrange[2 * mem], mhi = d.mrange[2 * mem + 1];
  const double rc2 = d.rc * d.rc;
  const int cx = cell_coord(xi.x, d.inv_cell), cy = cell_coord(xi.y, d.inv_cell), cz = cell_coord(xi.z, d.inv_cell);
  const int c = lane < 27 ? lane : 0;
  const unsigned key = cell_hash(cx + c % 3 - 1, cy + (c / 3) % 3 - 1, cz + c / 9 - 1, mem, d.cell_mask);
  bool scan = pv && lane < 27;
  for (int o = 0; o < 26; ++o) {
    unsigned ko = __shfl(key, o, 32);
    if (o < lane && ko == key) scan = false;
  }
  Fix3 sum{};
  auto take = [&](int j, int rj, V3<double> xj) {
    if (j == (int)i || j < mlo || j >= mhi) return;
    if (rj == rod && abs(j - (int)i) <= d.depth) return;
    const double r2 = r2x(xi, xj);
    if (!(r2 < rc2)) return;
    const double r = ::sqrt(r2);
    const V3<double> dd = xi - xj;
    const V3<double> gv = gi - ldv(a.Fe, N, j);
    const double s1 = d.kc * (d.rc / r - 1.0);
    const double s2 = d.kc * d.rc * dot(dd, gv) / (r * r2);
    fix_add(sum, s1 * gv - s2 * dd, d.fix_scale[0], d.flags + FLAG_CONTACT_RANGE);
  };
  const CellTab tab = cell_tab(d, d.step[d.lc]);
  if (scan) {
    const CellSlot* sl = tab.slot + (long)key * CELL_CAP;
    const int nb = min(tab.cnt[key], CELL_CAP);
    for (int s = 0; s < nb; ++s) {
      const CellSlot e = sl[s];
      take((int)(e.tag & 0xffffffffll), (int)(e.tag >> 32), V3<double>{e.x, e.y, e.z});
    }
  }
  if (pv && lane == 27) {
    const int no = min(*tab.ovf_cnt, OVF_CAP);
    for (int o = 0; o < no; ++o) {
      const int j = tab.ovf[o];
      take(j, d.rod[j], ldv(S1, N, j));
    }
  }
  sum = half_sum(sum);
  if (pv && lane == 0) st3(d.cF, N, i, fix_value(sum, d.fix_inv[0]));
}

// ---------------------------------------------------------------- field gradient
__device__ __forceinline__ void adj_field(const Dev& d, const Adj& a, int koff, int mem,
                                          double (*red)[256]) {
  const long long lvl = *a.lbase + koff;
  const int b = d.mrange[2 * mem], e = d.mrange[2 * mem + 1];
  const long N = d.n;
  const long long L = d.field_len;
  const long long row = ((lvl % L) + L) % L;
  double s[12];
  for (int k = 0; k < 12; ++k) s[k] = 0.0;
  for (int i = b + threadIdx.x; i < e; i += blockDim.x)
    for (int k = 0; k < 12; ++k) s[k] += a.fieldc[k * N + i];
  for (int k = 0; k < 12; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int k = 0; k < 12; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 12) a.fieldbar[(row * d.M + mem) * 12 + threadIdx.x] += red[threadIdx.x][0];
}

// ---------------------------------------------------------------- fused launch
// The reverse of the force terms in one launch: dipole work items (either
// layout), bond Jacobian columns, contact, and the per-member field gradient.
// Their outputs are disjoint (slots, per-bond columns, contact x-bar, field
// table), and all read only what the local kernel wrote before.
__global__ __launch_bounds__(256) void k_adj_forces(Dev d, Adj a, const double* S1,
                                                    const DipWork* __restrict__ work, int ndip,
                                                    int nbond, int ncont, int koff) {
  __shared__ AdjSmem sm;
  int b = blockIdx.x;
  if (b < ndip) {
    if (d.dip_small) adj_dipole_small_item(d, a, S1, work[b]);
    else adj_dipole_item(d, a, S1, work[b], sm);
    return;
  }
  b -= ndip;
  if (b < nbond) {
    adj_bond(d, a, S1, (long)b * blockDim.x + threadIdx.x);
    return;
  }
  b -= nbond;
  if (b < ncont) {
    adj_contact(d, a, S1, b);
    return;
  }
  adj_field(d, a, koff, b - ncont, sm.fred);
}

// ---------------------------------------------------------------- gather
// What the gather of a particle reads besides its force terms.
struct GatherIn {
  uint8_t bf;
  int b;
  double minv, Iinv;
  V3<double> cx, xloc, mloc, mb, mbbar, vbar, wbar, wh;
  Q4<double> cq, q1, q0;
};
__device__ __forceinline__ GatherIn adj_gather_in(const Dev& d, const Adj& a, long i,
                                                  const double* S0, const double* S1) {
  const long N = d.n;
  return {d.bflags[i],       d.bc[i],            d.minv[i],          d.Iinv[i],
          ldv(a.cx, N, i),   ldv(a.xloc, N, i),  ldv(a.mloc, N, i),  ldv(d.mb, N, i),
          ldv(a.mbbar, N, i), ldv(a.vbar, N, i), ldv(a.wbar, N, i),  ldv(a.wh, N, i),
          ld4(a.cq, N, i),   ld4(S1 + 6 * N, N, i), ld4(S0 + 6 * N, N, i)};
}

// Assemble x-bar and q-bar of the level, push m-bar through m = q m_body q*,
// then reverse the pre kick (ADJ_STEP: returns the cotangent of S0) or write the
// initial-state gradients (ADJ_PREPARE). bond(dir, which) is column `dir` of the
// particle's bond as its first (0) or second (1) particle; dipoles(xb, mbar) adds
// the dipole terms and contact() is the contact term.
template <class B, class D, class C>
__device__ __forceinline__ Cot adj_gather_of(const Dev& d, const Adj& a, long i, const GatherIn& in,
                                             int mode, const rod_gradients& gx, B&& bond,
                                             D&& dipoles, C&& contact) {
  const long N = d.n;
  V3<double> xb = in.cx + in.xloc;
  Q4<double> qb = in.cq;
  if (in.bf & 1) {  // bond (i, i+1): i is particle 1
    xb = xb - V3<double>{bond(0, 0), bond(1, 0), bond(2, 0)};
    qb = qadd(qb, Q4<double>{bond(3, 0), bond(4, 0), bond(5, 0), bond(6, 0)});
  }
  if (in.bf & 2) {  // bond (i-1, i): i is particle 2
    xb = xb + V3<double>{bond(0, 1), bond(1, 1), bond(2, 1)};
    qb = qadd(qb, Q4<double>{bond(7, 1), bond(8, 1), bond(9, 1), bond(10, 1)});
  }
  V3<double> mbar = in.mloc;
  if (d.dipole_on) dipoles(xb, mbar);
  if (d.contact_on) xb = xb + contact();
  // m = q m_body q*: m_body-bar += q* m-bar q; q-bar += -2 (0, m-bar) q (0, m_body)
  const Q4<double> q1 = in.q1;
  st3(a.mbbar, N, i, in.mbbar + qrot_inv(q1, mbar));
  qb = qadd(qb, qscale(-2.0, qmul(qmul(qv(mbar), q1), qv(in.mb))));
  const V3<double> z{0, 0, 0};
  Cot c{xb, z, z, z, z, {0, 0, 0, 0}};
  if (mode == ADJ_STEP) {
    if (in.b == 0) {
      c.w = in.wbar;
      richardson_vjp(in.q0, in.wh, d.dt, qb, c.q, c.w);
      c.v = in.vbar + d.dt * xb;
      const double h = 0.5 * d.dt;
      c.F = (h * in.minv) * c.v;
      c.T = (h * in.Iinv) * c.w;
    } else if (in.b == 1) {
      c.q = qb;
    }
  } else {
    if (gx.x0) st3(gx.x0, N, i, xb);
    if (gx.v0) st3(gx.v0, N, i, in.b == 0 ? in.vbar : z);
    if (gx.w0) st3(gx.w0, N, i, in.b == 0 ? in.wbar : z);
    if (gx.q0) {
      // q was normalised from the raw input: project out the radial part.
      Q4<double> g{0, 0, 0, 0};
      if (in.b != 2) g = qadd(qb, qscale(-qdot(q1, qb), q1));
      st4(gx.q0, N, i, g);
    }
  }
  return c;
}
__device__ __forceinline__ void store_cot(const Adj& a, long N, long i, const Cot& c) {
  st3(a.cx, N, i, c.x);
  st3(a.cv, N, i, c.v);
  st4(a.cq, N, i, c.q);
  st3(a.cw, N, i, c.w);
  st3(a.cF, N, i, c.F);
  st3(a.cT, N, i, c.T);
}

// The gather with the terms of the separate force launch.
__device__ __forceinline__ void adj_gather(const Dev& d, const Adj& a, long i, const double* S0,
                                           const double* S1, int nslot_max, int mode,
                                           const rod_gradients& gx) {
  const long N = d.n;
  const Cot c = adj_gather_of(
      d, a, i, adj_gather_in(d, a, i, S0, S1), mode, gx,
      [&](int dir, int which) { return a.bvjp[dir * N + i - which]; },
      [&](V3<double>& xb, V3<double>& mbar) {
        const int S = d.mslots[d.mem[i]];
        for (int s = 0; s < S && s < nslot_max; ++s) {
          const double* p = d.dpart + (long)s * 6 * N;
          xb = xb + V3<double>{p[i], p[N + i], p[2 * N + i]};
          mbar = mbar + V3<double>{p[3 * N + i], p[4 * N + i], p[5 * N + i]};
        }
      },
      [&] { return ldv(d.cF, N, i); });
  if (mode == ADJ_STEP) store_cot(a, N, i, c);
}

// Cell list of level lvl is done with: empty it.
__device__ __forceinline__ void clear_cells_of(const Dev& d, long i, long long lvl) {
  if (!d.contact_on) return;
  const CellTab tab = cell_tab(d, lvl);
  if (i == 0) *tab.ovf_cnt = 0;
  if (i < d.n) tab.cnt[d.key[i]] = 0;
}

// One reverse level in one pass per particle, for the state S1 of level
// lbase + koff (view v, whose level counter reads that level):
//  - when S2 (the state one level later) is given, the gather of that later
//    level, which hands over the cotangents of S1 and empties its cell list;
//  - the dipole moment and cell-list entry of S1 (the force evaluation being
//    reversed needs them);
//  - the local VJPs of level koff (kicks, damping, Zeeman, torques).
// Everything a particle reads was written by earlier kernels or by its own
// thread; the cell lists of consecutive levels alternate tables.
__global__ __launch_bounds__(256) void k_adj_level(Dev v, Adj a, const double* S0, const double* S1,
                                                   const double* S2, int koff, int mode,
                                                   int nslot_max) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long N = v.n;
  const long long lvl = v.step[v.lc];
  if (S2) {
    clear_cells_of(v, i, lvl + 1);
    if (i < N) adj_gather(v, a, i, S1, S2, nslot_max, ADJ_STEP, rod_gradients{});
  }
  if (i >= N) return;
  moment_and_cell(v, i, ld4(S1 + 6 * N, N, i), ldv(S1, N, i), ldv(v.mb, N, i), v.mem[i], v.rod[i],
                  lvl);
  adj_local(v, a, i, S0, S1, koff, mode);
}

// The gather of a level on its own (the last of a segment, and the initial
// force evaluation).
__global__ __launch_bounds__(256) void k_adj_gather(Dev v, Adj a, const double* S0, const double* S1,
                                                    int nslot_max, int mode, rod_gradients gx) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  clear_cells_of(v, i, v.step[v.lc]);
  if (i < v.n) adj_gather(v, a, i, S0, S1, nslot_max, mode, gx);
}

// ---------------------------------------------------------------- small systems
// Reverse of a whole step in one launch for systems whose forward steps are single
// launches (k_step.hip): a workgroup owns ADJ_T particles, a wave sums each one's
// dipole and contact terms, one wave evaluates the 11 Jacobian columns of the
// ADJ_T + 1 bonds around them, and one thread per particle then does the gather of
// the level and the local terms of the level before. Those publish what other
// particles need of them (AdjPub) in the set that nobody reads in this launch.
// Against a local and a force launch per level (8.8 and 6.6 us at N = 256, plus the
// gap between them): 18 -> 8.2 us per level (11.5 when the particle threads loaded
// their inputs after the barrier instead of before it).
constexpr int ADJ_T = 4;

// Dipole and contact terms of target i of the member [b, e), by one wave, into
// out[0..6) (x-bar, m-bar before the factor C) and out[6..9) (contact x-bar).
// Contact candidates are marked as in small_target; [xlo, xhi] are excluded.
__device__ __forceinline__ void adj_small_target(const Dev& d, const Adj& a, const double* S1, int i,
                                                 int b, int e, int xlo, int xhi, double* out) {
  constexpr int U = 2;  // rounds in flight
  const long N = d.n;
  const int lane = threadIdx.x & 63;
  const V3<double> xi = ldv(S1, N, i), mi = ldv(d.mu, N, i), gi = ldv(a.Fe, N, i),
                   hi = ldv(a.h, N, i);
  const bool dip = d.dipole_on, con = d.contact_on;
  const double rc2 = d.rc * d.rc;
  const unsigned span = (unsigned)(xhi - xlo);
  V3<double> xb{0, 0, 0}, mb{0, 0, 0};
  Fix3 f{};
  bool hit = false;
  unsigned near = 0;
  int round = 0, base = b;
  for (int j0 = b; j0 < e; j0 += U * 64) {
    V3<double> xj[U], mj[U], gj[U], hj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // loads first; out-of-range entries read the first source
      const int j = j0 + 64 * u + lane < e ? j0 + 64 * u + lane : b;
      xj[u] = ldv(S1, N, j); mj[u] = ldv(d.mu, N, j); gj[u] = ldv(a.Fe, N, j); hj[u] = ldv(a.h, N, j);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 64 * u + lane;
      if (j0 + 64 * u >= e) break;  // the whole wave
      if (con && j < e && r2x(xi, xj[u]) < rc2 && (unsigned)(j - xlo) > span) near |= 1u << (round + u);
      if (!dip || j >= e || j == i) continue;
      V3<double> dr, da, db;
      phi_grad(xi - xj[u], mi, mj[u], gi, hi, dr, da, db);  // i as target
      xb = xb - dr;
      mb = mb - da;
      phi_grad(xj[u] - xi, mj[u], mi, gj[u], hj[u], dr, da, db);  // i as source
      xb = xb + dr;
      mb = mb - db;
    }
    round += U;
    if (con && (round == 32 || j0 + U * 64 >= e)) {
      while (__any(near != 0u)) {
        if (near != 0u) {
          const int j = base + lane + 64 * (__ffs((int)near) - 1);
          near &= near - 1u;
          hit = true;
          const V3<double> xc = ldv(S1, N, j);
          const double r2 = r2x(xi, xc);
          const double r = ::sqrt(r2);
          const V3<double> dd = xi - xc, gv = gi - ldv(a.Fe, N, j);
          const double s1 = d.kc * (d.rc / r - 1.0);
          const double s2 = d.kc * d.rc * dot(dd, gv) / (r * r2);
          fix_add(f, s1 * gv - s2 * dd, d.fix_scale[0], d.flags + FLAG_CONTACT_RANGE);
        }
      }
      round = 0;
      base = j0 + U * 64;
    }
  }
  if (con) {
    V3<double> c{0.0, 0.0, 0.0};
    if (__any(hit)) c = wave_value<64>(f, d.fix_inv[0]);
    if (lane == 0) { out[6] = c.x; out[7] = c.y; out[8] = c.z; }
  }
  if (dip) {
    double v6[6] = {xb.x, xb.y, xb.z, mb.x, mb.y, mb.z};
    wave_sum6(v6, out);
  }
}

// `d` and `a` with what a level publishes in `p` and fieldc.
__device__ __forceinline__ void adj_publish(Dev& d, Adj& a, const AdjPub& p, double* fieldc) {
  d.mu = p.mu;
  a.Fe = p.Fe; a.Te = p.Te; a.h = p.h;
  a.fieldc = fieldc;
}

// The last level of a segment (state S1, the step from S0): its local terms.
__global__ __launch_bounds__(64) void k_adj_open(Dev d, Adj a, AdjPub p, const double* S0,
                                                 const double* S1, int koff, double* fieldc) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  adj_publish(d, a, p, fieldc);
  st3(d.mu, d.n, i, qrot(ld4(S1 + 6 * d.n, d.n, i), ldv(d.mb, d.n, i)));
  adj_local(d, a, i, S0, S1, koff, ADJ_STEP);
}

// Bond Jacobians of `levels` consecutive levels from the state S of the first (their
// states stride apart), one thread per level, column and bond, into
// J[level][column][9][N]. They depend on the recorded states alone, so they are
// taken for many levels at once, at full occupancy, and leave the level-to-level
// chain (N = 256: 23 us for 100 levels; 1.4 us per level inside the step).
__global__ __launch_bounds__(256) void k_adj_jacobians(Dev d, const double* S, long stride, int levels,
                                                       double* J) {
  const long N = d.n;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long col = t / N, k = t - col * N;  // level * 11 + column
  if (col >= 11L * levels || !(d.bflags[k] & 1)) return;
  const int dir = (int)(col % 11);
  const BondColumn c = bond_column(d, S + (col / 11) * stride, k, dir);
  double* o = J + col * 9 * N;
  st3(o, N, k, c.F);
  st3(o + 3 * N, N, k, c.Ts);
  st3(o + 6 * N, N, k, c.Tbt);
}

// Level lbase + koff with state S1 (the step from S0): force terms and gather, then
// (SP set: the state before S0) the local terms of S0's level, published in `next`.
__global__ __launch_bounds__(64 * (ADJ_T + 2)) void k_adj_step(Dev d, Adj a, AdjPub now, AdjPub next,
                                                               const double* SP, const double* S0,
                                                               const double* S1, const double* J,
                                                               int koff, double* fieldc) {
  __shared__ double sums[ADJ_T][10];
  __shared__ double cols[11][ADJ_T + 1];
  const long N = d.n;
  const int i0 = blockIdx.x * ADJ_T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wave < ADJ_T) {
    adj_publish(d, a, now, nullptr);
    const int i = i0 + wave;
    if (i < N) {
      int b = 0, e = (int)N, xlo, xhi;
      if (d.M > 1) {
        const int m = d.mem[i];
        b = d.mrange[2 * m];
        e = d.mrange[2 * m + 1];
      }
      excluded_range(d, i, xlo, xhi);
      adj_small_target(d, a, S1, i, b, e, xlo, xhi, sums[wave]);
    }
    __syncthreads();
    return;
  }
  if (wave == ADJ_T) {  // bonds i0 - 1 .. i0 + ADJ_T - 1, a lane per column
    adj_publish(d, a, now, nullptr);
    const int dir = lane / (ADJ_T + 1), u = lane - dir * (ADJ_T + 1);
    const long k = i0 - 1 + u;
    if (dir < 11 && k >= 0 && k < N && (d.bflags[k] & 1)) {
      const double* o = J + dir * 9 * N;
      cols[dir][u] = bond_contract(d, a, k, BondColumn{ld3(o, N, k), ld3(o + 3 * N, N, k), ld3(o + 6 * N, N, k)});
    }
    __syncthreads();
    return;
  }
  const bool valid = lane < ADJ_T && i0 + lane < N;
  const long i = valid ? i0 + lane : i0;
  adj_publish(d, a, next, fieldc);
  const GatherIn in = adj_gather_in(d, a, i, S0, S1);
  LocalIn loc{};
  if (SP) loc = adj_local_in(d, i, SP, S0, *a.lbase + koff - 1);
  __syncthreads();
  if (!valid) return;
  const double* u = sums[lane];
  const Cot c = adj_gather_of(
      d, a, i, in, ADJ_STEP, rod_gradients{},
      [&](int dir, int which) { return cols[dir][lane + 1 - which]; },
      [&](V3<double>& xb, V3<double>& mbar) {
        xb = xb + d.C * V3<double>{u[0], u[1], u[2]};
        mbar = mbar + d.C * V3<double>{u[3], u[4], u[5]};
      },
      [&] { return V3<double>{u[6], u[7], u[8]}; });
  store_cot(a, N, i, c);
  if (SP) {
    const V3<double> m = qrot(in.q0, in.mb);
    st3(d.mu, N, i, m);
    adj_local_of(d, a, i, loc, m, c, ADJ_STEP);
  }
}
static_assert(11 * (ADJ_T + 1) <= 64, "a lane per bond column");

// Field gradient of a segment of len levels: the member sums of every level (a workgroup
// each, levels past the grid's height in turn), then their addition to the table's rows,
// latest level first.
__global__ __launch_bounds__(256) void k_adj_field_sums(Dev d, const double* fieldc, double* part,
                                                        int len) {
  __shared__ double red[12][256];
  const int mem = blockIdx.x;
  const int b = d.mrange[2 * mem], e = d.mrange[2 * mem + 1];
  const long N = d.n;
  for (long koff = 1 + blockIdx.y; koff <= len; koff += gridDim.y) {
    const double* f = fieldc + koff * 12 * N;
    double s[12];
    for (int k = 0; k < 12; ++k) s[k] = 0.0;
    for (int i = b + threadIdx.x; i < e; i += blockDim.x)
      for (int k = 0; k < 12; ++k) s[k] += f[k * N + i];
    for (int k = 0; k < 12; ++k) red[k][threadIdx.x] = s[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w)
        for (int k = 0; k < 12; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x < 12) part[(koff * d.M + mem) * 12 + threadIdx.x] = red[threadIdx.x][0];
    __syncthreads();
  }
}
__global__ __launch_bounds__(64) void k_adj_field_rows(Dev d, Adj a, const double* __restrict__ part,
                                                       double* __restrict__ bar, int len) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 12 * d.M) return;
  const long long L = d.field_len;
  const long long base = *a.lbase;
  long long at = -1;  // the row being added to
  double sum = 0.0;
#pragma unroll 8
  for (int koff = len; koff > 0; --koff) {
    const double p = part[(long)koff * d.M * 12 + t];
    const long long lvl = base + koff, row = ((lvl % L) + L) % L;
    if (row != at) {
      if (at >= 0) bar[at * d.M * 12 + t] = sum;
      at = row;
      sum = bar[at * d.M * 12 + t];
    }
    sum += p;
  }
  if (at >= 0) bar[at * d.M * 12 + t] = sum;
}

__global__ void k_set_level(long long* p, long long v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { p[0] = v; p[1] = v; }
}
// First level of the segment, and the counters of the reverse views.
__global__ void k_set_base(long long* p, long long* levels, int nlev, long long v) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k == 0) p[0] = v;
  if (k < nlev) levels[3 * k] = levels[3 * k + 1] = levels[3 * k + 2] = v + k;
}

// ---------------------------------------------------------------- host side
template <class T>
static int adalloc(std::vector<void*>& allocs, T** p, size_t count) {
  void* q = nullptr;
  size_t bytes = std::max<size_t>(count * sizeof(T), 16);
  if (hipMalloc(&q, bytes) != hipSuccess) return rodmx_fail(ROD_E_HIP, "tape allocation failed");
  allocs.push_back(q);
  if (hipMemset(q, 0, bytes) != hipSuccess) return rodmx_fail(ROD_E_HIP, "tape memset failed");
  *p = (T*)q;
  return ROD_OK;
}

#define ACHK(expr)                                                                   \
  do {                                                                               \
    hipError_t _e = (expr);                                                          \
    if (_e != hipSuccess) return rodmx_fail(ROD_E_HIP, hipGetErrorString(_e));       \
  } while (0)
#define ATRY(expr)                   \
  do {                               \
    int _r = (expr);                 \
    if (_r != ROD_OK) return _r;     \
  } while (0)

int tape_init(Tape& t, const Dev& d, int every, int capacity, std::vector<void*>& allocs) {
  t.every = every;
  t.capacity = capacity;
  t.allocs = &allocs;
  if (capacity <= 0) return ROD_OK;
  const size_t N = d.n;
  const size_t nck = (size_t)capacity / every + 1;
  Adj& a = t.a;
  double* cot = nullptr;
  ATRY(adalloc(allocs, &t.ckpt, nck * STATE_PLANES * N));
  ATRY(adalloc(allocs, &t.seg, (size_t)(every + 1) * SEG_PLANES * N));
  ATRY(adalloc(allocs, &cot, STATE_PLANES * N));
  a.cx = cot; a.cv = cot + 3 * N; a.cq = cot + 6 * N; a.cw = cot + 10 * N;
  a.cF = cot + 13 * N; a.cT = cot + 16 * N;
  ATRY(adalloc(allocs, &a.Fe, 3 * N));
  ATRY(adalloc(allocs, &a.Te, 3 * N));
  ATRY(adalloc(allocs, &a.h, 3 * N));
  ATRY(adalloc(allocs, &a.mloc, 3 * N));
  ATRY(adalloc(allocs, &a.xloc, 3 * N));
  ATRY(adalloc(allocs, &a.vbar, 3 * N));
  ATRY(adalloc(allocs, &a.wbar, 3 * N));
  ATRY(adalloc(allocs, &a.wh, 3 * N));
  ATRY(adalloc(allocs, &a.fieldc, 12 * N));
  ATRY(adalloc(allocs, &a.bvjp, 11 * N));
  ATRY(adalloc(allocs, &a.mbbar, 3 * N));
  ATRY(adalloc(allocs, &a.fieldbar, (size_t)d.field_len * d.M * 12));
  ATRY(adalloc(allocs, &a.scratch, 6 * N));
  ATRY(adalloc(allocs, &a.level, 3));
  ATRY(adalloc(allocs, &a.lbase, 1));
  ATRY(adalloc(allocs, &a.levels, 3 * (size_t)(every + 1)));
  return ROD_OK;
}

// Copy the caller's state into a recorded-state slot (STATE_PLANES N).
static int save_state(const Dev& d, double* dst, hipStream_t s) {
  const size_t N = d.n, b3 = 3 * N * sizeof(double);
  ACHK(hipMemcpyAsync(dst, d.x, b3, hipMemcpyDeviceToDevice, s));
  ACHK(hipMemcpyAsync(dst + 3 * N, d.v, b3, hipMemcpyDeviceToDevice, s));
  ACHK(hipMemcpyAsync(dst + 6 * N, d.q, 4 * N * sizeof(double), hipMemcpyDeviceToDevice, s));
  ACHK(hipMemcpyAsync(dst + 10 * N, d.w, b3, hipMemcpyDeviceToDevice, s));
  ACHK(hipMemcpyAsync(dst + 13 * N, d.F, b3, hipMemcpyDeviceToDevice, s));
  ACHK(hipMemcpyAsync(dst + 16 * N, d.T, b3, hipMemcpyDeviceToDevice, s));
  return ROD_OK;
}

int tape_start(Tape& t, const Dev& d, hipStream_t s, int64_t step) {
  t.active = true;
  t.start_step = step;
  return save_state(d, t.ckpt, s);
}

int tape_before_step(Tape& t, const Dev& d, hipStream_t s, int64_t step) {
  const int64_t k = step - t.start_step;
  if (k >= t.capacity)
    return rodmx_fail(ROD_E_STATE, "tape capacity exceeded: raise tape_capacity or call rod_tape_begin");
  if (k > 0 && k % t.every == 0) return save_state(d, t.ckpt + (size_t)(k / t.every) * STATE_PLANES * d.n, s);
  return ROD_OK;
}

// A view of the device context whose state lives in a recorded-state slot.
static Dev view(const Dev& d, double* S, long long* level) {
  Dev v = d;
  const long N = d.n;
  v.x = S; v.v = S + 3 * N; v.q = S + 6 * N; v.w = S + 10 * N; v.F = S + 13 * N; v.T = S + 16 * N;
  v.step = level;
  return v;
}

static inline unsigned nblk(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Reverse the force evaluation of state S1 (level lbase + koff) and, in
// ADJ_STEP mode, the kicks of the step from S0: one per-particle pass (which
// first completes the later level S2 when given) and one launch for the force
// terms. The gather of S1's own level is left to the next call or to
// reverse_gather. Only device-side values vary between segments, so a full
// segment can be captured once and replayed.
static int reverse_level(Tape& t, const Dev& d, const DipWork* work, int nwork, int max_slots,
                         hipStream_t s, const double* S0, double* S1, const double* S2, int koff,
                         int mode) {
  const long N = d.n;
  Adj& a = t.a;
  Dev v = view(d, S1, a.levels + 3 * koff);
  hipLaunchKernelGGL(k_adj_level, dim3(nblk(N, 256)), dim3(256), 0, s, v, a, S0,
                     (const double*)S1, S2, koff, mode, max_slots);
  ACHK(hipGetLastError());
  const int ndip = d.dipole_on ? nwork : 0;
  const int nbond = (int)nblk(11 * N, 256);
  const int ncont = d.contact_on ? (int)nblk(32 * N, 256) : 0;
  hipLaunchKernelGGL(k_adj_forces, dim3(ndip + nbond + ncont + d.M), dim3(256), 0, s, v, a,
                     (const double*)S1, work, ndip, nbond, ncont, koff);
  ACHK(hipGetLastError());
  return ROD_OK;
}

// The gather of level lbase + koff on its own.
static int reverse_gather(Tape& t, const Dev& d, int max_slots, hipStream_t s, const double* S0,
                          double* S1, int koff, int mode, const rod_gradients& gx) {
  Adj& a = t.a;
  Dev v = view(d, S1, a.levels + 3 * koff);
  hipLaunchKernelGGL(k_adj_gather, dim3(nblk(d.n, 256)), dim3(256), 0, s, v, a, S0,
                     (const double*)S1, max_slots, mode, gx);
  ACHK(hipGetLastError());
  return ROD_OK;
}

// Recompute steps 0..len-1 of a segment from seg[0] (levels from the view's
// counters), with the forward's fused chain: pre, forces, then (kick, forces)
// per further step, and post. Each level's state goes to its own slot; the
// kick closes slot k (full-step v and w, forces, dipole field) and writes the
// advanced state into slot k + 1.
static int recompute(Tape& t, const Dev& d, int precision, const DipWork* work, int nwork,
                     const TapeSmall& small, hipStream_t s, int len) {
  const long N = d.n;
  const size_t SP = SEG_PLANES * (size_t)N;
  Dev v = view(d, t.seg + SP, t.a.level);
  if (small.mu) {  // the fused steps: level k reads its slot and writes the next
    v.src = t.seg;
    v.lazy_cells = 1;
    v.far_ok = 0;
    ACHK(launch_pre(v, PRE_STEP, s));
    for (int k = 1; k <= len; ++k) {
      double* Sk = t.seg + k * SP;
      Dev w = view(d, Sk, t.a.level);
      w.lc = k & 1 ? 1 : 2;
      double* mu[2] = {d.mu, small.mu};
      float* muf[2] = {d.muf, small.muf};
      w.mu = mu[(k + 1) & 1]; w.muf = muf[(k + 1) & 1];
      const StepOut o{Sk + SP, Sk + SP + 3 * N, Sk + SP + 6 * N, Sk + SP + 10 * N,
                      mu[k & 1], muf[k & 1], Sk + 19 * N, k == len, 1};
      ACHK(launch_step(w, precision, o, s));
    }
    return ROD_OK;
  }
  v.src = t.seg;  // the pre kernel reads step 0 and writes step 1
  ACHK(launch_pre(v, PRE_STEP, s));
  v.src = nullptr;
  ACHK(launch_force_pass(v, precision, work, nwork, 1, s));
  for (int k = 1; k < len; ++k) {
    double* Sk = t.seg + k * SP;
    v.nx = Sk + SP;
    ACHK(launch_kick(v, Sk + 19 * N, s));
    Dev w = view(d, Sk + SP, t.a.level);
    w.lc = 3 - v.lc;
    v = w;
    ACHK(launch_force_pass(v, precision, work, nwork, 1, s));
  }
  ACHK(launch_post(v, POST_KICK, ROD_TERM_ALL, nullptr, nullptr, t.seg + len * SP + 19 * N, s));
  return ROD_OK;
}

static int reverse_segment(Tape& t, const Dev& d, const DipWork* work, int nwork, int max_slots,
                           hipStream_t s, int len) {
  const size_t SP = SEG_PLANES * (size_t)d.n;
  for (int k = len - 1; k >= 0; --k) {
    double* Sk = t.seg + k * SP;
    const double* S2 = k + 1 < len ? Sk + 2 * SP : nullptr;
    ATRY(reverse_level(t, d, work, nwork, max_slots, s, Sk, Sk + SP, S2, k + 1, ADJ_STEP));
  }
  return reverse_gather(t, d, max_slots, s, t.seg, t.seg + SP, 1, ADJ_STEP, rod_gradients{});
}

// The same by the fused reverse steps of small systems.
static int reverse_small(Tape& t, const Dev& d, hipStream_t s, int len) {
  const long N = d.n;
  const size_t SP = SEG_PLANES * (size_t)N;
  const Adj& a = t.a;
  const AdjPub sets[2] = {{a.Fe, a.Te, a.h, d.mu},
                          {t.pub, t.pub + 3 * N, t.pub + 6 * N, t.pub + 9 * N}};
  const int chunk = t.jac_levels;
  double* S = t.seg + len * SP;
  hipLaunchKernelGGL(k_adj_open, dim3(nblk(N, 64)), dim3(64), 0, s, d, a, sets[len & 1],
                     (const double*)(S - SP), (const double*)S, len, t.fieldc + (size_t)len * 12 * N);
  ACHK(hipGetLastError());
  for (int k = len, first = len + 1; k >= 1; --k, S -= SP) {
    if (k < first) {  // Jacobians of the levels [first, k]
      first = std::max(1, k - chunk + 1);
      const int m = k - first + 1;
      hipLaunchKernelGGL(k_adj_jacobians, dim3(nblk(11L * m * N, 256)), dim3(256), 0, s, d,
                         (const double*)(t.seg + first * SP), (long)SP, m, t.jac);
      ACHK(hipGetLastError());
    }
    hipLaunchKernelGGL(k_adj_step, dim3(nblk(N, ADJ_T)), dim3(64 * (ADJ_T + 2)), 0, s, d, a,
                       sets[k & 1], sets[1 - (k & 1)], k > 1 ? (const double*)(S - 2 * SP) : nullptr,
                       (const double*)(S - SP), (const double*)S,
                       (const double*)(t.jac + (size_t)(k - first) * 99 * N), k,
                       t.fieldc + (size_t)(k - 1) * 12 * N);
    ACHK(hipGetLastError());
  }
  // (a grid is at most 65,535 high; 16,384 workgroups fill the chip many times over)
  hipLaunchKernelGGL(k_adj_field_sums, dim3(d.M, std::min(len, 16384)), dim3(256), 0, s, d,
                     (const double*)t.fieldc, t.fieldp, len);
  ACHK(hipGetLastError());
  hipLaunchKernelGGL(k_adj_field_rows, dim3(nblk(12 * d.M, 64)), dim3(64), 0, s, d, a,
                     (const double*)t.fieldp, a.fieldbar, len);
  ACHK(hipGetLastError());
  return ROD_OK;
}

template <class F>
static int capture(hipStream_t s, hipGraphExec_t* out, F body) {
  hipGraph_t g = nullptr;
  ACHK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  int rc = body();
  hipError_t e = hipStreamEndCapture(s, &g);
  if (rc != ROD_OK) { if (g) (void)hipGraphDestroy(g); return rc; }
  ACHK(e);
  e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  ACHK(e);
  return ROD_OK;
}

void tape_release(Tape& t) {
  if (t.g_recompute) (void)hipGraphExecDestroy(t.g_recompute);
  if (t.g_reverse) (void)hipGraphExecDestroy(t.g_reverse);
  t.g_recompute = t.g_reverse = nullptr;
}

// The buffers of the fused reverse steps, at their first use; false where they do not fit
// in memory (they add up to 55% to a tape: the reverse then takes two launches per step).
static bool fused_buffers(Tape& t, const Dev& d) {
  if (t.pub) return true;
  const size_t N = d.n, levels = (size_t)t.every + 1;
  // Jacobians of as many levels as fit in 128 MiB (at least one)
  const size_t jl = std::max<size_t>(1, std::min<size_t>(t.every, (128u << 20) / (99 * sizeof(double) * N)));
  const size_t count = 12 * levels * (N + d.M) + 99 * jl * N + 12 * N;
  void* q = nullptr;
  if (hipMalloc(&q, count * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  t.allocs->push_back(q);
  t.fieldc = (double*)q;
  t.fieldp = t.fieldc + 12 * levels * N;
  t.jac = t.fieldp + 12 * levels * d.M;
  t.jac_levels = (int)jl;
  t.pub = t.jac + 99 * jl * N;
  return true;
}

int adjoint_run(Tape& t, const Dev& d, int precision, const DipWork* work, int nwork,
                int max_slots, const TapeSmall& small, hipStream_t s, int64_t end_step,
                const rod_cotangent* gy, rod_gradients* gx) {
  const long N = d.n;
  const int64_t T = end_step - t.start_step;
  if (T <= 0) return rodmx_fail(ROD_E_NOTAPE, "no recorded steps");
  Adj& a = t.a;
  const size_t b3 = 3 * N * sizeof(double);
  ACHK(hipMemsetAsync(a.cx, 0, STATE_PLANES * N * sizeof(double), s));
  if (gy->x) ACHK(hipMemcpyAsync(a.cx, gy->x, b3, hipMemcpyDeviceToDevice, s));
  if (gy->v) ACHK(hipMemcpyAsync(a.cv, gy->v, b3, hipMemcpyDeviceToDevice, s));
  if (gy->q) ACHK(hipMemcpyAsync(a.cq, gy->q, 4 * N * sizeof(double), hipMemcpyDeviceToDevice, s));
  if (gy->w) ACHK(hipMemcpyAsync(a.cw, gy->w, b3, hipMemcpyDeviceToDevice, s));
  ACHK(hipMemsetAsync(a.mbbar, 0, b3, s));
  ACHK(hipMemsetAsync(a.fieldbar, 0, (size_t)d.field_len * d.M * 12 * sizeof(double), s));
  const bool fused_reverse = small.reverse && fused_buffers(t, d);
  auto redo = [&](int len, int64_t s0) -> int {
    if (!small.many) return recompute(t, d, precision, work, nwork, small, s, len);
    Dev v = view(d, t.seg, a.level);
    ACHK(launch_steps(v, precision, small.many, s0, len, s, t.seg, SEG_PLANES * N));
    return ROD_OK;
  };
  auto undo = [&](int len) {
    return fused_reverse ? reverse_small(t, d, s, len)
                    : reverse_segment(t, d, work, nwork, max_slots, s, len);
  };
  const int64_t nseg = (T + t.every - 1) / t.every;
  for (int64_t sg = nseg - 1; sg >= 0; --sg) {
    const int64_t s0 = t.start_step + sg * t.every;
    const int len = (int)std::min<int64_t>(t.every, T - sg * t.every);
    // recompute the segment from its checkpoint with the forward kernels
    ACHK(hipMemcpyAsync(t.seg, t.ckpt + (size_t)sg * STATE_PLANES * N,
                        STATE_PLANES * N * sizeof(double), hipMemcpyDeviceToDevice, s));
    hipLaunchKernelGGL(k_set_level, dim3(1), dim3(1), 0, s, a.level, (long long)s0);
    ACHK(hipGetLastError());
    hipLaunchKernelGGL(k_set_base, dim3(nblk(t.every + 1, 256)), dim3(256), 0, s, a.lbase,
                       a.levels, t.every + 1, (long long)s0);
    ACHK(hipGetLastError());
    if (len == t.every) {
      // (a many-steps launch takes its level as an argument and is not captured)
      if (!t.g_recompute && !small.many)
        ATRY(capture(s, &t.g_recompute, [&] { return redo(len, s0); }));
      if (!t.g_reverse) ATRY(capture(s, &t.g_reverse, [&] { return undo(len); }));
      if (small.many) ATRY(redo(len, s0));
      else ACHK(hipGraphLaunch(t.g_recompute, s));
      ACHK(hipGraphLaunch(t.g_reverse, s));
    } else {
      ATRY(redo(len, s0));
      ATRY(undo(len));
    }
  }
  // the initial force evaluation: dipole field of the start state, then its reverse
  {
    double* S = t.seg;
    ACHK(hipMemcpyAsync(S, t.ckpt, STATE_PLANES * N * sizeof(double), hipMemcpyDeviceToDevice, s));
    hipLaunchKernelGGL(k_set_level, dim3(1), dim3(1), 0, s, a.level, (long long)t.start_step);
    ACHK(hipGetLastError());
    hipLaunchKernelGGL(k_set_base, dim3(nblk(t.every + 1, 256)), dim3(256), 0, s, a.lbase,
                       a.levels, t.every + 1, (long long)t.start_step);
    ACHK(hipGetLastError());
    Dev v = view(d, S, a.level);
    ACHK(launch_pre(v, PRE_EVAL, s));
    ACHK(launch_force_pass(v, precision, work, nwork, 1, s));
    ACHK(launch_post(v, POST_EVAL, ROD_TERM_ALL, a.scratch, a.scratch + 3 * N, S + 19 * N, s));
    ATRY(reverse_level(t, d, work, nwork, max_slots, s, S, S, nullptr, 0, ADJ_PREPARE));
    ATRY(reverse_gather(t, d, max_slots, s, S, S, 0, ADJ_PREPARE, *gx));
  }
  if (gx->m_body) ACHK(hipMemcpyAsync(gx->m_body, a.mbbar, b3, hipMemcpyDeviceToDevice, s));
  if (gx->field)
    ACHK(hipMemcpyAsync(gx->field, a.fieldbar, (size_t)d.field_len * d.M * 12 * sizeof(double),
                        hipMemcpyDeviceToDevice, s));
  return ROD_OK;
}

}  // namespace rodmx
