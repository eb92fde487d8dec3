// Bonds, gather, second half-kick and the next step's half-kick, drift and rotation
// of large systems in one pass over the particles.
//
// The pass is bound by HBM. As two kernels (bond, kick) a step moved 165 B per bond
// and 506 B per particle; here the bond's results never leave the workgroup, and
// what no later kernel of the chain reads is not written (the forces of a step that
// is not the call's last, moments that only the all-pairs sum needs, cell-list
// entries between rebuilds): 182 B in, 104 B out per particle (64 more with the
// record of the dipole cutoff). Masses, inertias and the member come from a table by
// rod, which neighbours share, and the bond's reference length from its vector: 44 B
// less than from arrays by particle. 1.05M particles, mixed: 35 + 117 us per step as
// two kernels, 75 fused, 67 with the table (4.5 TB/s of these bytes; 5.1 of the 328 B per
// particle that the counters show, the rate of a plain copy).
//
// A bond needs both its particles at the level being closed, while the pass
// overwrites them with the next level. Inside a workgroup they pass through LDS;
// across workgroups through the halo: every kernel that sets positions also stores
// the first and last particle of each block of BK_OWN particles, by level parity.
// Thread t owns particle t - 1 of its block and evaluates the bond after it; thread
// 0 evaluates the block's first bond a second time (one bond in 256, against an
// exchange of results that would need a launch).
#include "rod.h"
#include "bond_core.h"
#include "particle_body.h"
#include "integrate_body.h"  // last: contraction within expressions from here on

namespace rodmx {

// The reference length of a bond as the host computes it for the other kernels:
// products and sums rounded one by one.
__device__ __forceinline__ double bond_length(V3<double> r) {
#pragma clang fp contract(off)
  return ::sqrt(r.x * r.x + r.y * r.y + r.z * r.z);
}

static_assert(BK_OWN == 255, "one thread of 256 evaluates the bond before the block");

template <class R, bool HM, bool DAMP>
__global__ __launch_bounds__(256) void k_bond_kick(Dev d, int last) {
  constexpr int C = DAMP ? 10 : 7;  // x, q (and v) of a particle; then the bond's nine
  __shared__ double sh[(DAMP ? 10 : 9) * 256];
  const long N = d.n;
  const int t = threadIdx.x;
  const long blk = blockIdx.x, nblk = gridDim.x;
  const long i = blk * BK_OWN + t - 1;
  const bool own = t > 0 && i < N, any = i >= 0 && i < N;
  const long ii = any ? i : 0;
  const long long L = d.step[d.lc];
  PIn p = {};
  double nb[10];  // the particle after the block's last
  if (any && t > 0) {
    p.x = ld3(d.x, N, ii);
    p.v = ld3(d.v, N, ii);
    p.q = ld4(d.q, N, ii);
    p.w = ld3(d.w, N, ii);
  }
  if ((t == 0 && blk > 0) || (t == 255 && blk + 1 < nblk)) {
    const double* h = d.halo + (((L & 1) * nblk + (t == 0 ? blk - 1 : blk + 1)) * 2 + (t == 0 ? 1 : 0)) * 10;
#pragma unroll
    for (int c = 0; c < 10; ++c) nb[c] = h[c];
    if (t == 0) {
      p.x = V3<double>{nb[0], nb[1], nb[2]};
      p.q = Q4<double>{nb[3], nb[4], nb[5], nb[6]};
      p.v = V3<double>{nb[7], nb[8], nb[9]};
    }
  }
  const uint8_t flags = any ? d.bflags[ii] : 0;
  const int rod = d.rod[ii];
  const V3<double> rref{d.bref[ii], d.bref[N + ii], d.bref[2 * N + ii]};
  const double r0 = bond_length(rref);
  p.mb = ld3(d.mb, N, ii);
  p.b = d.bc[ii];
  p.minv = d.rodI[4 * (long)rod];
  p.Iinv = d.rodI[4 * (long)rod + 1];
  const double mass = d.rodI[4 * (long)rod + 2], inertia = d.rodI[4 * (long)rod + 3];
  p.mem = d.rod_mem[rod];
  const V3<double> cF = d.contact_on ? ld3(d.cF, N, ii) : V3<double>{0.0, 0.0, 0.0};
  V3<double> cT{0.0, 0.0, 0.0}, Fd{0.0, 0.0, 0.0}, Bd{0.0, 0.0, 0.0};
  if constexpr (HM) cT = ld3(d.cT, N, ii);
  if (d.dipole_on) {  // the cutoff walk's slot
    Fd = ld3(d.dpart, N, ii);
    Bd = ld3(d.dpart + 3 * N, N, ii);
  }
  double hprev[5];
  if constexpr (DAMP) {
    const double* hp = d.hist + (long)((L - 1) & 1) * 5 * N;
#pragma unroll
    for (int c = 0; c < 5; ++c) hprev[c] = hp[c * N + ii];
  }
  st3(sh, 256, (long)t, p.x);
  st4(sh + 3 * 256, 256, (long)t, p.q);
  if constexpr (DAMP) st3(sh + 7 * 256, 256, (long)t, p.v);
  __syncthreads();
  V3<double> bF{0.0, 0.0, 0.0}, bTs{0.0, 0.0, 0.0}, bTb{0.0, 0.0, 0.0};
  if (flags & 1) {
    if (t < 255) {
#pragma unroll
      for (int c = 0; c < C; ++c) nb[c] = sh[c * 256 + t + 1];
    }
    const V3<double> x2{nb[0], nb[1], nb[2]};
    const Q4<double> q2{nb[3], nb[4], nb[5], nb[6]};
    if constexpr (DAMP) {
      BondDamp dm;
      dm.gr = d.bdamp[4 * rod]; dm.gs = d.bdamp[4 * rod + 1];
      dm.gt = d.bdamp[4 * rod + 2]; dm.gb = d.bdamp[4 * rod + 3];
      for (int c = 0; c < 5; ++c) dm.hprev[c] = hprev[c];
      dm.rates = L >= d.hist_from;
      dm.dv = V3<double>{nb[7], nb[8], nb[9]} - p.v;
      dm.idt = 1.0 / d.dt;
      bond_one<double, R, true>(p.x, x2, p.q, q2, rref, r0, d.rodK + 4 * rod, bF, bTs, bTb, nullptr, &dm);
      if (own) {
        double* hn = d.hist + (long)(L & 1) * 5 * N;
        for (int c = 0; c < 5; ++c) hn[c * N + i] = dm.hnow[c];
      }
    } else {
      bond_one<double, R>(p.x, x2, p.q, q2, rref, r0, d.rodK + 4 * rod, bF, bTs, bTb, nullptr);
    }
  }
  __syncthreads();
  st3(sh, 256, (long)t, bF);
  st3(sh + 3 * 256, 256, (long)t, bTs);
  st3(sh + 6 * 256, 256, (long)t, bTb);
  __syncthreads();
  if (blk == 0 && t == 0) {
    if (last) d.step[0] = L;
    else d.step[3 - d.lc] = L + 1;
    if (d.use_lists) {  // (the launches that read these are over)
      d.rebuild[d.lc & 1] = 0u;
      d.rebuild[3] = 0u;  // (and every list is the chain's)
      d.cell_dirty[(d.lc & 1) ^ 1] = 0;
    }
  }
  if (!own) return;
  const Bonds bd{bF, bTs, bTb, ld3(sh, 256, (long)t - 1), ld3(sh + 3 * 256, 256, (long)t - 1),
                 ld3(sh + 6 * 256, 256, (long)t - 1), flags};
  p.m = qrot(p.q, p.mb);
  V3<double> F, T;
  gather_sum<HM>(d, i, ROD_TERM_ALL, field_row(d, L, p.mem), p, bd, mass, inertia, Fd, Bd, cF, cT, F, T);
  kick(d, i, F, T, p, last, last);
  if (last) {
    if (d.contact_on && d.use_lists && d.cell_dirty[d.lc & 1] != 0) {  // leave the cell list empty
      const CellTab tab = cell_tab(d, L);
      tab.cnt[d.key[i]] = 0;
      if (i == 0) *tab.ovf_cnt = 0;
    }
    return;
  }
  advance(d, i, p.b, L + 1, p.x, p.v, p.q, p.w, F, T, p.minv, p.Iinv, false, (d.lc & 1) ^ 1);
  halo_store(d, i, L + 1, p.x, p.q, p.v);
  if (d.xm) xm_store(d, i, p.x, qrot(p.q, p.mb));
}

template <class R, bool HM>
static void variant(const Dev& d, int last, hipStream_t s, const hipEvent_t* ev) {
  const dim3 g((unsigned)((d.n + BK_OWN - 1) / BK_OWN)), b(256);
  if (d.bdamp) launch_k(ev, k_bond_kick<R, HM, true>, g, b, s, d, last);
  else launch_k(ev, k_bond_kick<R, HM, false>, g, b, s, d, last);
}

hipError_t launch_bond_kick(const Dev& d, int precision, int last, hipStream_t s, const hipEvent_t* ev) {
  if (precision == 1) {
    if (d.hm) variant<float, true>(d, last, s, ev);
    else variant<float, false>(d, last, s, ev);
  } else {
    if (d.hm) variant<double, true>(d, last, s, ev);
    else variant<double, false>(d, last, s, ev);
  }
  return hipGetLastError();
}

}  // namespace rodmx
