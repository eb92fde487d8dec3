// Forces of small systems (members in the small-member dipole layout), one wave
// per target particle: the dipole sum over the member and, from the same pass
// over its particles, the contact candidates.
#pragma once
#include "contact_body.h"
#include "dipole_body.h"

namespace rodmx {

// ---- sum of ten FP64 values over the 64 lanes of a wave
// The tree is that of the xor butterfly lane ^ 32, 16, 8, 4, 2, 1 (every value
// is the same sum of the same pairs), but the first two levels halve the values
// a lane carries: v_permlane32_swap exchanges the upper half of one register
// with the lower half of another, so one swap and one addition serve two
// values, and v_permlane16_swap likewise within the halves; the levels inside a
// row of 16 lanes are DPP moves. 68 vector instructions and no LDS traffic,
// against 180 (120 of them ds_bpermute) for a butterfly per value.
__device__ __forceinline__ void swap32(double& a, double& b) {
  const unsigned long long ua = __builtin_bit_cast(unsigned long long, a),
                           ub = __builtin_bit_cast(unsigned long long, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  a = __builtin_bit_cast(double, (unsigned long long)lo[0] | ((unsigned long long)hi[0] << 32));
  b = __builtin_bit_cast(double, (unsigned long long)lo[1] | ((unsigned long long)hi[1] << 32));
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  const unsigned long long ua = __builtin_bit_cast(unsigned long long, a),
                           ub = __builtin_bit_cast(unsigned long long, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  a = __builtin_bit_cast(double, (unsigned long long)lo[0] | ((unsigned long long)hi[0] << 32));
  b = __builtin_bit_cast(double, (unsigned long long)lo[1] | ((unsigned long long)hi[1] << 32));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double a) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, a);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}
constexpr int DPP_XOR1 = 0xb1, DPP_XOR2 = 0x4e, DPP_XOR3 = 0x1b;  // quad permutations
constexpr int DPP_ROR8 = 0x128;                                  // lane ^ 8 in a row of 16
constexpr int DPP_HALF_MIRROR = 0x141;                           // lane ^ 7

// The levels inside groups of W <= 16 lanes, of one register.
template <int W>
__device__ __forceinline__ double group_sum(double a) {
  if constexpr (W >= 16) a += dpp<DPP_ROR8>(a);
  if constexpr (W >= 8) a += dpp<DPP_XOR3>(dpp<DPP_HALF_MIRROR>(a));  // lane ^ 7 ^ 3 = lane ^ 4
  if constexpr (W >= 4) a += dpp<DPP_XOR2>(a);
  if constexpr (W >= 2) a += dpp<DPP_XOR1>(a);
  return a;
}
__device__ __forceinline__ double row_sum(double a) { return group_sum<16>(a); }

// The ten sums over each group of W lanes (64, 32 or 16), written to its out[0..10)
// (LDS) by the lanes that end up with them. A narrower group starts the tree at its
// own width: with nothing but zeros in the other lanes the sums are the same bits.
template <int W>
__device__ __forceinline__ void wave_sum10(double v[10], double* out) {
  const int lane = threadIdx.x & 63;
  if constexpr (W == 16) {
#pragma unroll
    for (int k = 0; k < 10; ++k) v[k] = row_sum(v[k]);
    if ((lane & 15) == 0)
#pragma unroll
      for (int k = 0; k < 10; ++k) out[k] = v[k];
    return;
  }
  if constexpr (W == 32) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      swap16(v[2 * k], v[2 * k + 1]);  // even rows: value 2k; odd rows: value 2k + 1
      const double r = row_sum(v[2 * k] + v[2 * k + 1]);
      if ((lane & 15) == 0) out[2 * k + ((lane >> 4) & 1)] = r;
    }
    return;
  }
  double h[6];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    swap32(v[2 * k], v[2 * k + 1]);
    h[k] = v[2 * k] + v[2 * k + 1];  // lanes < 32: value 2k; others: value 2k + 1
  }
  h[5] = h[4];
  double r[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    swap16(h[2 * k], h[2 * k + 1]);
    // rows 0..3 hold values 4k, 4k + 2, 4k + 1, 4k + 3 (k = 2: 8, 8, 9, 9)
    r[k] = row_sum(h[2 * k] + h[2 * k + 1]);
  }
  if ((lane & 15) == 0) {
    const int row = lane >> 4, at = ((row & 1) << 1) | (row >> 1);
    out[at] = r[0];
    out[4 + at] = r[1];
    if ((row & 1) == 0) out[8 + (row >> 1)] = r[2];
  }
}

// Six sums over the wave, as above.
__device__ __forceinline__ void wave_sum6(double v[6], double* out) {
  double h[4];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    swap32(v[2 * k], v[2 * k + 1]);
    h[k] = v[2 * k] + v[2 * k + 1];
  }
  h[3] = h[2];
  swap16(h[0], h[1]);
  swap16(h[2], h[3]);
  const double r0 = row_sum(h[0] + h[1]), r1 = row_sum(h[2] + h[3]);
  const int lane = threadIdx.x & 63;
  if ((lane & 15) == 0) {
    const int row = lane >> 4;
    out[((row & 1) << 1) | (row >> 1)] = r0;
    if ((row & 1) == 0) out[4 + (row >> 1)] = r1;
  }
}

template <int W>
__device__ __forceinline__ Fix128 wave_sum(Fix128 v) {
  for (int o = W / 2; o > 0; o >>= 1) {
    const Fix128 w{(unsigned long long)__shfl_xor((long long)v.lo, o), __shfl_xor(v.hi, o)};
    fix_add(v, w);
  }
  return v;
}
template <int W>
__device__ __forceinline__ V3<double> wave_value(const Fix3& v, double inv_scale) {
  return fix_value(Fix3{wave_sum<W>(v.x), wave_sum<W>(v.y), wave_sum<W>(v.z)}, inv_scale);
}

// A member's particles as a small step reads them: SoA planes of stride `st`
// (global memory or LDS) in which particle j is at index j - off.
template <class R>
struct SmallSrc {
  const double *x, *v, *w;
  const R* mu;
  long st;
  int off;
};

// Index range of the particles of i's rod within the exclusion depth of i.
__device__ __forceinline__ void excluded_range(const Dev& d, int i, int& lo, int& hi) {
  const int rod = d.rod[i], b = d.rod_off[rod], e = d.rod_off[rod + 1];
  lo = i - b > d.depth ? i - d.depth : b;
  hi = e - 1 - i > d.depth ? i + d.depth : e - 1;
}

// What a wave finds for one target: the ten dipole sums of pair_acc and, with
// contact, its force and torque.
constexpr int SMALL_OUT = 16;

// One target i of the member [b, e) per W lanes: a wave's for W = 64; with W = 32 or
// 16, for members no larger than that, a wave takes 2 or 4 targets (i, xlo, xhi and
// out differ between its groups; an idle group takes some valid target and an `out`
// that nobody reads). The dipole sum is
// dipole_small_item's, operation by operation. Contact candidates come from the
// same pass: the separation that the pair law needs anyway is compared with r_c
// (widened by 1e-4 where it is FP32), a lane keeps the particles that pass as
// bits, 32 rounds of W particles at a time, and tests those exactly afterwards,
// so that the pair loop carries five integer and compare instructions more and
// no cell list has to be filled, searched and emptied in the step. Excluded
// neighbours are the particles of the index range [xlo, xhi] (i among them).
template <class R, bool HM, int W = 64>
__device__ __forceinline__ void small_target(const Dev& d, const SmallSrc<R>& s, int i, int b, int e,
                                             int xlo, int xhi, long long L, double* out) {
  const int lane = threadIdx.x & (W - 1);
  const unsigned long long group = W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull) << (threadIdx.x & 63 & ~(W - 1));
  const long st = s.st, N = d.n;
  const int io = i - s.off;
  const V3<double> xi{s.x[io], s.x[st + io], s.x[2 * st + io]};
  const R mix = s.mu[io], miy = s.mu[st + io], miz = s.mu[2 * st + io];
  const bool dip = d.dipole_on, con = d.contact_on;
  const double rc2 = d.rc * d.rc;
  const R lim = sizeof(R) == 4 ? (R)fmax(rc2 * 1.0001, 4.8e-38) : (R)(rc2 * 1.000001);
  const unsigned span = (unsigned)(xhi - xlo);
  Acc<R> A{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const R m5 = minus5(R(0));
  Fix3 f{}, t{};
  unsigned near = 0;
  int found = 0, round = 0, base = b;  // round r of `near` is particle base + lane + W r
  const long pp = (long)((L - 1) & 1), pc = (long)(L & 1);
  bool hit = false;
  auto contacts = [&]() {  // the marked particles, exactly
    while (__any(near != 0u)) {
      bool in = false;
      HmOut o;
      int j = 0;
      if (near != 0u) {
        j = base + lane + W * (__ffs((int)near) - 1);
        near &= near - 1u;
        const int jo = j - s.off;
        const V3<double> xj{s.x[jo], s.x[st + jo], s.x[2 * st + jo]};
        const double r2 = r2_exact(xi, xj);
        in = r2 < rc2;
        if (in) {
          hit = true;
          if constexpr (HM) {
            const int np = L >= d.hist_from ? min(d.hc_cnt[pp * N + i], HM_CAP) : 0;
            const int* pj = d.hc_j + pp * HM_CAP * N;
            const double* ps = d.hc_s + pp * 3 * HM_CAP * N;
            V3<double> sprev;
            bool had = false;
            for (int k = 0; k < np; ++k)
              if (pj[(long)k * N + i] == j) {
                sprev = V3<double>{ps[(long)k * N + i], ps[(long)(HM_CAP + k) * N + i],
                                   ps[(long)(2 * HM_CAP + k) * N + i]};
                had = true;
              }
            const V3<double> vi = ld3(s.v, st, (long)io), wi = ld3(s.w, st, (long)io);
            o = hm_pair(d, xi, xj, r2, vi, ld3(s.v, st, (long)jo), wi, ld3(s.w, st, (long)jo),
                        had ? &sprev : nullptr);
            fix_add(f, o.F, d.fix_scale[0], d.flags + FLAG_CONTACT_RANGE);
            fix_add(t, o.T, d.fix_scale[1], d.flags + FLAG_CONTACT_RANGE);
          } else {
            const double r = sqrt(r2);
            const double ov = d.rc - r;
            const double k = (d.kc * ov) / r;
            fix_add(f, k * (xi - xj), d.fix_scale[0], d.flags + FLAG_CONTACT_RANGE);
          }
        }
      }
      if constexpr (HM) {  // this level's history, in the order found
        if (d.hist_write) {
          const unsigned long long who = __ballot(in) & group;
          const int k = found + __popcll(who & ((1ull << (threadIdx.x & 63)) - 1ull));
          if (in && k < HM_CAP) {
            int* cj = d.hc_j + pc * HM_CAP * N;
            double* cs = d.hc_s + pc * 3 * HM_CAP * N;
            cj[(long)k * N + i] = j;
            cs[(long)k * N + i] = o.s.x;
            cs[(long)(HM_CAP + k) * N + i] = o.s.y;
            cs[(long)(2 * HM_CAP + k) * N + i] = o.s.z;
          }
          found += __popcll(who);
        }
      }
    }
  };
  constexpr int U = W == 64 ? 4 : 1;  // rounds in flight
  for (int j0 = b; j0 < e; j0 += U * W) {
    const int jb = j0 + lane;
    double sx[U], sy[U], sz[U];
    R smx[U], smy[U], smz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // loads first; out-of-range entries read the first source
      const int j = (jb + W * u < e ? jb + W * u : b) - s.off;
      sx[u] = s.x[j]; sy[u] = s.x[st + j]; sz[u] = s.x[2 * st + j];
      smx[u] = s.mu[j]; smy[u] = s.mu[st + j]; smz[u] = s.mu[2 * st + j];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0 + W * u >= e) break;  // the whole wave
      const int j = jb + W * u;
      const R dx = (R)(xi.x - sx[u]), dy = (R)(xi.y - sy[u]), dz = (R)(xi.z - sz[u]);
      const R r2 = fma_(dz, dz, fma_(dy, dy, dx * dx));
      if (con && j < e && !(r2 > lim) && (unsigned)(j - xlo) > span) near |= 1u << (round + u);
      if (dip && j < e) {
        const R rinv = (j == i) ? R(0) : rsq(r2);
        pair_acc(dx, dy, dz, smx[u], smy[u], smz[u], mix, miy, miz, rinv, m5, A);
      }
    }
    round += U;
    if (con && (round == 32 || j0 + U * W >= e)) {
      contacts();
      round = 0;
      base = j0 + U * W;
    }
  }
  if (con) {
    V3<double> cF{0.0, 0.0, 0.0}, cT{0.0, 0.0, 0.0};
    if (__any(hit)) {
      cF = wave_value<W>(f, d.fix_inv[0]);
      if constexpr (HM) cT = wave_value<W>(t, d.fix_inv[1]);
    }
    if (lane == 0) {
      out[10] = cF.x; out[11] = cF.y; out[12] = cF.z;
      if constexpr (HM) {
        out[13] = cT.x; out[14] = cT.y; out[15] = cT.z;
        if (d.hist_write) {
          d.hc_cnt[pc * N + i] = min(found, HM_CAP);
          if (found > HM_CAP) atomicOr(&d.flags[FLAG_HM_OVF], 1u);
        }
      }
    }
  }
  if (dip) {
    double v[10] = {(double)A.fx,  (double)A.fy,  (double)A.fz,  (double)A.fm,  (double)A.bsx,
                    (double)A.bsy, (double)A.bsz, (double)A.bmx, (double)A.bmy, (double)A.bmz};
    wave_sum10<W>(v, out);
  }
}

// Dipole force and field of a target from its ten sums, rounded as the slot that
// the separate kernels pass them through (write_slot).
template <class R>
__device__ __forceinline__ void small_slot(double C, const double* F, double mix, double miy,
                                           double miz, V3<double>& Fd, V3<double>& Bd) {
  R p[6];
  write_slot(p, 1, 0, C, F, mix, miy, miz);
  Fd = V3<double>{(double)p[0], (double)p[1], (double)p[2]};
  Bd = V3<double>{(double)p[3], (double)p[4], (double)p[5]};
}

}  // namespace rodmx
