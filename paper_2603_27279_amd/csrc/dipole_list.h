// Dipole-dipole interaction with a cutoff (Methods, "Magnetic interactions",
// truncated as the paper's pair style truncates it): particle i feels the
// particles j of its member with r^2 = (dx dx + dy dy) + dz dz < dcut^2 (exact
// FP64 selection, as in the contact search), through the same pair law as the
// all-pairs sum. Each particle keeps a Verlet list of the member's particles
// closer than dcut + skin, rebuilt with the contact lists (see
// contact_listed).
//
// A rebuild first sorts the particles by cell (cells of side dcut + skin, so a
// particle's candidates lie in the 3 x 3 x 3 cells around its own). A cell's
// bucket is its member number above the low bits of its three coordinates,
// interleaved bit by bit (a Z-order curve), so that consecutive buckets are
// neighbouring cells. Counting sort: each particle's bucket and an atomic slot
// in it; exclusive sums of the counts in two passes; the particles grouped by
// bucket; within a bucket ranked by index (a fixed order). The list walk runs
// over the sorted positions, and the positions are dealt to the XCDs in
// contiguous ranges, so a workgroup's particles share their partners' lines
// with the workgroups running beside it on the same L2.
//
// Cells whose coordinates differ by a multiple of 2^bits along an axis share a
// bucket; every sorted record carries the high bits of its cell's coordinates
// (a tag), and a walk takes from a bucket only the records of the cell it
// visits. The list order and the summation are fixed by the sort: a run
// repeated gives the same bits.
#pragma once
#include "contact_body.h"
#include "small_body.h"

namespace rodmx {

// Cell coordinates of x relative to the key origin.
__device__ __forceinline__ int dl_coord(double x, double org, double inv) {
  return cell_coord(x - org, inv);
}

// The low bits of g deposited at the set bits of `mask`, lowest first.
__device__ __forceinline__ unsigned dl_spread(unsigned g, unsigned mask) {
  unsigned out = 0u;
  for (unsigned m = mask; m != 0u; m &= m - 1u, g >>= 1) out |= (g & 1u) ? (m & (0u - m)) : 0u;
  return out;
}

// High bits of a cell's coordinates (those above each axis's key bits), ten
// signed bits per axis; DL_TAG_FAR when one does not fit.
constexpr unsigned DL_TAG_FAR = 0xffffffffu;
__device__ __forceinline__ unsigned dl_tag(const Dev& d, int gx, int gy, int gz) {
  const int h[3] = {gx >> d.dl_bits[0], gy >> d.dl_bits[1], gz >> d.dl_bits[2]};
  unsigned t = 0u;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (h[a] < -512 || h[a] > 511) return DL_TAG_FAR;
    t |= ((unsigned)h[a] & 1023u) << (10 * a);
  }
  return t;
}

__device__ __forceinline__ unsigned dl_bucket(const Dev& d, int gx, int gy, int gz, int mem) {
  return ((unsigned)mem << d.dl_mshift) | dl_spread((unsigned)gx, d.dl_axis[0]) |
         dl_spread((unsigned)gy, d.dl_axis[1]) | dl_spread((unsigned)gz, d.dl_axis[2]);
}

// Bucket and counting slot of particle i (`valid`: it exists; whole waves call), and
// its share of its block of buckets, one addition per wave and block. The blocks are few,
// so workgroups add to one of DL_COPIES sets of sums: 87,000 particles in an evaluation
// 57 us on one set, 18 on eight and 13 on 16 as on 64, whose sums k_dl_start then reads
// in 11 us against 6. The evaluation whole: 285 us on one, 243 on 16 (262,144: 589, 452).
__device__ __forceinline__ void dl_bin(const Dev& d, long i, bool valid) {
  unsigned b = 0;
  if (valid) {
    const double* p = static_cast<const double*>(__builtin_assume_aligned(d.xm + 8 * i, 64));
    b = dl_bucket(d, dl_coord(p[0], d.dl_org[0], d.dl_inv), dl_coord(p[1], d.dl_org[1], d.dl_inv),
                  dl_coord(p[2], d.dl_org[2], d.dl_inv), d.mem[i]);
    d.dl_bkt[i] = (int)b;
    d.dl_slot[i] = atomicAdd(&d.dl_cnt[b], 1);
  }
  const int blk = (int)(b / DL_SCAN);
  unsigned long long todo = __ballot(valid);
  while (todo != 0ull) {
    const int lead = __ffsll((long long)todo) - 1;
    const unsigned long long same = __ballot(valid && blk == __builtin_amdgcn_readlane(blk, lead));
    if ((int)__lane_id() == lead)
      atomicAdd(&d.dl_aux[(long)(blockIdx.x % DL_COPIES) * (d.dl_nb / DL_SCAN) + blk], __popcll(same));
    todo &= ~same;
  }
}

// Workgroup b of G as dealt to the XCDs in turn, renumbered so that each XCD
// holds a contiguous range of the sorted positions.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned G) {
  const unsigned per = G >> 3, rem = G & 7u, x = b & 7u, k = b >> 3;
  return x < rem ? x * (per + 1u) + k : rem * (per + 1u) + (x - rem) * per + k;
}

// Lanes per particle in the list build and walk.
constexpr int DL_LANES = 8;

// The particle and sorted position served by lane group `g` of workgroup blk:
// over the whole system sorted position t (workgroups dealt to the XCDs in
// contiguous ranges), over one rod's range (the per-rod loop) the rod's
// particle i at its own position. False past the end.
__device__ __forceinline__ bool dl_target(const Dev& d, unsigned blk, unsigned blocks, long* i, long* t) {
  const long g = threadIdx.x / DL_LANES;
  const long per = blockDim.x / DL_LANES;
  if (d.i_lo == 0 && d.i_hi == d.n) {
    *t = (long)xcd_block(blk, blocks) * per + g;
    if (*t >= d.n) return false;
    *i = d.dl_sorted[*t];
  } else {
    *i = d.i_lo + (long)blk * per + g;
    if (*i >= d.i_hi) return false;
    *t = d.dl_pos[*i];
  }
  return true;
}

// Per lane group of a list-build workgroup: the 27 cells' first sorted
// position, the number of candidates before each cell, and each cell's tag.
struct DlCells { int qb[27]; int pre[28]; unsigned tag[27]; };
constexpr int DL_BUILD_GROUPS = 256 / DL_LANES;

// List rebuild. The candidates are the records of the 27 cells around the
// particle's own, taken in a fixed order (cells by z, y, x offset, each cell's
// records in sorted order). The particle's eight lanes first fetch the 27
// cells' ranges together (four cells per lane) and keep their first positions
// and running counts in LDS; they then take the candidates eight at a time,
// four such chunks in flight, and write the accepted ones in candidate order
// (each lane's place from a ballot), so the list is what one thread taking the
// candidates in that order would write.
__device__ __forceinline__ void dipole_list_build(const Dev& d, unsigned blk, unsigned blocks,
                                                  DlCells* cells) {
  constexpr int CH = 4;  // chunks of eight candidates in flight
  const long N = d.n;
  long i, t;
  const bool live = dl_target(d, blk, blocks, &i, &t);  // whole lane groups agree
  if (!live) return;
  const int s = threadIdx.x % DL_LANES;
  DlCells& cl = cells[threadIdx.x / DL_LANES];
  const int gshift = (int)(__lane_id() & ~(unsigned)(DL_LANES - 1));
  const unsigned gmask = (1u << DL_LANES) - 1u;
  const double* own = static_cast<const double*>(__builtin_assume_aligned(d.xm + 8 * i, 64));
  const V3<double> xi{own[0], own[1], own[2]};
  const double rs = d.dcut + d.skin, rs2 = rs * rs;
  const int mem = d.mem[i];
  const int gx = dl_coord(xi.x, d.dl_org[0], d.dl_inv), gy = dl_coord(xi.y, d.dl_org[1], d.dl_inv),
            gz = dl_coord(xi.z, d.dl_org[2], d.dl_inv);
  // cells s, s + 8, s + 16, s + 24 of this lane: ranges, then running counts
  int qb[4], len[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int c = s + DL_LANES * m;
    qb[m] = 0; len[m] = 0;
    if (c < 27) {
      const int cx = gx + c % 3 - 1, cy = gy + (c / 3) % 3 - 1, cz = gz + c / 9 - 1;
      const unsigned key = dl_bucket(d, cx, cy, cz, mem);
      qb[m] = d.dl_start[key];
      len[m] = d.dl_start[key + 1] - qb[m];
      cl.tag[c] = dl_tag(d, cx, cy, cz);
    }
  }
  int run = 0;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    int v = len[m];  // inclusive scan over the group's eight lanes
#pragma unroll
    for (int o = 1; o < DL_LANES; o <<= 1) {
      const int u = __shfl_up(v, o, DL_LANES);
      if (s >= o) v += u;
    }
    const int c = s + DL_LANES * m;
    if (c < 27) { cl.qb[c] = qb[m]; cl.pre[c] = run + v - len[m]; }
    run += __shfl(v, DL_LANES - 1, DL_LANES);
  }
  if (s == 0) cl.pre[27] = run;
  __builtin_amdgcn_wave_barrier();  // the group's LDS entries are written by its own wave
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int total = run;
  int nc = 0, c = 0;
  for (int p0 = 0; p0 < total; p0 += CH * DL_LANES) {
    DlRec e[CH];
    int cc[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int p = p0 + u * DL_LANES + s;
      cc[u] = -1;
      if (p < total) {
        while (cl.pre[c + 1] <= p) ++c;
        cc[u] = c;
        e[u] = d.dl_rec[cl.qb[c] + (p - cl.pre[c])];
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      bool acc = false;
      if (cc[u] >= 0) {
        const int k = cc[u];
        const unsigned tag = cl.tag[k];
        const V3<double> xj{e[u].x, e[u].y, e[u].z};
        bool same = e[u].tag == tag && tag != DL_TAG_FAR;
        if (!same && (e[u].tag == DL_TAG_FAR || tag == DL_TAG_FAR))  // another cell of the bucket?
          same = dl_coord(xj.x, d.dl_org[0], d.dl_inv) == gx + k % 3 - 1 &&
                 dl_coord(xj.y, d.dl_org[1], d.dl_inv) == gy + (k / 3) % 3 - 1 &&
                 dl_coord(xj.z, d.dl_org[2], d.dl_inv) == gz + k / 9 - 1;
        acc = same && e[u].i != (int)i && r2_exact(xi, xj) < rs2;
      }
      const unsigned grp = (unsigned)(__ballot(acc) >> gshift) & gmask;
      const int at = nc + __popc(grp & ((1u << s) - 1u));
      if (acc && at < DNBR_CAP) d.dnbr[(long)at * N + t] = e[u].i;
      nc += __popc(grp);
    }
  }
  if (s == 0) {
    d.dnbr_cnt[t] = min(nc, DNBR_CAP);
    if (nc > DNBR_CAP) atomicOr(&d.flags[FLAG_DIP_OVF], 1u);
    st3(d.xb, N, i, xi);
    if (i == 0) d.rebuild[3] = 1u;  // (k_bond_kick takes it back)
  }
}

// Dipole force and field of one particle from its list, written to slot 0 of
// the FP64 partial sums (the only slot in this mode). W lanes per particle: lane s
// takes entries s, s + W, s + 2W, ... in order; the W partial sums are added by a
// fixed xor tree.
//
// The walk is bound by the gathers of its partners' records. One lane fetching its
// own partner takes three 16-byte loads at 64 distinct lines each, and the texture
// addresser handles a line per clock. Here four lanes fetch one 64-byte record
// together (a line each four lanes, four loads for the wave's 64 partners) into
// registers a round ahead, pass it through a wave's 4 KiB of LDS and read back
// their own; the quarters of a record are rotated by its number so that the eight
// lanes of a read phase fall on all banks. 262,144 particles at cutoff 3 (38 entries
// each): 58 -> 50 us with four lanes per
// particle (eight 55, sixteen 84, two 49).
constexpr int DL_WALK_LANES = 4;
struct DlStage { double2 quarter[64 * 4]; };  // one wave's records of a round
__device__ __forceinline__ void dipole_list_walk(const Dev& d, unsigned blk, DlStage* stages) {
  constexpr int W = DL_WALK_LANES;
  const long N = d.n;
  const int lane = threadIdx.x & 63;
  DlStage& st = stages[threadIdx.x >> 6];
  long i, t;
  bool live;
  {
    const long g = threadIdx.x / W, per = blockDim.x / W;
    if (d.i_lo == 0 && d.i_hi == N) {
      t = (long)xcd_block(blk, gridDim.x) * per + g;
      live = t < N;
      if (!live) t = N - 1;
      i = d.dl_sorted[t];
    } else {
      i = d.i_lo + (long)blk * per + g;
      live = i < d.i_hi;
      if (!live) i = d.i_lo;
      t = d.dl_pos[i];
    }
  }
  const int s = threadIdx.x % W;
  const double* own = static_cast<const double*>(__builtin_assume_aligned(d.xm + 8 * i, 64));
  const V3<double> xi{own[0], own[1], own[2]}, mi{own[3], own[4], own[5]};
  const double rd2 = d.dcut * d.dcut;
  Acc<double> A{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  auto pair = [&](V3<double> xj, V3<double> mj) {
    const double r2 = r2_exact(xi, xj);
    if (!(r2 < rd2)) return;
    const V3<double> r = xi - xj;
    pair_acc(r.x, r.y, r.z, mj.x, mj.y, mj.z, mi.x, mi.y, mi.z, rsqrt_pair(r2), -5.0, A);
  };
  const int nc = live ? d.dnbr_cnt[t] : 0;
  int most = nc;  // of the wave's particles
#pragma unroll
  for (int o = W; o < 64; o <<= 1) most = max(most, __shfl_xor(most, o, 64));
  // Lane l fetches quarter (l & 3) ^ f of the records of partners 16 m + l / 4, m =
  // 0 .. 3, f the record's rotation; entry k of the round is the lane's own partner.
  // Entries past the end of a list are read too (they hold older particles, or 0), so
  // that no load waits for the count.
  const int rec = lane >> 2, quarter = (lane & 3) ^ ((rec >> 1) & 3);
  auto entry = [&](int k) { return d.dnbr[(long)(k < DNBR_CAP ? k : s) * N + t]; };
  auto fetch = [&](int j, int m) {
    const long p = __shfl(j, 16 * m + rec, 64);
    double2 v{0.0, 0.0};
    if (quarter < 3) v = reinterpret_cast<const double2*>(d.xm + 8 * p)[quarter];
    return v;
  };
  const int first = entry(s);
  int next = entry(s + W), after = entry(s + 2 * W);
  double2 v0 = fetch(first, 0), v1 = fetch(first, 1), v2 = fetch(first, 2), v3 = fetch(first, 3);
  for (int k0 = 0; k0 < most; k0 += W) {
    st.quarter[lane] = v0;
    st.quarter[64 + lane] = v1;
    st.quarter[128 + lane] = v2;
    st.quarter[192 + lane] = v3;
    if (k0 + W < most) {
      v0 = fetch(next, 0);
      v1 = fetch(next, 1);
      v2 = fetch(next, 2);
      v3 = fetch(next, 3);
      next = after;
      after = entry(k0 + 3 * W + s);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS is the wave's own
    __builtin_amdgcn_wave_barrier();
    if (k0 + s < nc) {
      const double2* r = st.quarter + 4 * lane;
      const int f = (lane >> 1) & 3;
      const double2 a = r[f], b = r[1 ^ f], c = r[2 ^ f];
      pair(V3<double>{a.x, a.y, b.x}, V3<double>{b.y, c.x, c.y});
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  double sum[NACC] = {A.fx, A.fy, A.fz, A.fm, A.bsx, A.bsy, A.bsz, A.bmx, A.bmy, A.bmz}, w[6];
  write_slot(w, 1, 0, d.C, sum, mi.x, mi.y, mi.z);
#pragma unroll
  for (int c = 0; c < 6; ++c) w[c] = group_sum<W>(w[c]);
  if (s == 0 && live) {
    double* p = d.dpart;
#pragma unroll
    for (int c = 0; c < 6; ++c) p[c * N + i] = w[c];
  }
}

}  // namespace rodmx
