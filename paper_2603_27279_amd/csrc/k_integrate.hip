// Per-particle kernels of the time step: the first half-kick / drift / Richardson
// quaternion update with boundary conditions and dipole rotation (pre), and the
// force gather with Zeeman, damping and external terms followed by the second
// half-kick (post). SI "Equations of motion"; dipoles rotate with the particle
// (main text, magnetised beams); Zeeman force and torque (Methods).
#include <algorithm>

#include "rod.h"
#include "rod_internal.h"
#include "rod_math.h"
#include "particle_body.h"
#include "dipole_list.h"
#include "integrate_body.h"  // last: contraction within expressions from here on

namespace rodmx {

__device__ __forceinline__ V3<double> pre_particle(const Dev& d, long i, int mode, long long n,
                                                   long long lvl);

__global__ __launch_bounds__(256) void k_pre(Dev d, int mode) {
  const long i = d.i_lo + (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long n = d.step[0];
  const long long lvl = n + (mode == PRE_STEP ? 1 : 0);  // level of the coming force evaluation
  if (i == 0) d.step[d.lc] = lvl;
  const bool valid = i < d.i_hi;
  V3<double> x{0.0, 0.0, 0.0};
  if (valid) x = pre_particle(d, i, mode, n, lvl);
  chunk_box(d, i, x, valid);
}

// Cell-list entries of the level being evaluated, when its contact lists are
// rebuilt (lazy_cells: the particle kernels left the list empty). Most steps
// keep their lists, and then every workgroup only reads the flag: the grid is
// capped (gated_blocks), each thread
// striding over the particles CELL_INSERT_ILP at a time, so that their loads
// and slot claims are in flight together.
constexpr int CELL_INSERT_ILP = 4;
__global__ __launch_bounds__(256) void k_cell_insert(Dev d, int build) {
  // three flags that nothing else has to be loaded for: an idle launch is their latency
  const bool stale = build || d.rebuild[d.lc & 1] != 0u, over = d.rebuild[2] != 0u;
  const bool dirty = d.cell_dirty[(d.lc & 1) ^ 1] != 0;
  if (!stale && !over && !dirty) return;
  const long long lvl = d.step[d.lc];
  const long N = d.n;
  const long G = (long)gridDim.x * blockDim.x;
  if (dirty) {  // the table filled a step ago is done with
    const CellTab old = cell_tab(d, lvl - 1);
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += G) old.cnt[d.key[i]] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *old.ovf_cnt = 0;
  }
  if (!stale && !over) return;  // the lists stay, and hold every candidate
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    d.cell_dirty[d.lc & 1] = 1;
    if (stale) d.rebuild[2] = 0u;  // (the build of this level sets it again; all fill either way)
  }
  if (stale && d.dcut > 0.0 && d.halo) {  // the cutoff sort's buckets in the same launch
    for (long i0 = (long)blockIdx.x * blockDim.x; i0 < N; i0 += G) dl_bin(d, i0 + threadIdx.x, i0 + threadIdx.x < N);
  }
  const CellTab t = cell_tab(d, lvl);
  for (long i0 = (long)blockIdx.x * blockDim.x + threadIdx.x; i0 < N; i0 += CELL_INSERT_ILP * G) {
    V3<double> x[CELL_INSERT_ILP];
    int rod[CELL_INSERT_ILP], slot[CELL_INSERT_ILP];
    unsigned key[CELL_INSERT_ILP];
#pragma unroll
    for (int u = 0; u < CELL_INSERT_ILP; ++u) {
      const long i = i0 + u * G < N ? i0 + u * G : i0;
      x[u] = ld3(d.x, N, i);
      rod[u] = d.rod[i];
      key[u] = cell_key(d, x[u], d.mem[i]);
    }
#pragma unroll
    for (int u = 0; u < CELL_INSERT_ILP; ++u)  // the claims, all in flight
      slot[u] = i0 + u * G < N ? atomicAdd(&t.cnt[key[u]], 1) : 0;
#pragma unroll
    for (int u = 0; u < CELL_INSERT_ILP; ++u)
      if (i0 + u * G < N) cell_place(d, t, i0 + u * G, x[u], rod[u], key[u], slot[u]);
  }
}

hipError_t launch_cell_insert(const Dev& d, int build, hipStream_t s, const hipEvent_t* ev) {
  const long blocks = (d.n + 255) / 256;
  launch_k(ev, k_cell_insert, dim3(gated_blocks(blocks)), dim3(256), s, d, build);
  return hipGetLastError();
}

// The pre kernel's work for particle i; returns its position at level lvl.
__device__ __forceinline__ V3<double> pre_particle(const Dev& d, long i, int mode, long long n,
                                                   long long lvl) {
  const long N = d.n;
  const int b = d.bc[i];
  // state read in place, or from separate planes (out-of-place step)
  const double* sx = d.src ? d.src : d.x;
  const double* sv = d.src ? d.src + 3 * N : d.v;
  const double* sq = d.src ? d.src + 6 * N : d.q;
  const double* sw = d.src ? d.src + 10 * N : d.w;
  const double* sF = d.src ? d.src + 13 * N : d.F;
  const double* sT = d.src ? d.src + 16 * N : d.T;
  Q4<double> q = ld4(sq, N, i);
  V3<double> x = ld3(sx, N, i);
  const V3<double> mb = ld3(d.mb, N, i);
  const int mem = d.mem[i], rod = d.rod[i];
  V3<double> vh{0.0, 0.0, 0.0};  // half-step velocity
  if (mode == PRE_STEP) {
    V3<double> v = ld3(sv, N, i), w = ld3(sw, N, i);
    advance(d, i, b, lvl, x, v, q, w, ld3(sF, N, i), ld3(sT, N, i), d.minv[i], d.Iinv[i],
            d.src != nullptr || d.nx != nullptr, d.lc & 1, d.halo == nullptr);
    vh = v;
  } else if (mode == PRE_PREPARE) {
    q = qnormalize(q);
    if (b != 0) {
      V3<double> z{0.0, 0.0, 0.0};
      st3(d.v, N, i, z);
      st3(d.w, N, i, z);
    }
    if (b == 2) {
      q = drive_q(d, n);
      double om = 2.0 * 3.14159265358979323846 / ((double)d.period * d.dt);
      st3(d.w, N, i, V3<double>{om * d.axis[0], om * d.axis[1], om * d.axis[2]});
    }
    st4(d.q, N, i, q);
  }
  moment_and_cell(d, i, q, x, mb, mem, rod, lvl, !(d.lazy_cells && mode == PRE_STEP));
  if (d.halo) {  // opening the fused bond and kick chain: lists still good at these positions?
    halo_store(d, i, lvl, x, q, vh);
    if (d.use_lists) {
      const V3<double> m = x - ld3(d.xb, N, i);
      const double lim = NBR_MOVE * d.skin;
      // (positions the caller has changed count too; particle 0 speaks for a mark, or
      // every wave's atomic would meet at the flag)
      const bool far = !(dot(m, m) <= lim * lim) || (i == 0 && d.rebuild[3] != 0u);
      const unsigned long long who = __ballot(far);
      if (far && __lane_id() == (unsigned)(__ffsll((long long)who) - 1))
        atomicOr(&d.rebuild[d.lc & 1], 1u);
    }
  }
  return x;
}

// Dipole force and field of particle i: its S slots added in slot order, in
// FP64, B slots per round trip (FP32 slots of the mixed path: 16; FP64: 8).
// Slots past the member's own count hold zeros.
template <class T, int B>
__device__ __forceinline__ void slot_sum(const T* dp, long N, int s_begin, int s_end, long i,
                                         V3<double>& Fd, V3<double>& Bd) {
  for (int s0 = s_begin; s0 < s_end; s0 += B) {
    T v[B][6];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const T* q = dp + (long)(s0 + k) * 6 * N;
      if (s0 + k < s_end)
#pragma unroll
        for (int c = 0; c < 6; ++c) v[k][c] = q[c * N + i];
    }
#pragma unroll
    for (int k = 0; k < B; ++k)
      if (s0 + k < s_end) {
        Fd = Fd + V3<double>{(double)v[k][0], (double)v[k][1], (double)v[k][2]};
        Bd = Bd + V3<double>{(double)v[k][3], (double)v[k][4], (double)v[k][5]};
      }
  }
}

// The same over slots in FP64 parts: a slot is the sum of its parts rounded to FP32, as
// one work item would have stored it.
__device__ __forceinline__ void slot_sum_parts(const double* dp, long N, int parts, int s_begin,
                                               int s_end, long i, V3<double>& Fd, V3<double>& Bd) {
  for (int s = s_begin; s < s_end; ++s) {
    double v[PARTS_MAX][6];
#pragma unroll
    for (int k = 0; k < PARTS_MAX; ++k) {
      const double* q = dp + ((long)s * parts + k) * 6 * N;
#pragma unroll
      for (int c = 0; c < 6; ++c) v[k][c] = k < parts ? q[c * N + i] : 0.0;
    }
    float f[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) f[c] = (float)(((v[0][c] + v[1][c]) + v[2][c]) + v[3][c]);
    Fd = Fd + V3<double>{(double)f[0], (double)f[1], (double)f[2]};
    Bd = Bd + V3<double>{(double)f[3], (double)f[4], (double)f[5]};
  }
}

// The dipole force and field of particle i from slots [s_begin, s_end) when
// `mask` asks for them (zero otherwise). Called first in the particle
// kernels: the slot loads are the longest chain of the gather, and few other
// values are live yet.
__device__ __forceinline__ void dipole_sums(const Dev& d, long i, int mask, V3<double>& Fd,
                                            V3<double>& Bd, int s_begin, int s_end) {
  Fd = V3<double>{0.0, 0.0, 0.0};
  Bd = V3<double>{0.0, 0.0, 0.0};
  if (!((mask & 2) && d.dipole_on)) return;
  if (d.parts > 1) slot_sum_parts(d.dpart, d.n, d.parts, s_begin, s_end, i, Fd, Bd);
  else if (d.dslotf) slot_sum<float, 8>(d.dslotf, d.n, s_begin, s_end, i, Fd, Bd);
  else slot_sum<double, 8>(d.dpart, d.n, s_begin, s_end, i, Fd, Bd);
}

// Systems below 65,536 particles spread the gather over four waves per 64
// particles (a quarter of the workgroups a particle per thread would give):
// wave w adds the slots [w G, (w + 1) G), G = ceil(S / 4), of each of the 64
// particles, the four partial sums meet in LDS, and wave 0 adds them in wave
// order and completes the kernel alone. Every gather of such a system (fused
// kick and unfused post) sums in this order, so launch forms stay bitwise
// equal; larger systems add the slots one after another.
constexpr int SPLIT_WAVES = 4;
inline bool particle_split(long n) { return n < 65536; }

// Slot sums of particle i in the kernel's layout: all slots (SPLIT false), or
// this wave's group, combined through `part` ([SPLIT_WAVES][64][6]); returns
// false on waves other than the first, which then leave the kernel.
template <bool SPLIT>
__device__ __forceinline__ bool dipole_sums_of(const Dev& d, long i, bool valid, int mask,
                                               V3<double>& Fd, V3<double>& Bd, double* part) {
  if constexpr (!SPLIT) {
    if (valid) dipole_sums(d, i, mask, Fd, Bd, 0, d.max_slots);
    return true;
  } else {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int G = (d.max_slots + SPLIT_WAVES - 1) / SPLIT_WAVES;
    const int sb = min(w * G, d.max_slots), se = min(sb + G, d.max_slots);
    V3<double> f{0.0, 0.0, 0.0}, b{0.0, 0.0, 0.0};
    if (valid) dipole_sums(d, i, mask, f, b, sb, se);
    double* o = part + 6 * (w * 64 + lane);
    o[0] = f.x; o[1] = f.y; o[2] = f.z; o[3] = b.x; o[4] = b.y; o[5] = b.z;
    __syncthreads();
    if (w != 0) return false;
    Fd = V3<double>{0.0, 0.0, 0.0};
    Bd = V3<double>{0.0, 0.0, 0.0};
    for (int u = 0; u < SPLIT_WAVES; ++u) {
      const double* q = part + 6 * (u * 64 + lane);
      Fd = Fd + V3<double>{q[0], q[1], q[2]};
      Bd = Bd + V3<double>{q[3], q[4], q[5]};
    }
    return true;
  }
}

template <bool HM, bool FL, bool SPLIT>
__global__ __launch_bounds__(256) void k_post(Dev d, int mode, int mask, double* Fo, double* To,
                                              double* Bo) {
  __shared__ double part[SPLIT ? 6 * 64 * SPLIT_WAVES : 1];
  const long i = d.i_lo + (SPLIT ? (long)blockIdx.x * 64 + (threadIdx.x & 63)
                                 : (long)blockIdx.x * blockDim.x + threadIdx.x);
  const long N = d.n;
  const long long lvl = d.step[d.lc];  // level of the forces being gathered
  if (i == 0 && (!SPLIT || threadIdx.x < 64)) {
    if (mode == POST_KICK) d.step[0] = lvl;
    *cell_tab(d, lvl).ovf_cnt = 0;  // the contact pass that used the overflow list has finished
    if (d.use_lists) d.rebuild[d.lc & 1] = 0u;  // and so has the one that read this flag
  }
  V3<double> Fd, Bd;
  if (!dipole_sums_of<SPLIT>(d, i, i < d.i_hi, mask, Fd, Bd, part)) return;
  if (i >= d.i_hi) return;
  PIn p = load_particle(d, i);
  const int key = d.contact_on ? d.key[i] : 0;
  V3<double> F, T;
  gather<HM, FL>(d, i, mask, lvl, Bo, p, Fd, Bd, F, T);
  if (mode == POST_EVAL) {
    st3(Fo, N, i, F);
    st3(To, N, i, T);
  } else if (mode == POST_KICK) {
    kick(d, i, F, T, p, true);
  } else {  // prepare: forces of the initial state, no kick
    st3(d.F, N, i, F);
    st3(d.T, N, i, T);
    if (!finite3(F) || !finite3(T) || !finite3(p.x)) atomicOr(&d.flags[FLAG_NONFINITE], 1u);
  }
  if (d.contact_on) cell_tab(d, lvl).cnt[key] = 0;  // empty the cell list for the next build
}

// The end of one step and the start of the next in one pass: gather and second
// half-kick at level L = step[lc], then half-kick, drift, rotation, moments and
// cell insertion for level L + 1 (written to step[3 - lc]). The cell list and
// overflow list of level L are emptied while those of level L + 1 are filled.
// FL: with the immersed-boundary penalty, whose positions are put aside (d.ibm_x) for
// the spreading in the next force launch.
template <bool HM, bool SPLIT, bool FL>
__global__ __launch_bounds__(256) void k_kick(Dev d, double* Bo) {
  __shared__ double part[SPLIT ? 6 * 64 * SPLIT_WAVES : 1];
  const long i = d.i_lo + (SPLIT ? (long)blockIdx.x * 64 + (threadIdx.x & 63)
                                 : (long)blockIdx.x * blockDim.x + threadIdx.x);
  const long long L = d.step[d.lc];
  if (i == 0 && (!SPLIT || threadIdx.x < 64)) {
    d.step[3 - d.lc] = L + 1;
    *cell_tab(d, L).ovf_cnt = 0;
    if (d.use_lists) d.rebuild[d.lc & 1] = 0u;
  }
  const bool valid = i < d.i_hi;
  V3<double> x{0.0, 0.0, 0.0};
  V3<double> Fd, Bd;
  if (!dipole_sums_of<SPLIT>(d, i, valid, ROD_TERM_ALL, Fd, Bd, part)) return;
  if (valid) {
    PIn p = load_particle(d, i);
    const int key = d.contact_on ? d.key[i] : 0;
    V3<double> F, T;
    gather<HM, FL>(d, i, ROD_TERM_ALL, L, Bo, p, Fd, Bd, F, T);
    if constexpr (FL) st3(d.ibm_x, d.n, i, p.x);
    // in place, the next half-kick overwrites v and w; out of place (a recorded
    // state) the full-step v and w stay with level L
    const bool apart = d.nx != nullptr;
    kick(d, i, F, T, p, apart);
    if (d.contact_on) cell_tab(d, L).cnt[key] = 0;
    advance(d, i, p.b, L + 1, p.x, p.v, p.q, p.w, F, T, p.minv, p.Iinv, apart, (d.lc & 1) ^ 1);
    moment_and_cell(d, i, p.q, p.x, p.mb, p.mem, p.rod, L + 1, !d.lazy_cells);
    x = p.x;
  }
  chunk_box(d, i, x, valid);
}

// Energies: bond terms attributed to the bond's first particle, Zeeman -m.B, dipole
// -1/2 m.B_dip, contact (pairs halved), kinetic. A workgroup forms the nine terms of
// 256 particles of one member and adds them up; a second kernel adds a member's
// workgroups. Sums in a fixed order. (One workgroup per member over [9][N] stored
// terms took 104 us for a member of 10,368.)
constexpr int ENERGY_BLOCK = 256;
// First partial sum of member m, which begins at particle b: a member of n particles
// has ceil(n / 256) of them, at most floor((b + n) / 256) - floor(b / 256) + 1.
__device__ __forceinline__ long energy_base(int m, int b) { return b / ENERGY_BLOCK + m; }

__device__ __forceinline__ double lanes_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__global__ __launch_bounds__(ENERGY_BLOCK) void k_energy_part(Dev d, const double* Bdip, double* part) {
  __shared__ double sums[ENERGY_BLOCK / 64][9];
  const int m = blockIdx.x;
  const int b = d.mrange[2 * m], e = d.mrange[2 * m + 1];
  for (int c = blockIdx.y; c * ENERGY_BLOCK < e - b; c += gridDim.y) {
    const long i = b + (long)c * ENERGY_BLOCK + threadIdx.x;
    const long N = d.n;
    double E[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (i < e) {
      if (d.bflags[i] & 1)
        for (int t = 0; t < 4; ++t) E[t] = d.bE[t * N + i];
      const V3<double> mu = ld3(d.mu, N, i);
      const double* f = field_row(d, d.step[d.lc], m);
      const V3<double> x = ld3(d.x, N, i);
      const V3<double> B{f[0] + f[3] * x.x + f[4] * x.y + f[5] * x.z,
                         f[1] + f[6] * x.x + f[7] * x.y + f[8] * x.z,
                         f[2] + f[9] * x.x + f[10] * x.y + f[11] * x.z};
      E[4] = -dot(mu, B);
      if (d.dipole_on) E[5] = -0.5 * dot(mu, ld3(Bdip, N, i));
      if (d.contact_on) E[6] = d.cE[i];
      const V3<double> v = ld3(d.v, N, i), w = ld3(d.w, N, i);
      E[7] = 0.5 * d.mass[i] * dot(v, v);
      E[8] = 0.5 * d.inertia[i] * dot(w, w);
    }
    for (int t = 0; t < 9; ++t) E[t] = lanes_sum(E[t]);
    if ((threadIdx.x & 63) == 0)
      for (int t = 0; t < 9; ++t) sums[threadIdx.x >> 6][t] = E[t];
    __syncthreads();
    if (threadIdx.x < 9) {
      double s = 0.0;
      for (int w = 0; w < ENERGY_BLOCK / 64; ++w) s += sums[w][threadIdx.x];
      part[(energy_base(m, b) + c) * 9 + threadIdx.x] = s;
    }
    __syncthreads();
  }
}

// One wave per member and term.
__global__ __launch_bounds__(64) void k_energy_reduce(Dev d, const double* part, double* out) {
  const int m = blockIdx.x, t = blockIdx.y;
  const int b = d.mrange[2 * m], e = d.mrange[2 * m + 1];
  const double* p = part + energy_base(m, b) * 9 + t;
  double s = 0.0;
  for (int c = threadIdx.x; c < (e - b + ENERGY_BLOCK - 1) / ENERGY_BLOCK; c += 64) s += p[9 * c];
  s = lanes_sum(s);
  if (threadIdx.x == 0) out[m * 9 + t] = s;
}

static inline unsigned blocks_for(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_pre(const Dev& d, int mode, hipStream_t s, const hipEvent_t* ev) {
  const int bs = particle_block(d.n);
  launch_k(ev, k_pre, dim3(blocks_for(d.i_hi - d.i_lo, bs)), dim3(bs), s, d, mode);
  return hipGetLastError();
}

template <bool SPLIT>
static void post_variant(const Dev& d, int mode, int mask, double* Fo, double* To, double* Bo,
                         hipStream_t s, const hipEvent_t* ev, dim3 g, dim3 b) {
  if (d.ibm_u) {
    if (d.hm) launch_k(ev, k_post<true, true, SPLIT>, g, b, s, d, mode, mask, Fo, To, Bo);
    else launch_k(ev, k_post<false, true, SPLIT>, g, b, s, d, mode, mask, Fo, To, Bo);
  } else if (d.hm) {
    launch_k(ev, k_post<true, false, SPLIT>, g, b, s, d, mode, mask, Fo, To, Bo);
  } else {
    launch_k(ev, k_post<false, false, SPLIT>, g, b, s, d, mode, mask, Fo, To, Bo);
  }
}

hipError_t launch_post(const Dev& d, int mode, int mask, double* Fo, double* To, double* Bo,
                       hipStream_t s, const hipEvent_t* ev) {
  if (particle_split(d.n)) {  // four waves per 64 particles
    post_variant<true>(d, mode, mask, Fo, To, Bo, s, ev, dim3(blocks_for(d.i_hi - d.i_lo, 64)),
                       dim3(64 * SPLIT_WAVES));
  } else {
    const int bs = particle_block(d.n);
    post_variant<false>(d, mode, mask, Fo, To, Bo, s, ev, dim3(blocks_for(d.i_hi - d.i_lo, bs)),
                        dim3(bs));
  }
  return hipGetLastError();
}

template <bool SPLIT>
static void kick_variant(const Dev& d, double* Bo, hipStream_t s, const hipEvent_t* ev, dim3 g, dim3 b) {
  if (d.ibm_u) {
    if (d.hm) launch_k(ev, k_kick<true, SPLIT, true>, g, b, s, d, Bo);
    else launch_k(ev, k_kick<false, SPLIT, true>, g, b, s, d, Bo);
  } else if (d.hm) {
    launch_k(ev, k_kick<true, SPLIT, false>, g, b, s, d, Bo);
  } else {
    launch_k(ev, k_kick<false, SPLIT, false>, g, b, s, d, Bo);
  }
}

hipError_t launch_kick(const Dev& d, double* Bo, hipStream_t s, const hipEvent_t* ev) {
  if (particle_split(d.n)) {
    kick_variant<true>(d, Bo, s, ev, dim3(blocks_for(d.i_hi - d.i_lo, 64)), dim3(64 * SPLIT_WAVES));
  } else {
    const int bs = particle_block(d.n);
    kick_variant<false>(d, Bo, s, ev, dim3(blocks_for(d.i_hi - d.i_lo, bs)), dim3(bs));
  }
  return hipGetLastError();
}

// Kinetic energy, translational plus rotational, of each member from the
// state's velocities: one block per member, fixed-order tree sum.
__global__ __launch_bounds__(256) void k_kinetic(Dev d, double* out) {
  __shared__ double red[256];
  const int mem = blockIdx.x;
  const int b = d.mrange[2 * mem], e = d.mrange[2 * mem + 1];
  const long N = d.n;
  double s = 0.0;
  for (int i = b + threadIdx.x; i < e; i += blockDim.x) {
    const V3<double> v = ld3(d.v, N, i), w = ld3(d.w, N, i);
    s += 0.5 * d.mass[i] * dot(v, v) + 0.5 * d.inertia[i] * dot(w, w);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[mem] = red[0];
}

// Positions of the listed particles, [n][3].
__global__ __launch_bounds__(256) void k_gather_x(Dev d, const int* idx, int n, double* out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const V3<double> x = ld3(d.x, d.n, idx[k]);
  out[3 * k] = x.x; out[3 * k + 1] = x.y; out[3 * k + 2] = x.z;
}

hipError_t launch_kinetic(const Dev& d, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_kinetic, dim3(d.M), dim3(256), 0, s, d, out);
  return hipGetLastError();
}

hipError_t launch_gather_x(const Dev& d, const int* idx, int n, double* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_x, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, idx, n, out);
  return hipGetLastError();
}

hipError_t launch_energy(const Dev& d, int max_member, double* Epart, double* out, hipStream_t s) {
  // Epart holds the [3][N] dipole field, [3][N] and [3][N] scratch, then the partial sums.
  double* Bd = Epart;
  double* part = Epart + 9 * d.n;
  hipError_t e = launch_post(d, POST_EVAL, 2, Bd + 3 * d.n, Bd + 6 * d.n, Bd, s);
  if (e != hipSuccess) return e;
  const dim3 g((unsigned)d.M, std::min(blocks_for(max_member, ENERGY_BLOCK), 4096u));
  hipLaunchKernelGGL(k_energy_part, g, dim3(ENERGY_BLOCK), 0, s, d, (const double*)Bd, part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_energy_reduce, dim3((unsigned)d.M, 9), dim3(64), 0, s, d, (const double*)part, out);
  return hipGetLastError();
}

}  // namespace rodmx
