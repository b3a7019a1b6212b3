// Near-field force (Sec. 2.1, Eq. 7-8, 10-11): erfc-screened Coulomb plus
// 12-6 Lennard-Jones over a cell list, with the core-shell random batch list.
//
// Full neighbour sums per particle i (cell order), no atomics, in one of
// these forms (pair_device.h; the rules and what they measured stand at
// group_most and launch_rbl):
//   k_pair_group      plain sums of few particles: 64 or 32 lanes share one,
//                     over its own trimmed stencil rows put end to end;
//   k_pair_queue      plain sums of many, FP64: one lane per particle,
//                     candidates filtered on packed 16-bit positions, the
//                     pairs that pass evaluated from queues in LDS;
//   k_pair_plain      plain sums of many, FP32C: one thread per particle
//                     walking the stencil rows of its own cell;
//   k_pair_rbl_group  random batch list, FP64: 64, 32 or 16 lanes per particle;
//   k_pair_rbl        random batch list of large FP64 systems and in FP32C: one
//                     wave per cluster of 8 consecutive particles. Lane l
//                     takes i = cluster[l / 8] and every 8th record of one
//                     candidate sequence shared by the wave (the union of the
//                     cluster's stencils), so the candidate loads are
//                     contiguous and the loop is uniform; the 8 partial sums
//                     of an i are added in a fixed order at the end.
//
// Species blocks: charged particles occupy keys [0, C), neutral ones
// [C, 2C). Coulomb terms only involve charged pairs, so without the random
// batch list a charged i walks the charged block out to r_coul and the
// neutral block out to r_lj; a neutral i walks both blocks out to r_lj.
//
// Random batch list (Eq. 10-11): every j within r_coul is classified with the
// squared distance computed without contraction (the same IEEE expression as
// the CPU oracle). Core terms (r^2 <= r_core^2) are summed exactly. Shell
// members (r_core^2 < r^2 <= r_coul^2) are counted, #S_i, and ranked by the
// 32-bit key of Eq. 11's batch: the batch B_i is the min(p, #S_i) members
// with the smallest keys, summed with the weight #S_i/|B_i|. Selection in one
// pass: keys below a threshold T are appended to a buffer in LDS.
// T is chosen so that about 3p keys fall below it for the mean shell size; if
// the buffer ends with fewer than min(p, #S_i) keys or overflows, a pass that
// only collects keys is repeated with T moved by bisection (keys are distinct,
// so some T always works). The batch is read back through the key's inverse
// (key -> id_j -> sorted slot) and its terms use the minimum image.
//
// Pair force on i: (kc q_i q_j G(r) + G_LJ(r)) d, d = r_i - r_j,
//   G(r)    = erfc(sqrt(a) r)/r^3 + 2 sqrt(a) exp(-a r^2)/(sqrt(pi) r^2),
//   G_LJ(r) = 24 eps (2 sigma^12/r^14 - sigma^6/r^8).
#include <algorithm>
#include <type_traits>

#include "pair_device.h"

namespace rbe {

struct PairCtx {
  PairParams pp;
  PairF32 pf;
  const double4 *__restrict__ xq;
  const int32_t *__restrict__ ids;
  const int32_t *__restrict__ cell_start;
  const int32_t *__restrict__ inv_id;
  double *__restrict__ fx;
  double *__restrict__ fy;
  double *__restrict__ fz;
  unsigned long long *__restrict__ counters;  // [4] when counting
  const int32_t *__restrict__ nq_ptr;         // charged count (device): [0, nq) charged, [nq, n) neutral
  int charged;                                // this launch: 1 the charged range, 0 the neutral range
  int group_plain;                            // plain sums: largest part of the group walk
  int64_t n;                                  // all particles
  // ghost shell (GHOST kernels only)
  const double4 *__restrict__ gxq;
  const int32_t *__restrict__ gid;
  const int32_t *__restrict__ gcell_start;
  // packed positions of both, and the squared reaches in their units (FP64)
  const uint2 *__restrict__ pk;
  const uint2 *__restrict__ gpk;
  double pk_scale;
  uint32_t t2_q, t2_lj;  // max(r_coul, r_lj), r_lj
  // random batch list: no pair outside r_coul up to t2_out, every one inside
  // it below t2_in; no pair inside r_core above t2_core
  uint32_t t2_out, t2_in, t2_core;
  int group_rbl;  // random batch list: largest part of the group form
};

// Cluster walk of one species block for a row group.
template <bool GHOST, bool WITH_ID, class Fn>
__device__ inline void walk(const PairCtx &c, int blk, int xa, int xb, int cy, int cz, const Sten &s, int b,
                            Fn &&fn) {
  auto no_tick = []() {};
  if (GHOST)
    cluster_walk_ghost<WITH_ID>(c.pp.g, c.cell_start, c.xq, c.ids, c.gcell_start, c.gxq, c.gid, (int)c.n, blk, xa, xb,
                                cy, cz, s, b, fn, no_tick);
  else
    cluster_walk<WITH_ID>(c.pp.g, c.cell_start, c.xq, c.ids, (int64_t)blk * c.pp.g.ncell, xa, xb, cy, cz, s, b, fn,
                          no_tick);
}

template <bool COUNT>
__device__ inline void flush_counts(const PairCtx &c, unsigned long long n_coul, unsigned long long n_lj,
                                    unsigned long long n_tested, unsigned long long n_shell) {
  if (COUNT) {
    atomicAdd(&c.counters[0], n_coul);
    atomicAdd(&c.counters[1], n_lj);
    atomicAdd(&c.counters[2], n_tested);
    atomicAdd(&c.counters[3], n_shell);
  }
}

// Particle range of this launch, read on the device (the charged count is the
// first neutral cell start), and the first particle of this block's share of
// per_block particles: the grid is sized for all n particles, blocks past the
// range's share exit at once, and the active blocks are spread over the XCDs
// (each XCD takes a contiguous run of the range).
__device__ inline bool part_block(const PairCtx &c, int per_block, int64_t *first, int64_t *end) {
  const int64_t nq = *c.nq_ptr;
  const int64_t a = c.charged ? 0 : nq, b = c.charged ? nq : c.n;
  const int64_t nb = (b - a + per_block - 1) / per_block;
  if ((int64_t)blockIdx.x >= nb) return false;
  *first = a + xcd_block(blockIdx.x, nb) * per_block;
  *end = b;
  return true;
}

// i-side data of a cluster lane.
struct ClusterI {
  int a, b;
  bool valid;
  int64_t i;
  double xi, yi, zi, qi;
  int cx, cy, cz;
};

__device__ inline ClusterI load_cluster_i(const PairCtx &c, int64_t first, int64_t end) {
  ClusterI r;
  const int lane = threadIdx.x;
  r.a = lane / kCJ;
  r.b = lane % kCJ;
  const int64_t i_raw = first + r.a;
  r.valid = i_raw < end;
  r.i = r.valid ? i_raw : end - 1;
  const double4 p = c.xq[r.i];
  r.xi = p.x;
  r.yi = p.y;
  r.zi = p.z;
  r.qi = p.w;
  const Grid &g = c.pp.g;
  r.cx = cell_coord(p.x, g.inv_h[0], g.nx);
  r.cy = cell_coord(p.y, g.inv_h[1], g.ny);
  r.cz = cell_coord(p.z, g.inv_h[2], g.nz);
  return r;
}

// Periodic or ghost-shell stencil walk of one particle (thread form).
template <bool GHOST, class Fn, class RowEnd>
__device__ inline void stencil(const PairCtx &c, int blk, int cx, int cy, int cz, const Sten &s, const double4 &p,
                               double r2, Fn &&fn, RowEnd &&row_end) {
  if (GHOST)
    for_stencil_ghost(c.pp.g, c.cell_start, c.xq, c.gcell_start, c.gxq, (int)c.n, blk, cx, cy, cz, s, p.x, p.y, p.z,
                      r2, fn, row_end);
  else
    for_stencil(c.pp.g, c.cell_start, c.xq, blk, cx, cy, cz, s, p.x, p.y, p.z, r2, fn, 0, row_end);
}

// Plain cutoff sums, one thread per particle i walking its own stencil (on
// MI355X this beats the cluster form when most candidates within reach are
// summed, i.e. without the shell test of the random batch list). MODE 0:
// neutral i (LJ over both species blocks out to r_lj); MODE 1: charged i
// (charged block out to max(r_coul, r_lj), neutral block out to r_lj); MODE
// 2: charged i, screened Coulomb terms only (charged block out to r_coul),
// added to f, which holds the LJ terms of the tile pass.
// The FP32C form: its pair terms are cheap beside a queue entry's fetch, so
// it evaluates each candidate where it finds it (6M ions 6.4 ms, as a queue
// walk 7.4; the FP64 form 12.3 and 9.8).
// Occupancy asked of the compiler: five (charged) or six (neutral) waves per
// SIMD, the most without spills once a row's partial sums are held.
template <bool COUNT, int MODE, bool GHOST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MODE ? 5 : 6)))
k_pair_plain(PairCtx c) {
  constexpr bool F32 = true;
  static_assert(MODE >= 0 && MODE <= 2, "mode");
  const int64_t nq = *c.nq_ptr;
  if ((MODE ? nq : c.n - nq) <= c.group_plain) return;  // too few particles: k_pair_group
  int64_t first, end;
  if (!part_block(c, blockDim.x, &first, &end)) return;
  const int64_t i = first + threadIdx.x;
  if (i >= end) return;
  const PairParams &pp = c.pp;
  const Grid &g = pp.g;
  const double4 pi4 = c.xq[i];
  const double xi = pi4.x, yi = pi4.y, zi = pi4.z, qi = pi4.w;
  const int cx = cell_coord(xi, g.inv_h[0], g.nx);
  const int cy = cell_coord(yi, g.inv_h[1], g.ny);
  const int cz = cell_coord(zi, g.inv_h[2], g.nz);
  ForceAcc<F32> acc;
  unsigned long long n_coul = 0, n_lj = 0, n_tested = 0;
  // Coulomb + LJ against charged j (block 0 of a charged i)
  auto visit_q = [&](int j, const double4 &pj, double shx, double shy, double shz) {
    const double dx = (xi - pj.x) - shx, dy = (yi - pj.y) - shy, dz = (zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    if (COUNT) ++n_tested;
    if (j == (int)i) return;  // ghosts are indexed from n on
    if (r2 <= pp.rq2) {
      acc.template add_row<true>(pp, c.pf, r2, qi, pj.w, dx, dy, dz);
      if (COUNT) {
        n_coul += (pp.do_coul && r2 <= pp.rc2);
        n_lj += (pp.do_lj && r2 <= pp.rlj2);
      }
    }
  };
  // LJ only (every other species pairing)
  auto visit_lj = [&](int j, const double4 &pj, double shx, double shy, double shz) {
    const double dx = (xi - pj.x) - shx, dy = (yi - pj.y) - shy, dz = (zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    if (COUNT) ++n_tested;
    if (j == (int)i) return;  // ghosts are indexed from n on
    if (r2 <= pp.rlj2) {
      acc.template add_row<false>(pp, c.pf, r2, qi, pj.w, dx, dy, dz);
      if (COUNT) n_lj += pp.do_lj;
    }
  };
  auto row_end = [&]() { acc.flush_row(); };
  if (MODE == 2) {
    // pp.do_lj is off for this launch: visit_q adds the screened Coulomb term only
    stencil<GHOST>(c, 0, cx, cy, cz, pp.s_coul, pi4, pp.rc2, visit_q, row_end);
    c.fx[i] += acc.get(0);
    c.fy[i] += acc.get(1);
    c.fz[i] += acc.get(2);
  } else {
    if (MODE == 1) {
      stencil<GHOST>(c, 0, cx, cy, cz, pp.s_coul, pi4, pp.rq2, visit_q, row_end);
      if (pp.do_lj) stencil<GHOST>(c, 1, cx, cy, cz, pp.s_lj, pi4, pp.rlj2, visit_lj, row_end);
    } else if (pp.do_lj) {
      stencil<GHOST>(c, 0, cx, cy, cz, pp.s_lj, pi4, pp.rlj2, visit_lj, row_end);
      stencil<GHOST>(c, 1, cx, cy, cz, pp.s_lj, pi4, pp.rlj2, visit_lj, row_end);
    }
    c.fx[i] = acc.get(0);
    c.fy[i] = acc.get(1);
    c.fz[i] = acc.get(2);
  }
  flush_counts<COUNT>(c, n_coul, n_lj, n_tested, 0);
}

// The FP64 form, one lane per particle (pair_device.h, queue walks), MODE 0
// and 1 as above. Bound by the issue of the FP64 pair terms and by the gather
// of the queued records. Against one thread evaluating each candidate as it
// meets it, 6M particles: ions 12.3 -> 9.8 ms, half-charged fluid 6.6 -> 5.5
// and (neutral part) 1.20 -> 1.05 ms, 10 % charged with ghosts 1.02 -> 0.86
// and 2.32 -> 1.97 ms.
template <bool COUNT, int MODE, bool GHOST>
__global__ void __launch_bounds__(kQueueThreads) __attribute__((amdgpu_waves_per_eu(4))) k_pair_queue(PairCtx c) {
  constexpr bool F32 = false;
  static_assert(MODE == 0 || MODE == 1, "mode");
  __shared__ uint32_t queue[kQueueCap * kQueueThreads];
  const int64_t nq = *c.nq_ptr;
  if ((MODE ? nq : c.n - nq) <= c.group_plain) return;  // too few particles: k_pair_group
  int64_t first, end;
  if (!part_block(c, blockDim.x, &first, &end)) return;
  const int64_t i = first + threadIdx.x;
  const bool active = i < end;  // the whole wave takes part
  const PairParams &pp = c.pp;
  const Grid &g = pp.g;
  const double4 pi = c.xq[active ? i : end - 1];
  ForceAcc<F32> acc;
  unsigned long long n_coul = 0, n_lj = 0, n_tested = 0;
  HitQueue Q(queue);
  const bool coded = c.n <= (1ll << kIndexBits);
  // an entry: the record, its exact classification, the pair term (COUL:
  // Coulomb and LJ; else LJ only)
  auto one = [&](uint32_t e, auto coul) {
    constexpr bool COUL = decltype(coul)::value;
    const uint32_t code = GHOST ? kNoShift : coded ? e >> kIndexBits : Q.now;
    const int j = (int)(GHOST || !coded ? e : e & ((1u << kIndexBits) - 1u));
    const double4 pj = GHOST && j >= c.n ? c.gxq[j - c.n] : c.xq[j];
    double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
    if (!GHOST && wave_count(code != kNoShift)) {
      dx -= code_shift(code, 0) * g.L[0];
      dy -= code_shift(code, 1) * g.L[1];
      dz -= code_shift(code, 2) * g.L[2];
    }
    const double r2 = sq_dist(dx, dy, dz);
    if ((r2 <= (COUL ? pp.rq2 : pp.rlj2)) & (j != (int)i)) {  // ghosts are indexed from n on
      acc.template add<COUL, true>(pp, c.pf, r2, pi.w, pj.w, dx, dy, dz);
      if (COUNT) {
        n_coul += (COUL && pp.do_coul && r2 <= pp.rc2);
        n_lj += (pp.do_lj && r2 <= pp.rlj2);
      }
    }
  };
  auto tested = [&](int len) {
    if (COUNT) n_tested += len;
  };
  auto walk = [&](auto coul, int blk, const Sten &s, double r2, uint32_t t2) {
    auto drain = [&](bool all) { drain_queue(Q, all, [&](uint32_t e) { one(e, coul); }); };
    queue_walk<GHOST>(g, c.cell_start + (int64_t)blk * g.ncell, c.pk,
                      GHOST ? c.gcell_start + (int64_t)blk * g.pncell : nullptr, c.gpk, (int)c.n, active, pi, s, r2,
                      t2, c.pk_scale, coded, Q, tested, drain);
    drain(true);
  };
  constexpr std::true_type coul_lj{};
  constexpr std::false_type lj_only{};
  if (MODE == 1) walk(coul_lj, 0, pp.s_coul, pp.rq2, c.t2_q);
  else if (pp.do_lj) walk(lj_only, 0, pp.s_lj, pp.rlj2, c.t2_lj);
  if (pp.do_lj) walk(lj_only, 1, pp.s_lj, pp.rlj2, c.t2_lj);
  if (active) {
    c.fx[i] = acc.get(0);
    c.fy[i] = acc.get(1);
    c.fz[i] = acc.get(2);
  }
  flush_counts<COUNT>(c, n_coul, n_lj, n_tested, 0);
}

// Plain cutoff sums of particles too few to fill the chip with one thread
// each: G lanes share one (pair_device.h, group walks). c.charged: 1 the
// charged range, 0 the neutral one, 2 both; coulomb: the charged range's
// screened Coulomb terms only, added to f. Small launches are bound by the
// latency of a particle's chain of loads, large ones by the issue of the pair
// terms (about half the lanes hold a pair inside the cutoff): 2,000 ions out
// to r = 8 in FP64 13 us (422 us as one thread each), 50,000 147 us (357).
template <bool F32, bool COUNT, bool GHOST, int G>
__global__ void __launch_bounds__(256) k_pair_group(PairCtx c, int coulomb) {
  __shared__ GroupRows<G> rows[256 / G];
  __shared__ GroupTerms<F32 ? G : 1> terms[256 / G];
  const int64_t nq = *c.nq_ptr;
  const int64_t a = c.charged ? 0 : nq, end = c.charged == 1 ? nq : c.n;
  if (end - a > c.group_plain) return;  // enough particles: k_pair_plain or k_pair_queue
  const int64_t per = (end - a + gridDim.x - 1) / gridDim.x;  // consecutive particles per block
  const int64_t first = a + blockIdx.x * per, last = min(end, first + per);
  const PairParams &pp = c.pp;
  unsigned long long n_coul = 0, n_lj = 0, n_tested = 0;
  for (int64_t i = first + threadIdx.x / G; i < last; i += 256 / G) {  // the lanes of a group together
    const double4 pi4 = c.xq[i];
    ForceAcc<F32> acc;
    group_sums<F32, GHOST, G>(
        pp, c.pf, pp.g, pp.s_coul, pp.s_lj, c.cell_start, c.xq, c.gcell_start, c.gxq, (int)c.n, (int)i, pi4,
        coulomb != 0, rows[threadIdx.x / G], &terms[threadIdx.x / G].t[0], acc, [&](bool coul, bool other, double r2) {
          if (COUNT) {
            ++n_tested;
            n_coul += (other && coul && pp.do_coul && r2 <= pp.rc2);
            n_lj += (other && !coulomb && pp.do_lj && r2 <= pp.rlj2);
          }
        });
    const double f0 = acc.template total<G>(0), f1 = acc.template total<G>(1), f2 = acc.template total<G>(2);
    if (threadIdx.x % G == 0) {
      if (coulomb) {
        c.fx[i] += f0;
        c.fy[i] += f1;
        c.fz[i] += f2;
      } else {
        c.fx[i] = f0;
        c.fy[i] = f1;
        c.fz[i] = f2;
      }
    }
  }
  flush_counts<COUNT>(c, n_coul, n_lj, n_tested, 0);
}

// Random batch list (Eq. 10-11) for the particles of the launch range: exact
// core, counted and ranked shell, one walk of both species blocks out to
// r_coul.
// QSHELL: the shell holds charged particles only (variant of Eq. 10; the
// neutral j beyond the core then carry no force, since r_lj <= r_core).
// EITHER: the group form was launched as well, for parts of up to group_rbl.
template <bool F32, bool COUNT, bool GHOST, bool QSHELL, bool EITHER>
__global__ void __launch_bounds__(64, 5) k_pair_rbl(PairCtx c) {
  __shared__ uint32_t kbuf[kCI * kShellCap];
  __shared__ uint32_t ksel[kCI * RBE_MAX_SHELL_BATCH];
  __shared__ int kcnt[kCI];
  int64_t first, end;
  if (EITHER && (c.charged ? *c.nq_ptr : c.n - *c.nq_ptr) <= c.group_rbl) return;
  if (!part_block(c, kCI, &first, &end)) return;
  const ClusterI I = load_cluster_i(c, first, end);
  const PairParams &pp = c.pp;
  const Grid &g = pp.g;
  const int p = pp.p_shell;
  const ShellKey sk = shell_key_of(pp.shell_key, c.ids[I.i]);
  ForceAcc<F32> acc;
  unsigned long long n_coul = 0, n_lj = 0, n_tested = 0;
  int ns = 0;  // shell members seen by this lane
  // keys below T are collected; the mean shell of the charged-only variant
  // holds charged particles, whose count is known on the device only
  uint64_t T = QSHELL ? shell_first_threshold(pp, *c.nq_ptr) : pp.shell_T0;
  bool in_group = false;
  if (I.b == 0) kcnt[I.a] = 0;
  __syncthreads();
  auto collect = [&](uint32_t k) {
    if ((uint64_t)k < T) {
      const int s = atomicAdd(&kcnt[I.a], 1);
      if (s < kShellCap) kbuf[I.a * kShellCap + s] = k;
    }
  };
  auto visit = [&](bool ok, int j, const double4 &pj, int idj, double shx, double shy, double shz) {
    const double dx = (I.xi - pj.x) - shx, dy = (I.yi - pj.y) - shy, dz = (I.zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    // flat predicates (bitwise, so no branch per condition)
    // j indexes natives, or ghosts offset by n: only i itself has j == i (its
    // periodic images lie at least L >= 2 r_coul away)
    const bool live = ok & in_group & (j != (int)I.i);
    const bool core = live & (r2 <= pp.rcore2);
    const bool shell = live & (r2 > pp.rcore2) & (r2 <= pp.rc2) & (!QSHELL | (pj.w != 0.0));
    if (COUNT) n_tested += ok & in_group;
    if (core) {
      acc.template add<true, true>(pp, c.pf, r2, I.qi, pj.w, dx, dy, dz);
      if (COUNT) {
        n_coul += (pp.do_coul && I.qi != 0.0 && pj.w != 0.0);
        n_lj += (pp.do_lj && r2 <= pp.rlj2);
      }
    }
    ns += shell;
    if (shell) collect(shell_rank(sk, idj));
  };
  auto visit_collect = [&](bool ok, int, const double4 &pj, int idj, double shx, double shy, double shz) {
    const double dx = (I.xi - pj.x) - shx, dy = (I.yi - pj.y) - shy, dz = (I.zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    if (ok & in_group & (r2 > pp.rcore2) & (r2 <= pp.rc2) & (!QSHELL | (pj.w != 0.0)))
      collect(shell_rank(sk, idj));
  };
  const int64_t rowkey = (int64_t)I.cz * g.ny + I.cy;
  auto walk_all = [&](bool active, auto &&fn) {
    for_each_row_group(active, rowkey, I.cx, [&](bool in, int leader, int xa, int xb) {
      in_group = in;
      const int cy = __shfl(I.cy, leader, 64), cz = __shfl(I.cz, leader, 64);
      walk<GHOST, true>(c, 0, xa, xb, cy, cz, pp.s_coul, I.b, fn);
      // with a charged-only shell the neutral block matters inside the core
      // only (r_lj <= r_core): its walk covers r_core instead of r_coul
      walk<GHOST, true>(c, 1, xa, xb, cy, cz, QSHELL ? pp.s_core : pp.s_coul, I.b, fn);
    });
  };
  walk_all(I.valid, visit);
  __syncthreads();
  const int m = sum_j_lanes(ns);  // #S_i
  const int need = m < p ? m : p;
  int got = kcnt[I.a];
  // bisection on T when the buffer missed [need, cap] (rare; distinct keys
  // end it within 33 rounds, the bound only guards against duplicate ids,
  // which the inverse id map reports)
  uint64_t lo = 0, hi = 1ull << 32;
  bool pend = I.valid && need > 0 && (got < need || got > kShellCap);
  for (int round = 0; __any(pend) && round < 40; ++round) {
    if (pend) {
      if (got < need) lo = T;
      else hi = T;
      T = (m <= kShellCap) ? (1ull << 32) : lo + (hi - lo) / 2;
    }
    __syncthreads();
    if (pend && I.b == 0) kcnt[I.a] = 0;
    __syncthreads();
    walk_all(pend, visit_collect);
    __syncthreads();
    if (pend) got = kcnt[I.a];
    pend = pend && (got < need || got > kShellCap);
  }
  got = min(got, kShellCap);
  const int nb = min(need, got);  // = need unless ids repeat
  // ranks of the collected keys (distinct); the first `need` form the batch
  if (I.valid && nb > 0) {
    const uint32_t *kb = kbuf + I.a * kShellCap;
    for (int t = I.b; t < got; t += kCJ) {
      const uint32_t k = kb[t];
      int rank = 0;
      for (int u = 0; u < got; ++u) rank += kb[u] < k;
      if (rank < nb) ksel[I.a * RBE_MAX_SHELL_BATCH + rank] = k;
    }
  }
  __syncthreads();
  ForceAcc<F32> sh;
  if (I.valid) {
    for (int r = I.b; r < nb; r += kCJ) {
      const int32_t idj = shell_id_of(sk, ksel[I.a * RBE_MAX_SHELL_BATCH + r]);
      if ((uint32_t)idj >= (uint32_t)c.n) continue;  // bad ids (flagged by the inverse map)
      const int j = c.inv_id[idj];
      if ((uint32_t)j >= (uint32_t)c.n) continue;
      const double4 pj = c.xq[j];
      const double dx = min_image(I.xi - pj.x, g.L[0]);
      const double dy = min_image(I.yi - pj.y, g.L[1]);
      const double dz = min_image(I.zi - pj.z, g.L[2]);
      const double r2 = sq_dist(dx, dy, dz);
      sh.template add<true, true>(pp, c.pf, r2, I.qi, pj.w, dx, dy, dz);
      if (COUNT) {
        n_coul += (pp.do_coul && I.qi != 0.0 && pj.w != 0.0);
        n_lj += (pp.do_lj && r2 <= pp.rlj2);
      }
    }
  }
  double f0 = sum_j_lanes(acc.get(0)), f1 = sum_j_lanes(acc.get(1)), f2 = sum_j_lanes(acc.get(2));
  const double s0 = sum_j_lanes(sh.get(0)), s1 = sum_j_lanes(sh.get(1)), s2 = sum_j_lanes(sh.get(2));
  if (nb > 0) {
    const double scale = (double)m / (double)nb;
    f0 = fma(scale, s0, f0);
    f1 = fma(scale, s1, f1);
    f2 = fma(scale, s2, f2);
  }
  if (I.valid && I.b == 0) {
    c.fx[I.i] = f0;
    c.fy[I.i] = f1;
    c.fz[I.i] = f2;
  }
  flush_counts<COUNT>(c, n_coul, n_lj, n_tested, I.b == 0 && I.valid ? (unsigned long long)m : 0ull);
}

// Random batch list, FP64 group form: G lanes per particle (pair_device.h,
// group walks). The candidates are read as packed positions and ids, 12 bytes
// each, and classified by integer distances: sure shell members are counted
// and keyed without their FP64 record; those in the core, or within the grid's
// rounding of either radius, go to a list that is classified exactly and
// evaluated G at a time. Counts, places and the batch selection are ballots,
// so nothing is atomic: the batch is the keys below a threshold that is moved
// until exactly `need` lie below it.
// Bound by issue: the key hash and the ballots' bookkeeping, about 80
// instructions a trip; the cluster form spends 35 per candidate on a stencil
// that holds 4.3 candidates per shell member, the trimmed rows about 2. What
// it gains is the lanes: 20,000 electrolyte 250 -> 73 us, 1M 1.40 -> 1.35 ms.
template <int G>
struct RblLists {
  uint2 near[kGroupList<G> + G];  // records to classify exactly: index, row code (sign bit: ghost)
  uint32_t key[kShellCap];        // shell keys below the threshold
  uint32_t sel[RBE_MAX_SHELL_BATCH];
};
template <bool COUNT, bool GHOST, bool QSHELL, int G, bool EITHER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_pair_rbl_group(PairCtx c) {
  __shared__ GroupRows<G> rows_lds[256 / G];
  __shared__ RblLists<G> lists[256 / G];
  const int64_t nq = *c.nq_ptr;
  const int64_t a = c.charged ? 0 : nq, end = c.charged ? nq : c.n;
  if (EITHER && end - a > c.group_rbl) return;  // k_pair_rbl
  const int64_t per = (end - a + gridDim.x - 1) / gridDim.x;  // consecutive particles per block
  const int64_t first = a + xcd_block(blockIdx.x, gridDim.x) * per, last = min(end, first + per);
  const int sub = threadIdx.x & (G - 1);
  GroupRows<G> &rows = rows_lds[threadIdx.x / G];
  RblLists<G> &Ls = lists[threadIdx.x / G];
  const PairParams &pp = c.pp;
  const Grid &g = pp.g;
  const int p = pp.p_shell;
  unsigned long long n_coul = 0, n_lj = 0, n_tested = 0, n_shell = 0;
  for (int64_t i = first + threadIdx.x / G; i < last; i += 256 / G) {  // the lanes of a group together
    const double4 pi = c.xq[i];
    const ShellKey sk = shell_key_of(pp.shell_key, c.ids[i]);
    const uint2 home = pack_position(pi.x, pi.y, pi.z, c.pk_scale);
    ForceAcc<false> acc;
    uint64_t T = QSHELL ? shell_first_threshold(pp, *c.nq_ptr) : pp.shell_T0, lo = 0, hi = 1ull << 32;
    int m = 0, got = 0, need = 0;  // the same in all lanes of the group
    struct Cand {
      uint2 pk;
      int id;
    };
    // keys of the lanes with `in` that lie below T join the list
    auto collect = [&](bool in, uint32_t key) {
      const bool take = in & (key <= (uint32_t)(T - 1));  // 0 < T <= 2^32
      const uint64_t who = group_ballot<G>(take);
      const int at = got + bits_below<G>(who);
      if (take & (at < kShellCap)) Ls.key[at] = key;
      got += __popcll(who);
    };
    // with a charged-only shell the neutral block matters inside the core only
    // (r_lj <= r_core)
    const Block A{pp.s_coul, pp.rc2};
    const Block B = QSHELL ? Block{pp.s_core, fmax(pp.rcore2, pp.rlj2)} : A;
    for (int round = 0; round < 40; ++round) {
      // round 0 sums the core, counts the shell and collects its keys; the
      // rounds after it (the list missed [need, kShellCap]; rare) collect only
      int nn = 0;
      got = 0;
      auto classify = [&](int from, int cnt) {
        wave_sync();
        bool shell = false;
        uint32_t key = 0;
        if (sub < cnt) {
          const uint2 e = Ls.near[from + sub];
          const bool ghost = GHOST && (int)e.y < 0;
          const int j = (int)e.x, code = (int)(e.y & 0x7FFFFFFFu);
          const double4 pj = ghost ? c.gxq[j] : c.xq[j];
          double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
          if (!GHOST && code > 1) {
            dx -= row_shift(code, 0) * g.L[0];
            dy -= row_shift(code, 1) * g.L[1];
            dz -= row_shift(code, 2) * g.L[2];
          }
          const double r2 = sq_dist(dx, dy, dz);
          const bool live = ghost || j != (int)i;
          if (live && r2 <= pp.rcore2) {
            if (round == 0) {
              acc.template add<true, true>(pp, c.pf, r2, pi.w, pj.w, dx, dy, dz);
              if (COUNT) {
                n_coul += (pp.do_coul && pi.w != 0.0 && pj.w != 0.0);
                n_lj += (pp.do_lj && r2 <= pp.rlj2);
              }
            }
          } else if (live && r2 <= pp.rc2 && (!QSHELL || pj.w != 0.0)) {
            shell = true;
            key = shell_rank(sk, ghost ? c.gid[j] : c.ids[j]);
          }
        }
        if (round == 0) m += __popcll(group_ballot<G>(shell));
        collect(shell, key);
        wave_sync();
      };
      group_list<G, GHOST, 2>(
          g, c.cell_start, c.gcell_start, pi, A, B, rows,
          [&](int j, bool ghost) {
            return Cand{ghost ? c.gpk[j] : c.pk[j], ghost ? c.gid[j] : c.ids[j]};
          },
          [&](bool ok, int, int j, int code, bool ghost, bool shifted, const Cand &f) {
            uint2 own = home;
            if (shifted && code > 1)
              own = pack_position(pi.x - row_shift(code, 0) * g.L[0], pi.y - row_shift(code, 1) * g.L[1],
                                  pi.z - row_shift(code, 2) * g.L[2], c.pk_scale);
            const uint32_t d2 = packed_dist2(own.x, own.y, f.pk.x, f.pk.y);
            if (COUNT) n_tested += ok && round == 0;
            const bool in = ok & (d2 <= c.t2_out);
            const bool sure = in & (d2 > c.t2_core) & (d2 < c.t2_in);
            // (QSHELL: a neutral record beyond the core is no shell member)
            const bool shell = sure & (!QSHELL | ((code & 1) == 0));
            const uint64_t who = group_ballot<G>(in & !sure);
            if (who) {
              if (in & !sure)
                Ls.near[nn + bits_below<G>(who)] = make_uint2((uint32_t)j, (uint32_t)code | (ghost ? 0x80000000u : 0u));
              nn += __popcll(who);
            }
            if (round == 0) m += __popcll(group_ballot<G>(shell));
            collect(shell, shell_rank(sk, f.id));
          },
          [&](int, int) {
            // whole batches of the chunk's records; the rest joins the next chunk's
            int done = 0;
            for (; nn - done >= G; done += G) classify(done, G);
            if (done) {
              const uint2 rest = Ls.near[done + sub];
              nn -= done;
              wave_sync();
              if (sub < nn) Ls.near[sub] = rest;
              wave_sync();
            }
          },
          [](uint64_t) {});
      classify(0, nn);
      if (round == 0) need = min(m, p);
      if (need == 0 || (got >= need && got <= kShellCap)) break;
      // bisection on T (distinct keys end it within 33 rounds; the bound only
      // guards against duplicate ids, which the inverse id map reports)
      if (got < need) lo = T;
      else hi = T;
      T = m <= kShellCap ? 1ull << 32 : lo + (hi - lo) / 2;
    }
    // the `need` smallest of the keys: those below X
    got = min(got, kShellCap);
    const int nb = min(need, got);  // = need unless ids repeat
    constexpr int KL = kShellCap / G;  // keys per lane
    wave_sync();
    uint32_t mine[KL];
    bool held[KL];
#pragma unroll
    for (int u = 0; u < KL; ++u) {
      held[u] = sub + G * u < got;
      mine[u] = held[u] ? Ls.key[sub + G * u] : 0u;
    }
    auto count_below = [&](uint64_t X) {
      int n = 0;
#pragma unroll
      for (int u = 0; u < KL; ++u) n += __popcll(group_ballot<G>(held[u] && (uint64_t)mine[u] < X));
      return n;
    };
    // `need` of them lie below X: found by interpolation (the keys are uniform
    // below T), with every other step a bisection so that it ends in any case
    uint64_t X = T;
    if (got > nb) {
      uint64_t xl = 0, xh = T;
      int nl = 0, nh = got;
      for (int k = 0; k < 66 && xh - xl > 1; ++k) {
        const uint64_t w = xh - xl;
        X = xl + ((k & 1) ? w / 2 : (uint64_t)((float)w * ((float)(nb - nl) / (float)(nh - nl))));
        if (X <= xl) X = xl + 1;
        if (X >= xh) X = xh - 1;
        const int n = count_below(X);
        if (n == nb) break;
        if (n < nb) {
          xl = X;
          nl = n;
        } else {
          xh = X;
          nh = n;
        }
        X = xh;
      }
    }
    int at = 0;
#pragma unroll
    for (int u = 0; u < KL; ++u) {
      const bool in = held[u] && (uint64_t)mine[u] < X;
      const uint64_t who = group_ballot<G>(in);
      const int k = at + bits_below<G>(who);
      if (in && k < nb) Ls.sel[k] = mine[u];
      at += __popcll(who);
    }
    wave_sync();
    ForceAcc<false> sh;
    for (int r = sub; r < nb; r += G) {
      const int32_t idj = shell_id_of(sk, Ls.sel[r]);
      if ((uint32_t)idj >= (uint32_t)c.n) continue;  // bad ids (flagged by the inverse map)
      const int j = c.inv_id[idj];
      if ((uint32_t)j >= (uint32_t)c.n) continue;
      const double4 pj = c.xq[j];
      const double dx = min_image(pi.x - pj.x, g.L[0]);
      const double dy = min_image(pi.y - pj.y, g.L[1]);
      const double dz = min_image(pi.z - pj.z, g.L[2]);
      const double r2 = sq_dist(dx, dy, dz);
      sh.template add<true, true>(pp, c.pf, r2, pi.w, pj.w, dx, dy, dz);
      if (COUNT) {
        n_coul += (pp.do_coul && pi.w != 0.0 && pj.w != 0.0);
        n_lj += (pp.do_lj && r2 <= pp.rlj2);
      }
    }
    // f = core + (#S_i / |B_i|) shell
    const double scale = nb > 0 ? (double)m / (double)nb : 0.0;
    const double f0 = group_sum<G>(fma(scale, sh.get(0), acc.get(0))),
                 f1 = group_sum<G>(fma(scale, sh.get(1), acc.get(1))),
                 f2 = group_sum<G>(fma(scale, sh.get(2), acc.get(2)));
    if (sub == 0) {
      // (a non-finite position is within no reach of anything)
      const bool here = __builtin_isfinite(pi.x + pi.y + pi.z);
      c.fx[i] = here ? f0 : 0.0;
      c.fy[i] = here ? f1 : 0.0;
      c.fz[i] = here ? f2 : 0.0;
    }
    if (sub == 0) n_shell += (unsigned long long)m;
  }
  flush_counts<COUNT>(c, n_coul, n_lj, n_tested, n_shell);
}

PairF32 make_pair_f32(const PairParams &pp) {
  PairF32 pf;
  pf.sqrt_alpha = (float)pp.sqrt_alpha;
  pf.neg_alpha_log2e = (float)(-pp.alpha * 1.4426950408889634074);
  pf.two_sqrt_alpha_over_sqrt_pi = (float)pp.two_sqrt_alpha_over_sqrt_pi;
  pf.kc = (float)pp.kc;
  pf.eps24 = (float)pp.eps24;
  pf.sig2 = (float)pp.sig2;
  return pf;
}

// Random batch list of a part. FP32C: the cluster form, whose lanes add their
// terms in its own order. FP64: the group form, 64 lanes per particle, or 32
// and 16 where the mean shell would leave most of 64 without a candidate or
// there are waves enough with fewer, up to the size from which the cluster
// form's waves fill the chip. A whole force call in us with 64, 32 and 16 lanes
// and clusters, all charged unless said (m: particles within r_coul):
//   wide shells    50,000, m = 60 195, 164, 146, 200; 300: 264, 251, 239, 295;
//                  200,000, 60: 561, 442, 425, 471; 300: 781, 714, 780, 713;
//                  1M, 60: 2679, 2011, 1848, 1991; 300: 3697, 3212, 3372, 3000;
//                  a quarter charged, m = 724 50,000: 217, 245, 320, 376;
//                  200,000: 542, 551, 610, 682; 500,000: 1107, 1082, 1158, 1203;
//                  1M, 300: 1408, 1315, 1318, 1498
//   narrow shells  3,000, m = 25 74, 76, 82, 145; 8,000: 68, 62, 66, 104;
//                  50,000, 45: 192, 161, 140, 190; 100,000, 25: 291, 240, 233, 242
// What counts for wide shells is the part, whose size is known on the device
// only: between kRblWide32 and kRblEither particles both kernels are launched,
// and one of them exits (the clusters' blocks in 9 us at 280,000, 26 at 1M;
// beyond, that costs as much as it gains). Shells so full that 64 lanes are
// busy keep them longer.
// The clusters' candidates come in few long rows where the cells are hardly
// wider than the reach (9 rows of them; the default grid with r_lj = r_coul),
// and they win sooner there, by most where the density varies. 32 lanes and
// clusters, parts of 70,000, m = 60: 208, 199; 200: 300, 312; 100,000: 264, 237
// and 392, 411, half charged 454, 438 and 715, 672; 200,000: 443, 388 and 671,
// 642; 138,000 in a box that they fill to an eighth, half charged: 3796, 3100
// and 11906, 10077. Cells from 1.3 times the reach on are as the narrow ones:
// parts of 140,000, m = 300, half charged, 1.05: 1243, 1113; 1.3: 1444, 1584;
// 1.6: 1853, 2349; 0.85 (m = 200): 965, 1380. 64 lanes, 32 and clusters there,
// half charged, 30,000, m = 200: 185, 190, 282; 500: 270, 321, 470; 60,000,
// 60: 230, 177, 221; 200: 303, 262, 351; LJ alone with ghosts, 57,000, 110:
// 261, 221, 198.
constexpr double kRblWide = 48.0, kRblFull = 500.0;  // particles within r_coul of one, on average
constexpr int64_t kRblWide64 = 65536, kRblFull64 = 393216, kRblWide32 = 262144, kRblEither = 1 << 20;
constexpr int64_t kRblTight64 = 32768, kRblTight32 = 65536;
static bool rbl_tight(const PairParams &pp) {
  return pp.s_coul.y == 1 && pp.s_coul.z == 1 && 1.44 * pp.rq2 * pp.g.inv_h[1] * pp.g.inv_h[2] >= 1.0;
}
constexpr int64_t kRblNarrow32 = 8192, kRblNarrow16 = 65536;
template <bool F32, bool COUNT, bool GHOST, bool QSHELL>
static void launch_rbl(PairCtx c, hipStream_t st) {
  const double mean = mean_within(c.pp.g, c.n, std::sqrt(c.pp.rc2));
  const bool wide = mean >= kRblWide, tight = rbl_tight(c.pp);
  const int64_t wide32 = tight ? kRblTight32 : kRblWide32;
  const unsigned clusters = (unsigned)((c.n + kCI - 1) / kCI);
  if constexpr (F32) {
    k_pair_rbl<F32, COUNT, GHOST, QSHELL, false><<<clusters, 64, 0, st>>>(c);
  } else if (c.n > (wide ? kRblEither : kRblNarrow16)) {
    k_pair_rbl<F32, COUNT, GHOST, QSHELL, false><<<clusters, 64, 0, st>>>(c);
  } else if (wide && c.n <= (tight ? kRblTight64 : mean >= kRblFull ? kRblFull64 : kRblWide64)) {
    k_pair_rbl_group<COUNT, GHOST, QSHELL, 64, false><<<group_blocks(c.n, 64), 256, 0, st>>>(c);
  } else if (c.n <= (wide ? wide32 : kRblNarrow32)) {
    k_pair_rbl_group<COUNT, GHOST, QSHELL, 32, false><<<group_blocks(c.n, 32), 256, 0, st>>>(c);
  } else if (wide) {
    c.group_rbl = (int)wide32;
    k_pair_rbl_group<COUNT, GHOST, QSHELL, 32, true><<<group_blocks(wide32, 32), 256, 0, st>>>(c);
    k_pair_rbl<F32, COUNT, GHOST, QSHELL, true><<<clusters, 64, 0, st>>>(c);
  } else {
    k_pair_rbl_group<COUNT, GHOST, QSHELL, 16, false><<<group_blocks(c.n, 16), 256, 0, st>>>(c);
  }
}

// Plain sums of a part (c.charged): one thread per particle, or a group of
// lanes when the part is small (group_most). Whether a part of a large system
// is small is known on the device only, so both kernels are launched then and
// one of them exits at once (about 3 us beside a walk of hundreds). A group has
// 64 lanes in systems of up to 8,192 particles, whatever their parts (25,000
// charged: 64 lanes 86 us, 32 88), and 32 in larger ones.
static int64_t plain_group_most(bool f32, bool charged, const PairParams &pp, int64_t n) {
  return group_most(f32, charged, mean_within(pp.g, n, std::sqrt(charged ? pp.rq2 : pp.rlj2)));
}
template <bool F32, bool COUNT, int MODE, bool GHOST>
static void launch_plain(PairCtx c, hipStream_t st) {
  c.group_plain = (int)(c.charged == 2 ? c.n : plain_group_most(F32, MODE, c.pp, c.n));
  const int64_t most = std::min<int64_t>(c.n, c.group_plain);
  if (c.n <= 8192)
    k_pair_group<F32, COUNT, GHOST, 64><<<group_blocks(most, 64), 256, 0, st>>>(c, MODE == 2);
  else
    k_pair_group<F32, COUNT, GHOST, 32><<<group_blocks(most, 32), 256, 0, st>>>(c, MODE == 2);
  if (c.n <= c.group_plain) return;
  const unsigned blocks = (unsigned)((c.n + 255) / 256);
  if constexpr (F32) k_pair_plain<COUNT, MODE, GHOST><<<blocks, 256, 0, st>>>(c);
  else k_pair_queue<COUNT, MODE, GHOST><<<blocks, kQueueThreads, 0, st>>>(c);
}

// Charged particles occupy [0, nq) of the sorted order, neutral ones [nq, n).
// With the random batch list the charged particles take the RBL kernel; the
// neutral ones too when r_lj > r_core (their LJ terms then reach the shell),
// else their sums are plain (every LJ term lies in the core).
// part: PAIR_PART_CHARGED, PAIR_PART_SHELL (nothing left to do: the shell is
// fused into the charged part), PAIR_PART_NEUTRAL, PAIR_PART_COULOMB or
// PAIR_PART_BOTH.
template <bool F32, bool COUNT, bool GHOST>
static void launch_part(PairCtx c, int part, hipStream_t st) {
  const PairParams pp = c.pp;
  if (part == PAIR_PART_CHARGED) {
    c.charged = 1;
    if (pp.rbl && pp.shell_charged) launch_rbl<F32, COUNT, GHOST, true>(c, st);
    else if (pp.rbl) launch_rbl<F32, COUNT, GHOST, false>(c, st);
    else launch_plain<F32, COUNT, 1, GHOST>(c, st);
  } else if (part == PAIR_PART_COULOMB) {
    c.charged = 1;
    c.pp.do_lj = 0;
    if constexpr (F32) launch_plain<F32, COUNT, 2, GHOST>(c, st);  // the tile pass is FP32C
  } else if (part == PAIR_PART_NEUTRAL) {
    c.charged = 0;
    if (pp.rbl && pp.rlj2 > pp.rcore2 && pp.do_lj) launch_rbl<F32, COUNT, GHOST, false>(c, st);
    else launch_plain<F32, COUNT, 0, GHOST>(c, st);
  } else if (part == PAIR_PART_BOTH) {
    c.charged = 2;
    launch_plain<F32, COUNT, 0, GHOST>(c, st);
  }
}

bool pair_grouped(int prec, const PairParams &pp, int64_t n) {
  const bool f32 = prec == RBE_FP32C;
  return n <= std::min(plain_group_most(f32, true, pp, n), pp.do_lj ? plain_group_most(f32, false, pp, n) : 65536);
}

template <bool GHOST>
static void launch_prec(int prec, PairCtx c, int part, hipStream_t st) {
  if (prec == RBE_FP32C) {
    if (c.counters) launch_part<true, true, GHOST>(c, part, st);
    else launch_part<true, false, GHOST>(c, part, st);
  } else {
    if (c.counters) launch_part<false, true, GHOST>(c, part, st);
    else launch_part<false, false, GHOST>(c, part, st);
  }
}

void launch_pair(int prec, int part, const PairParams &pp, int64_t n, const int32_t *nq, const Sorted &s,
                 const int32_t *cell_start, const int32_t *inv_id, const GhostBuffers *gb, double *fx, double *fy,
                 double *fz, PairCounters cnt, hipStream_t st) {
  if (n <= 0) return;
  PairCtx c;
  c.pp = pp;
  c.pf = make_pair_f32(pp);
  c.xq = s.xq;
  c.ids = s.id;
  c.cell_start = cell_start;
  c.inv_id = inv_id;
  c.fx = fx;
  c.fy = fy;
  c.fz = fz;
  c.counters = cnt.c;
  c.n = n;
  c.nq_ptr = nq;
  c.charged = part == PAIR_PART_CHARGED;
  c.gxq = gb ? gb->xq : nullptr;
  c.gid = gb ? gb->id : nullptr;
  c.gcell_start = gb ? gb->cell_start : nullptr;
  c.pk = s.pk;
  c.gpk = gb ? gb->pk : nullptr;
  c.pk_scale = s.pk_scale;
  c.t2_q = pack_reach2(std::sqrt(pp.rq2), s.pk_scale);
  c.t2_lj = pack_reach2(std::sqrt(pp.rlj2), s.pk_scale);
  c.t2_out = pack_reach2(std::sqrt(pp.rc2), s.pk_scale);
  c.t2_in = pack_inside2(std::sqrt(pp.rc2), s.pk_scale);
  c.t2_core = pack_reach2(std::sqrt(std::max(pp.rcore2, 0.0)), s.pk_scale);
  if (gb) launch_prec<true>(prec, c, part, st);
  else launch_prec<false>(prec, c, part, st);
}

}  // namespace rbe
