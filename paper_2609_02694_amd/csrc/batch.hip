// Batched form: many independent systems ("replicas") of uneven size advanced
// together.
//
// All replicas live in concatenated arrays; replica r owns particles
// [p0, p0 + n) and binning keys [c0, c0 + 2 C_r) (its charged cells, then its
// neutral cells), so one counting sort, one launch per pass, serves every
// replica:
//
//   half-kick + drift + wrap, binning keys + histogram, and the mode samples
//     of every replica (Eq. 9)                              k_batch_drift
//   scan, scatter and stable placement of the keys          bin.hip
//   reorder of the state, packing of the sorted records     k_batch_reorder
//   near field of every particle                            k_batch_near*
//   structure-factor partials (chunk x mode)                k_batch_rho
//   structure factors: fixed-order sums of the partials     k_batch_rho_final
//   Fourier gather + second half-kick                       k_batch_gather
//
// Plain launches: a launch boundary costs 2-4 us here, while a barrier across
// the resident blocks of one persistent kernel cost about 40 us (every block's
// arrival is an atomic on one address, seen from eight L2s), and each pass
// then has the registers, and so the waves per SIMD, of its own code. The
// passes other than the near field took 715 us of a step of 24 replicas
// (150,000 particles, FP64) and 2,150 us of one of 256 (3.4M, FP32C) as two
// persistent launches, 100 and 580 us as these.
#include "fourier_device.h"
#include "pair_device.h"
#include "sampler_device.h"

namespace rbe {

constexpr int kBatchThreads = 256;

// ---------------------------------------------------------------------------
// drift, keys and mode samples
// ---------------------------------------------------------------------------
// Blocks [0, nb): one thread per particle. mode 0: v += h f, x <- wrap(x + dt
// v) in place; both modes: the binning key of the (wrapped) position, its run
// slot and the histogram (count, cleared before; nullptr: the key alone).
// Blocks from nb on: one thread per (replica, mode) of evaluation `eval`.
__global__ void __launch_bounds__(kBatchThreads) k_batch_drift(BatchArgs a, uint64_t eval, unsigned nb,
                                                               int32_t *count) {
  if (blockIdx.x >= nb) {
    const int64_t it = (blockIdx.x - nb) * (int64_t)kBatchThreads + threadIdx.x;
    if (it >= (int64_t)a.nrep * a.P) return;
    const int r = (int)(it / a.P), l = (int)(it % a.P);
    const RepDesc &R = a.reps[r];
    const uint64_t ek = stream_out(R.seed ^ kTagModes, eval);
    int mv[3];
    if (!draw_mode(R.mt, a.cdf + R.cdf_off, ek, l, mv)) {
      atomicOr(a.err, kErrSampler);
      mv[0] = 1;
      mv[1] = 0;
      mv[2] = 0;
    }
    GatherMode gm;
    gm.mx = (double)mv[0];
    gm.my = (double)mv[1];
    gm.mz = (double)mv[2];
    gm.a = 0.0;
    gm.b = 0.0;
    gather_floats(gm);
    a.modes[it] = gm;
    a.wk[it] = mode_weight(R.mt, a.P, mv[0], mv[1], mv[2]);
    return;
  }
  const int64_t i = blockIdx.x * (int64_t)kBatchThreads + threadIdx.x;
  const bool active = i < a.ntot;
  int k = -1 - (int)(threadIdx.x & 63);  // lanes past the end: a key no other lane has
  if (active) {
    const RepDesc &R = a.reps[a.rep_of[i]];
    double x = a.ix[i], y = a.iy[i], z = a.iz[i];
    if (a.mode == 0) {
      const double u = a.ivx[i] + a.h * a.ifx[i], v = a.ivy[i] + a.h * a.ify[i], w = a.ivz[i] + a.h * a.ifz[i];
      a.ivx[i] = u;
      a.ivy[i] = v;
      a.ivz[i] = w;
      x = wrap_coord(x + a.dt * u, R.g.L[0]);
      y = wrap_coord(y + a.dt * v, R.g.L[1]);
      z = wrap_coord(z + a.dt * w, R.g.L[2]);
      a.ix[i] = x;
      a.iy[i] = y;
      a.iz[i] = z;
      if (!isfinite(u) || !isfinite(v) || !isfinite(w)) atomicOr(a.err, kErrNonFinite);
    } else {
      x = wrap_coord(x, R.g.L[0]);
      y = wrap_coord(y, R.g.L[1]);
      z = wrap_coord(z, R.g.L[2]);
    }
    const int cx = cell_coord(x, R.g.inv_h[0], R.g.nx);
    const int cy = cell_coord(y, R.g.inv_h[1], R.g.ny);
    const int cz = cell_coord(z, R.g.inv_h[2], R.g.nz);
    k = (int)(R.c0 + (a.iq[i] == 0.0 ? R.g.ncell : 0) + (cz * R.g.ny + cy) * R.g.nx + cx);
    a.bin.key[i] = k;
  }
  if (!count) return;
  const int sl = run_slot(k, active, count);  // every lane of the wave takes part in the vote
  if (active) a.bin.slot[i] = sl;
}

// ---------------------------------------------------------------------------
// reorder + pack
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBatchThreads) k_batch_reorder(BatchArgs a) {
  const int64_t k = blockIdx.x * (int64_t)kBatchThreads + threadIdx.x;
  if (k >= a.ntot) return;
  const int j = a.perm[k];
  const RepDesc &R = a.reps[a.rep_of[k]];
  const double x = wrap_coord(a.ix[j], R.g.L[0]), y = wrap_coord(a.iy[j], R.g.L[1]),
               z = wrap_coord(a.iz[j], R.g.L[2]), q = a.iq[j];
  if (a.mode == 0) {
    a.ox[k] = x;
    a.oy[k] = y;
    a.oz[k] = z;
    a.oq[k] = q;
    a.oid[k] = a.iid[j];
    a.ovx[k] = a.ivx[j];
    a.ovy[k] = a.ivy[j];
    a.ovz[k] = a.ivz[j];
  }
  a.xq[k] = make_double4(x, y, z, q);
  if (q != 0.0) a.sq[k] = make_double4(x / R.g.L[0], y / R.g.L[1], z / R.g.L[2], q);
  if (a.pk) a.pk[k] = pack_record(x, y, z, a.pk_scale);
}

// ---------------------------------------------------------------------------
// near field
// ---------------------------------------------------------------------------
// FP32C: one thread per particle walking the stencil rows of its own cell in
// its replica. Four waves per SIMD (no spills; five, with 13 VGPRs spilled,
// ran no faster).
__global__ void __launch_bounds__(kBatchThreads) __attribute__((amdgpu_waves_per_eu(4))) k_batch_near(BatchArgs a) {
  const int64_t i = blockIdx.x * (int64_t)kBatchThreads + threadIdx.x;
  if (i >= a.ntot) return;
  const RepDesc &R = a.reps[a.rep_of[i]];
  const Grid &g = R.g;
  const PairParams &pp = a.pp;
  const double4 pi4 = a.xq[i];
  const double xi = pi4.x, yi = pi4.y, zi = pi4.z, qi = pi4.w;
  const int cx = cell_coord(xi, g.inv_h[0], g.nx);
  const int cy = cell_coord(yi, g.inv_h[1], g.ny);
  const int cz = cell_coord(zi, g.inv_h[2], g.nz);
  ForceAcc<true> acc;
  auto visit_q = [&](int j, const double4 &pj, double shx, double shy, double shz) {
    const double dx = (xi - pj.x) - shx, dy = (yi - pj.y) - shy, dz = (zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    if (r2 == 0.0 && j == (int)i) return;
    if (r2 <= pp.rq2) acc.template add_row<true>(pp, a.pf, r2, qi, pj.w, dx, dy, dz);
  };
  auto visit_lj = [&](int j, const double4 &pj, double shx, double shy, double shz) {
    const double dx = (xi - pj.x) - shx, dy = (yi - pj.y) - shy, dz = (zi - pj.z) - shz;
    const double r2 = sq_dist(dx, dy, dz);
    if (r2 == 0.0 && j == (int)i) return;
    if (r2 <= pp.rlj2) acc.template add_row<false>(pp, a.pf, r2, qi, pj.w, dx, dy, dz);
  };
  // a row's terms summed plainly, the row sum added with Kahan compensation
  auto row_end = [&]() { acc.flush_row(); };
  auto walk = [&](int blk, const Sten &s, double r2, auto &&fn) {
    for_stencil(g, a.cell_start, a.xq, blk, cx, cy, cz, s, xi, yi, zi, r2, fn, R.c0, row_end);
  };
  if (qi != 0.0) {
    if (pp.do_coul || pp.do_lj) walk(0, R.s_coul, pp.rq2, visit_q);
    if (pp.do_lj) walk(1, R.s_lj, pp.rlj2, visit_lj);
  } else if (pp.do_lj) {
    walk(0, R.s_lj, pp.rlj2, visit_lj);
    walk(1, R.s_lj, pp.rlj2, visit_lj);
  }
  a.ofx[i] = acc.get(0);
  a.ofy[i] = acc.get(1);
  a.ofz[i] = acc.get(2);
}

// FP64: one lane per particle, candidates filtered on packed positions
// (pair_device.h, queue walks).
__global__ void __launch_bounds__(kBatchThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_batch_near_queue(BatchArgs a) {
  static_assert(kBatchThreads == kQueueThreads, "queue layout");
  __shared__ uint32_t queue[kQueueCap * kQueueThreads];
  const int64_t i = blockIdx.x * (int64_t)kBatchThreads + threadIdx.x;
  const bool active = i < a.ntot;  // the whole wave takes part
  const int64_t ia = active ? i : a.ntot - 1;
  const RepDesc &R = a.reps[a.rep_of[ia]];
  const PairParams &pp = a.pp;
  const double4 pi = a.xq[ia];
  const bool charged = pi.w != 0.0;
  ForceAcc<false> acc;
  HitQueue Q(queue);
  const bool coded = a.ntot <= (1ll << kIndexBits);
  auto one = [&](uint32_t e) {
    const uint32_t code = coded ? e >> kIndexBits : Q.now;
    const int j = (int)(coded ? e & ((1u << kIndexBits) - 1u) : e);
    const double4 pj = a.xq[j];
    double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
    if (wave_count(code != kNoShift)) {
      dx -= code_shift(code, 0) * R.g.L[0];
      dy -= code_shift(code, 1) * R.g.L[1];
      dz -= code_shift(code, 2) * R.g.L[2];
    }
    const double r2 = sq_dist(dx, dy, dz);
    const bool coul = charged && pj.w != 0.0;
    if ((r2 <= (coul ? pp.rq2 : pp.rlj2)) & (j != (int)i)) {
      if (coul) acc.template add<true, true>(pp, a.pf, r2, pi.w, pj.w, dx, dy, dz);
      else acc.template add<false>(pp, a.pf, r2, pi.w, pj.w, dx, dy, dz);
    }
  };
  auto drain = [&](bool all) { drain_queue(Q, all, one); };
  const bool far = charged && (pp.do_coul || pp.do_lj);
  const bool some = far || pp.do_lj;
  const int32_t *cs = a.cell_start + R.c0;
  queue_walk<false>(R.g, cs, a.pk, nullptr, nullptr, 0, active && some, pi, far ? R.s_coul : R.s_lj,
                    far ? pp.rq2 : pp.rlj2, far ? a.t2_q : a.t2_lj, a.pk_scale, coded, Q, [](int) {}, drain);
  queue_walk<false>(R.g, cs + R.g.ncell, a.pk, nullptr, nullptr, 0, active && pp.do_lj, pi, R.s_lj, pp.rlj2, a.t2_lj,
                    a.pk_scale, coded, Q, [](int) {}, drain);
  drain(true);
  if (!active) return;
  a.ofx[i] = acc.get(0);
  a.ofy[i] = acc.get(1);
  a.ofz[i] = acc.get(2);
}

// The same for batches of too few particles to fill the chip with one thread
// each: G lanes share a particle (pair_device.h, group walks).
template <bool F32, int G>
__global__ void __launch_bounds__(kBatchThreads) k_batch_near_group(BatchArgs a) {
  __shared__ GroupRows<G> rows[kBatchThreads / G];
  __shared__ GroupTerms<F32 ? G : 1> terms[kBatchThreads / G];
  const int64_t per = (a.ntot + gridDim.x - 1) / gridDim.x;  // consecutive particles per block
  const int64_t first = blockIdx.x * per, last = min(a.ntot, first + per);
  for (int64_t i = first + threadIdx.x / G; i < last; i += kBatchThreads / G) {  // the lanes of a group together
    const RepDesc &R = a.reps[a.rep_of[i]];
    ForceAcc<F32> acc;
    group_sums<F32, false, G>(a.pp, a.pf, R.g, R.s_coul, R.s_lj, a.cell_start + R.c0, a.xq, nullptr, nullptr, 0,
                              (int)i, a.xq[i], false, rows[threadIdx.x / G], &terms[threadIdx.x / G].t[0], acc,
                              [](bool, bool, double) {});
    const double f0 = acc.template total<G>(0), f1 = acc.template total<G>(1), f2 = acc.template total<G>(2);
    if (threadIdx.x % G == 0) {
      a.ofx[i] = f0;
      a.ofy[i] = f1;
      a.ofz[i] = f2;
    }
  }
}

// Near-field kernel of a batch and its blocks. The group form up to these
// sizes of the whole batch; a step of 8 to 128 replicas in us, thread form
// against group form: FP64 20,000 particles 1190, 789; 150,000: 1604, 1311;
// 300,000: 2016, 2003; 600,000: 2696, 3019. FP32C 20,000: 1154, 872; 150,000:
// 1411, 1332; 300,000: 1733, 1929.
constexpr int64_t kBatchGroupMost64 = 262144, kBatchGroupMost32 = 131072;
using BatchKernel = void (*)(BatchArgs);
static BatchKernel batch_near_kernel(int prec, int64_t ntot, unsigned *blocks) {
  if (ntot <= (prec == RBE_FP32C ? kBatchGroupMost32 : kBatchGroupMost64)) {
    *blocks = group_blocks(ntot, 32);
    return prec == RBE_FP32C ? k_batch_near_group<true, 32> : k_batch_near_group<false, 32>;
  }
  *blocks = (unsigned)((ntot + kBatchThreads - 1) / kBatchThreads);
  return prec == RBE_FP32C ? k_batch_near : k_batch_near_queue;
}

// ---------------------------------------------------------------------------
// structure factors
// ---------------------------------------------------------------------------
// A block takes `sub` consecutive chunks (of all replicas' chunks) and every
// mode of theirs, one lane per (chunk, mode): with P = 100 two chunks keep 200
// of 256 lanes busy where whole waves of modes would keep 100 of 128. The
// chunks' records are staged in LDS; a lane sums its chunk's terms in order.
constexpr int kBatchSubMax = 4;
template <bool F32>
__global__ void __launch_bounds__(kBatchThreads) k_batch_rho(BatchArgs a, const RepDesc *__restrict__ reps,
                                                             const double4 *__restrict__ sq,
                                                             const GatherMode *__restrict__ modes,
                                                             const double2 *__restrict__ turn_tab, int sub) {
  static_assert(kBatchThreads == kTurnTable, "one table entry per thread");
  __shared__ double4 rec[kBatchSubMax * kBatchChunk];
  __shared__ double2 tab[F32 ? 1 : kTurnTable];
  __shared__ int srep[kBatchSubMax], scnt[kBatchSubMax];
  __shared__ int64_t sfirst[kBatchSubMax];
  const int tid = threadIdx.x, P = a.P;
  const int chunks = *a.rho_chunks, c0 = blockIdx.x * sub;
  if (c0 >= chunks) return;  // uniform over the block
  if (!F32) tab[tid] = turn_tab[tid];
  if (tid < sub) {
    // replica of the chunk: the last r with chunk_off <= c
    const int c = c0 + tid;
    int lo = 0, hi = a.nrep - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (reps[mid].chunk_off <= c) lo = mid;
      else hi = mid - 1;
    }
    const int first = (c - reps[lo].chunk_off) * kBatchChunk;
    srep[tid] = lo;
    scnt[tid] = c < chunks ? min(reps[lo].nq - first, kBatchChunk) : 0;
    sfirst[tid] = reps[lo].p0 + first;
  }
  __syncthreads();
  for (int u = tid; u < sub * kBatchChunk; u += kBatchThreads) {
    const int s = u / kBatchChunk, v = u % kBatchChunk;
    if (v < scnt[s]) rec[u] = sq[sfirst[s] + v];
  }
  __syncthreads();
  for (int it = tid; it < sub * P; it += kBatchThreads) {
    const int s = it / P, l = it % P;
    const int cnt = scnt[s];
    if (cnt <= 0) continue;
    const GatherMode &gm = modes[(int64_t)srep[s] * P + l];
    const double unit = F32 ? 1.0 : kTurnTable;
    const double mx = unit * gm.mx, my = unit * gm.my, mz = unit * gm.mz;
    const double4 *p = rec + s * kBatchChunk;
    double2 out;
    if (F32) {
      float re = 0.f, rc = 0.f, im = 0.f, ic = 0.f;
#pragma unroll 4
      for (int j = 0; j < cnt; ++j) {
        const double4 v = p[j];
        const float t = turn_f32(mx, my, mz, v.x, v.y, v.z);
        const float q = (float)v.w;
        kahan_fma(re, rc, q, __builtin_amdgcn_cosf(t));
        kahan_fma(im, ic, q, __builtin_amdgcn_sinf(t));
      }
      out = make_double2((double)re - (double)rc, (double)im - (double)ic);
    } else {
      double re = 0.0, im = 0.0;
#pragma unroll 4
      for (int j = 0; j < cnt; ++j) {
        const double4 v = p[j];
        double sn, cs;
        sincos_phase_f64(phase_dot(mx, my, mz, v.x, v.y, v.z), tab, &sn, &cs);
        re = fma(v.w, cs, re);
        im = fma(v.w, sn, im);
      }
      out = make_double2(re, im);
    }
    a.part[(int64_t)(c0 + s) * P + l] = out;
  }
}

// One wave per (replica, mode): the chunk partials in a fixed order, and the
// gather coefficients.
__global__ void __launch_bounds__(kBatchThreads) k_batch_rho_final(BatchArgs a) {
  const int64_t it = (blockIdx.x * (int64_t)kBatchThreads + threadIdx.x) >> 6;
  if (it >= (int64_t)a.nrep * a.P) return;
  const int lane = threadIdx.x & 63, P = a.P;
  const int r = (int)(it / P), l = (int)(it % P);
  const RepDesc &R = a.reps[r];
  double re = 0.0, im = 0.0;
  for (int c = lane; c < R.nchunks; c += 64) {
    const double2 v = a.part[(int64_t)(R.chunk_off + c) * P + l];
    re += v.x;
    im += v.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    re += __shfl_xor(re, o, 64);
    im += __shfl_xor(im, o, 64);
  }
  if (lane == 0) {
    const double w = a.pp.kc * a.wk[it];
    GatherMode &gm = a.modes[it];
    gm.a = w * im;
    gm.b = w * re;
    gm.af = (float)(w * im);
    gm.bf = (float)(w * re);
  }
}

// ---------------------------------------------------------------------------
// Fourier gather + second half-kick
// ---------------------------------------------------------------------------
// Sum over the modes md of one particle at s: (g_x, g_y, g_z) of F^F = -q (2
// pi / L) g.
template <bool F32>
__device__ inline void batch_gather_sum(const GatherMode *__restrict__ md, int P, const double4 &s,
                                        const double2 *tab, double g[3]) {
  if (F32) {
    float gx = 0.f, gy = 0.f, gz = 0.f, ex = 0.f, ey = 0.f, ez = 0.f;
#pragma unroll 4
    for (int l = 0; l < P; ++l) {
      const GatherMode gm = md[l];
      const float t = turn_f32(gm.mx, gm.my, gm.mz, s.x, s.y, s.z);
      const float h = fmaf(gm.af, __builtin_amdgcn_cosf(t), -gm.bf * __builtin_amdgcn_sinf(t));
      kahan_fma(gx, ex, h, gm.mxf);
      kahan_fma(gy, ey, h, gm.myf);
      kahan_fma(gz, ez, h, gm.mzf);
    }
    g[0] = (double)gx - (double)ex;
    g[1] = (double)gy - (double)ey;
    g[2] = (double)gz - (double)ez;
  } else {
    const double sx = kTurnTable * s.x, sy = kTurnTable * s.y, sz = kTurnTable * s.z;
    double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll 4
    for (int l = 0; l < P; ++l) {
      const GatherMode gm = md[l];
      double sn, cs;
      sincos_phase_f64(phase_dot(gm.mx, gm.my, gm.mz, sx, sy, sz), tab, &sn, &cs);
      const double h = gm.a * cs - gm.b * sn;
      gx = fma(h, gm.mx, gx);
      gy = fma(h, gm.my, gy);
      gz = fma(h, gm.mz, gz);
    }
    g[0] = gx;
    g[1] = gy;
    g[2] = gz;
  }
}

template <bool F32>
__global__ void __launch_bounds__(kBatchThreads) k_batch_gather(BatchArgs a, const GatherMode *__restrict__ modes,
                                                                const double2 *__restrict__ turn_tab) {
  __shared__ double2 tab[F32 ? 1 : kTurnTable];
  if (!F32) {
    tab[threadIdx.x] = turn_tab[threadIdx.x];
    __syncthreads();
  }
  const int64_t i = blockIdx.x * (int64_t)kBatchThreads + threadIdx.x;
  if (i >= a.ntot) return;
  const int r = a.rep_of[i];
  const RepDesc &R = a.reps[r];
  double fx = a.ofx[i], fy = a.ofy[i], fz = a.ofz[i];
  if (a.do_far && i < R.p0 + R.nq) {
    const double4 s = a.sq[i];
    double g[3];
    // a wave inside one replica reads its modes as scalars
    const int r0 = __builtin_amdgcn_readfirstlane(r);
    if (__all(r == r0)) batch_gather_sum<F32>(modes + (int64_t)r0 * a.P, a.P, s, tab, g);
    else batch_gather_sum<F32>(modes + (int64_t)r * a.P, a.P, s, tab, g);
    fx -= s.w * (kTwoPi / R.g.L[0]) * g[0];
    fy -= s.w * (kTwoPi / R.g.L[1]) * g[1];
    fz -= s.w * (kTwoPi / R.g.L[2]) * g[2];
  }
  if (a.mode == 0) {
    a.ofx[i] = fx;
    a.ofy[i] = fy;
    a.ofz[i] = fz;
    const double u = a.ovx[i] + a.h * fx, v = a.ovy[i] + a.h * fy, w = a.ovz[i] + a.h * fz;
    a.ovx[i] = u;
    a.ovy[i] = v;
    a.ovz[i] = w;
    if (!isfinite(u) || !isfinite(v) || !isfinite(w)) atomicOr(a.err, kErrNonFinite);
  } else {
    const int j = a.perm[i];
    a.cfx[j] = fx;
    a.cfy[j] = fy;
    a.cfz[j] = fz;
  }
}

void launch_batch_step(int prec, const BatchArgs &a, uint64_t eval, bool first, bool last, hipStream_t st) {
  const unsigned nb = (unsigned)((a.ntot + kBatchThreads - 1) / kBatchThreads);
  const int64_t nm = (int64_t)a.nrep * a.P;
  const unsigned mb = a.do_far ? (unsigned)((nm + kBatchThreads - 1) / kBatchThreads) : 0u;
  const bool f32 = prec == RBE_FP32C;
  if (first) launch_bin_clear(a.bin, a.nkeys, a.ntot, st);
  k_batch_drift<<<nb + mb, kBatchThreads, 0, st>>>(a, eval, nb,
                                                   bin_keys_out(a.bin, a.nkeys, a.ntot, nullptr).count);
  launch_bin_place(a.bin, a.nkeys, a.ntot, a.cell_start, a.perm, !last, st);
  k_batch_reorder<<<nb, kBatchThreads, 0, st>>>(a);
  unsigned near_blocks;
  const BatchKernel near = batch_near_kernel(prec, a.ntot, &near_blocks);
  near<<<near_blocks, kBatchThreads, 0, st>>>(a);
  if (a.do_far) {
    int sub = a.P < kBatchThreads ? kBatchThreads / a.P : 1;
    if (sub > kBatchSubMax) sub = kBatchSubMax;
    const unsigned rb = (unsigned)((a.chunk_cap + sub - 1) / sub);
    if (f32) k_batch_rho<true><<<rb, kBatchThreads, 0, st>>>(a, a.reps, a.sq, a.modes, a.turn_tab, sub);
    else k_batch_rho<false><<<rb, kBatchThreads, 0, st>>>(a, a.reps, a.sq, a.modes, a.turn_tab, sub);
    k_batch_rho_final<<<(unsigned)((nm * 64 + kBatchThreads - 1) / kBatchThreads), kBatchThreads, 0, st>>>(a);
  }
  if (f32) k_batch_gather<true><<<nb, kBatchThreads, 0, st>>>(a, a.modes, a.turn_tab);
  else k_batch_gather<false><<<nb, kBatchThreads, 0, st>>>(a, a.modes, a.turn_tab);
}

// ---------------------------------------------------------------------------
// per-replica charge checks and layout
// ---------------------------------------------------------------------------
constexpr int kQstatThreads = 1024;
__global__ void __launch_bounds__(kQstatThreads) k_qstats_rep(const int64_t *__restrict__ off,
                                                              const double *__restrict__ q, int32_t *__restrict__ nq,
                                                              double *__restrict__ qs) {
  __shared__ int lc[kQstatThreads / 64];
  __shared__ double ls[kQstatThreads / 64], la[kQstatThreads / 64];
  const int r = blockIdx.x;
  const int64_t lo = off[r], hi = off[r + 1];
  int c = 0;
  double s = 0.0, a = 0.0;
#pragma unroll 4
  for (int64_t i = lo + threadIdx.x; i < hi; i += kQstatThreads) {
    const double v = q[i];
    c += v != 0.0;
    s += v;
    a += fabs(v);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    c += __shfl_xor(c, o, 64);
    s += __shfl_xor(s, o, 64);
    a += __shfl_xor(a, o, 64);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    lc[w] = c;
    ls[w] = s;
    la[w] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c = 0;
    s = a = 0.0;
    for (int k = 0; k < kQstatThreads / 64; ++k) {
      c += lc[k];
      s += ls[k];
      a += la[k];
    }
    nq[r] = c;
    qs[2 * r] = s;
    qs[2 * r + 1] = a;
  }
}

void launch_qstats_rep(int nrep, const int64_t *off, const double *q, int32_t *nq, double *qs, hipStream_t st) {
  k_qstats_rep<<<nrep, kQstatThreads, 0, st>>>(off, q, nq, qs);
}

// Per-replica checks of Eq. 1 (flags kErrNonNeutral / kErrNonFinite) and the
// structure-factor layout of this call from the device counts: replica r's
// charged particles in chunks of kBatchChunk, its chunk partials at chunk_off;
// *rho_chunks receives the total, *bad_rep the first replica that failed a
// check (-1: none). One block, 256 replicas at a time.
__global__ void __launch_bounds__(256) k_batch_layout(int nrep, const int32_t *__restrict__ nq,
                                                      const double *__restrict__ qs, RepDesc *__restrict__ reps,
                                                      int *__restrict__ rho_chunks, int *__restrict__ bad_rep,
                                                      int *err) {
  __shared__ int wsum[4], bad;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) bad = 0x7FFFFFFF;
  int carry = 0;
  for (int b = 0; b < nrep; b += 256) {
    const int r = b + threadIdx.x;
    int chunks = 0, f = 0;
    if (r < nrep) {
      const double sq = qs[2 * r], sa = qs[2 * r + 1];
      if (!isfinite(sq) || !isfinite(sa)) f = kErrNonFinite;
      else if (fabs(sq) > 1e-10 * fmax(sa, 1e-300) && fabs(sq) > 1e-12) f = kErrNonNeutral;
      chunks = (nq[r] + kBatchChunk - 1) / kBatchChunk;
    }
    int incl = chunks;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    __syncthreads();  // wsum of the previous round is read
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int off = carry;
    for (int w = 0; w < 4; ++w) {
      if (w < wave) off += wsum[w];
      carry += wsum[w];
    }
    if (r < nrep) {
      RepDesc &d = reps[r];
      d.nq = nq[r];
      d.nchunks = chunks;
      d.chunk_off = off + incl - chunks;
      if (f) {
        atomicOr(err, f);
        atomicMin(&bad, r);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    *rho_chunks = carry;
    *bad_rep = bad == 0x7FFFFFFF ? -1 : bad;
  }
}

void launch_batch_layout(int nrep, const int32_t *nq, const double *qs, RepDesc *reps, int *rho_chunks, int *bad_rep,
                         int *err, hipStream_t st) {
  k_batch_layout<<<1, 256, 0, st>>>(nrep, nq, qs, reps, rho_chunks, bad_rep, err);
}

}  // namespace rbe
