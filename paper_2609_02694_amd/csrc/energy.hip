// Energy terms of the Ewald splitting (Sec. 2.1): the screened real-space
// Coulomb energy (Eq. 4) and the LJ energy (Eq. 2) over every pair inside
// the cutoffs, the importance-sampled Fourier energy of a mode sample
// (Eq. 5 with the sampling of Eq. 9), the self energy (Eq. 6), the kinetic
// energy, and the virials of the three potential terms (minus their
// derivatives under a uniform dilation of positions and box), from which
// the pressure follows. Diagnostics, so always FP64, with the device
// library's sqrt, division, exp and erfc rather than the force kernels'
// polynomials.
//
// Every sum has one fixed order: per-thread sums, a fixed butterfly in each
// wave, the waves of a block in index order, then the block partials in
// index order (thread-strided sums, butterfly, waves) in a one-block final
// kernel. Results are a pure function of the inputs and the grid.
#include "pair_device.h"

namespace rbe {

constexpr int kEnergyThreads = 256;
// Lanes per particle of the near field: 64 or 32 (group walk), or one (queue
// walk), the faster form from the size at which its waves fill the chip, sooner
// where the cutoff sphere is nearly empty. A whole call in us with 64, 32 and
// one: electrolyte 4,000 particles 82, 87, 455; 20,000: 131, 119, 459; 130,000:
// 386, 351, 446; 260,000: 653, 575, 508; LJ electrolyte (21 particles in the
// sphere) 20,000: 107, 90, 123; 65,000: 220, 164, 134.
constexpr int64_t kEnergyWide = 196608, kEnergyNarrow = 40960;
static bool energy_narrow(const PairParams &pp, int64_t n) {
  return mean_within(pp.g, n, std::sqrt(pp.rq2)) < 48.0;
}
static int energy_lanes(bool narrow, int64_t n) {
  return n <= 4096 ? 64 : n <= (narrow ? kEnergyNarrow : kEnergyWide) ? 32 : 1;
}
bool energy_packed(const PairParams &pp, int64_t n) { return energy_lanes(energy_narrow(pp, n), n) == 1; }
constexpr int64_t kEnergyNearBlocks = 16384;  // most blocks of the near field (each leaves one partial sum)
constexpr int kEnergySqBlocks = 1024;  // grid of the q^2 / v^2 sums

// Sum of v over the block; the result is valid in thread 0.
__device__ inline double block_sum(double v, double *lds) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();  // lds may still be read from a previous call
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < kEnergyThreads / 64; ++k) s += lds[k];
  return s;
}

// Near-field energy and virial of particle i (sorted order), halved so that
// the sum over i counts each pair once:
//   u_i = 1/2 sum_{j != i} [kc q_i q_j erfc(sqrt(a) r)/r   (r <= r_coul)
//                           + 4 eps ((sigma/r)^12 - (sigma/r)^6) (r <= r_lj)]
//   w_i = 1/2 sum_{j != i} d_ij . F_ij = 1/2 sum r^2 (kc q_i q_j G(r) + G_LJ(r)),
//         r^2 G = erfc(sqrt(a) r)/r + 2 sqrt(a/pi) exp(-a r^2),
//         r^2 G_LJ = 24 eps (2 (sigma/r)^12 - (sigma/r)^6)        (Eq. 8)
// over the minimum image. Species layout as in the force kernels: charged i
// (q_i != 0, the range [0, nq) of the cell order) walk the charged block out to max(r_coul, r_lj) and the neutral
// block out to r_lj; neutral i walk both blocks out to r_lj.
// part[4 b + 0..3] = Coulomb energy, LJ energy, Coulomb virial, LJ virial of
// block b.
struct EnergyNear {
  PairParams pp;
  double lj4, two_sqrt_a_pi;
  int64_t n;
  const double4 *__restrict__ xq;
  const uint2 *__restrict__ pk;
  double pk_scale;
  uint32_t t2_q, t2_lj;  // squared reaches in packed units
  bool queue_lj;         // queue walk: LJ pairs too (k_energy_near_queue)
  const int32_t *__restrict__ cell_start;
  double *__restrict__ part;
};
// A thread's share of the four sums.
struct EnergySums {
  double uc = 0.0, ul = 0.0, wc = 0.0, wl = 0.0;
  __device__ inline void add(const EnergyNear &a, double qi, double qj, double r2) {
    const PairParams &pp = a.pp;
    if (pp.do_coul && r2 <= pp.rc2 && qi != 0.0 && qj != 0.0) {
      const double r = sqrt(r2);
      const double qq = pp.kc * qi * qj;
      const double er = erfc(pp.sqrt_alpha * r) / r;
      uc += qq * er;
      wc += qq * (er + a.two_sqrt_a_pi * exp(-pp.alpha * r2));
    }
    if (pp.do_lj && r2 <= pp.rlj2) add_lj(pp, r2);
  }
  __device__ inline void add_lj(const PairParams &pp, double r2) {
    const double s2 = pp.sig2 / r2, s6 = s2 * s2 * s2;
    ul += s6 * s6 - s6;
    wl += 2.0 * s6 * s6 - s6;
  }
  __device__ inline void put(const EnergyNear &a, double *lds) {
    const double sc = block_sum(0.5 * uc, lds), sl = block_sum(0.5 * a.lj4 * ul, lds);
    const double vc = block_sum(0.5 * wc, lds), vl = block_sum(0.5 * a.pp.eps24 * wl, lds);
    if (threadIdx.x == 0) ((double4 *)a.part)[blockIdx.x] = make_double4(sc, sl, vc, vl);
  }
};

// Bound by the issue of the library's erfc and exp, about 250 instructions a
// pair: the pairs wait until all lanes have one (GroupHits). 130,000 ions 590
// -> 500 us a call, 20,000 145 -> 130.
template <int G>
__global__ void __launch_bounds__(kEnergyThreads) k_energy_near(EnergyNear a) {
  __shared__ double lds[kEnergyThreads / 64];
  __shared__ GroupRows<G> rows[kEnergyThreads / G];
  __shared__ GroupHits<G, double2> hits[kEnergyThreads / G];
  const int64_t per = (a.n + gridDim.x - 1) / gridDim.x;  // consecutive particles per block
  const int64_t end = min(a.n, (blockIdx.x + 1) * per);
  const PairParams &pp = a.pp;
  const Block near_lj = pp.do_lj ? Block{pp.s_lj, pp.rlj2} : no_block();
  EnergySums sums;
  for (int64_t i = blockIdx.x * per + threadIdx.x / G; i < end; i += kEnergyThreads / G) {
    const double4 pi = a.xq[i];
    const bool charged = pi.w != 0.0;
    GroupHits<G, double2> &H = hits[threadIdx.x / G];
    int pending = 0;
    auto eval = [&](const double2 &h) { sums.add(a, pi.w, h.y, h.x); };  // r^2, q_j
    group_walk<G, false>(
        pp.g, a.cell_start, a.xq, nullptr, nullptr, 0, pi, charged ? Block{pp.s_coul, pp.rq2} : near_lj, near_lj,
        rows[threadIdx.x / G],
        [&](bool ok, int, int blk, int j, const double4 &pj, double, double, double, double r2) {
          const double reach2 = charged && blk == 0 ? pp.rq2 : pp.rlj2;
          put_hits<G>(H, pending, ok & (j != (int)i) & (r2 <= reach2), make_double2(r2, pj.w), eval);
        },
        [](int, int) {}, [](uint64_t) {});
    take_hits<G>(H, pending, eval);
  }
  sums.put(a, lds);
}

// The same with one lane per particle, the candidates filtered on packed
// positions and the terms of those that pass evaluated from the lanes' queues
// (pair_device.h, queue walks): the error function runs with three quarters of
// the lanes or more instead of the half whose candidate is inside the cutoff,
// and the walk's set-up is a lane's, not a wave's. 1M ions 3.78 -> 3.00 ms a
// call, 1M LJ electrolyte 1.26 -> 0.72.
// A pair without a Coulomb term costs less than a queue entry's fetch: such
// blocks are summed as they are met, but for nearly empty spheres, whose rows
// leave most lanes idle. A whole call in us, queued and as met: neutral
// particles, 400,000, 1,000 in the sphere 5851, 4370; 120: 622, 562; a tenth
// charged, 200,000, 300 in the sphere 1020, 767; 30: 202, 203; 60,000, 30: 114,
// 139.
__global__ void __launch_bounds__(kEnergyThreads) __attribute__((amdgpu_waves_per_eu(3)))
k_energy_near_queue(EnergyNear a) {
  static_assert(kEnergyThreads == kQueueThreads, "queue layout");
  __shared__ double lds[kEnergyThreads / 64];
  __shared__ uint32_t queue[kQueueCap * kQueueThreads];
  const PairParams &pp = a.pp;
  const Grid &g = pp.g;
  const bool coded = a.n <= (1ll << kIndexBits);
  const int64_t tiles = (a.n + kEnergyThreads - 1) / kEnergyThreads;  // of consecutive particles
  EnergySums sums;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t i = t * kEnergyThreads + threadIdx.x;
    const bool active = i < a.n;  // the whole wave takes part
    const double4 pi = a.xq[active ? i : a.n - 1];
    HitQueue Q(queue);
    auto one = [&](uint32_t e) {
      const uint32_t code = coded ? e >> kIndexBits : Q.now;
      const int j = (int)(coded ? e & ((1u << kIndexBits) - 1u) : e);
      const double4 pj = a.xq[j];
      double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
      if (wave_count(code != kNoShift)) {
        dx -= code_shift(code, 0) * g.L[0];
        dy -= code_shift(code, 1) * g.L[1];
        dz -= code_shift(code, 2) * g.L[2];
      }
      if (j != (int)i) sums.add(a, pi.w, pj.w, sq_dist(dx, dy, dz));
    };
    auto drain = [&](bool all) { drain_queue(Q, all, one); };
    const bool charged = pi.w != 0.0, coul = charged && pp.do_coul;
    const bool some = coul || (a.queue_lj && pp.do_lj);
    queue_walk<false>(g, a.cell_start, a.pk, nullptr, nullptr, 0, active && some, pi, charged ? pp.s_coul : pp.s_lj,
                      charged ? pp.rq2 : pp.rlj2, charged ? a.t2_q : a.t2_lj, a.pk_scale, coded, Q, [](int) {}, drain);
    if (a.queue_lj)
      queue_walk<false>(g, a.cell_start + g.ncell, a.pk, nullptr, nullptr, 0, active && pp.do_lj, pi, pp.s_lj,
                        pp.rlj2, a.t2_lj, a.pk_scale, coded, Q, [](int) {}, drain);
    drain(true);
    if (a.queue_lj || !pp.do_lj || !active) continue;
    const int cx = cell_coord(pi.x, g.inv_h[0], g.nx), cy = cell_coord(pi.y, g.inv_h[1], g.ny),
              cz = cell_coord(pi.z, g.inv_h[2], g.nz);
    for (int blk = coul; blk < 2; ++blk)
      for_stencil(g, a.cell_start, a.xq, blk, cx, cy, cz, pp.s_lj, pi.x, pi.y, pi.z, pp.rlj2,
                  [&](int j, const double4 &pj, double shx, double shy, double shz) {
                    const double dx = (pi.x - pj.x) - shx, dy = (pi.y - pj.y) - shy, dz = (pi.z - pj.z) - shz;
                    const double r2 = sq_dist(dx, dy, dz);
                    if (j != (int)i && r2 <= pp.rlj2) sums.add_lj(pp, r2);
                  });
  }
  sums.put(a, lds);
}

// part[2 b] = sum q_i^2 and part[2 b + 1] = sum |v_i|^2 over the particles
// of block b's grid-stride sequence (caller order; v may be absent).
__global__ void __launch_bounds__(kEnergyThreads) k_energy_sq(int64_t n, const double *__restrict__ q,
                                                              const double *__restrict__ vx,
                                                              const double *__restrict__ vy,
                                                              const double *__restrict__ vz,
                                                              double *__restrict__ part) {
  __shared__ double lds[kEnergyThreads / 64];
  double sq = 0.0, sv = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)kEnergyThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kEnergyThreads) {
    sq += q[i] * q[i];
    if (vx) sv += vx[i] * vx[i] + vy[i] * vy[i] + vz[i] * vz[i];
  }
  const double a = block_sum(sq, lds);
  const double b = block_sum(sv, lds);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = a;
    part[2 * blockIdx.x + 1] = b;
  }
}

// One block: out[0] Coulomb real, out[1] LJ, out[2] Fourier, out[3] self,
// out[4] kinetic, out[5..7] virials of the Coulomb real, LJ and Fourier terms.
__global__ void __launch_bounds__(kEnergyThreads) k_energy_final(EnergyFinal a) {
  __shared__ double lds[kEnergyThreads / 64];
  // thread-strided sums of the partials, several loads in flight: bound by
  // their latency (16,384 partials one load at a time, 43 us; now 6.7)
  double near[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int64_t b = threadIdx.x; b < a.nb_near; b += kEnergyThreads) {
    const double4 v = ((const double4 *)a.near_part)[b];
    near[0] += v.x;
    near[1] += v.y;
    near[2] += v.z;
    near[3] += v.w;
  }
  for (int t = 0; t < 4; ++t) near[t] = block_sum(near[t], lds);
  double uf = 0.0, wf = 0.0;
  if (a.rho) {
    // U^{F,*} = kc (1/2) sum_l w_l |rho_l|^2 and its virial
    // W^{F,*} = kc (1/2) sum_l w_l |rho_l|^2 (1 - k_l^2/(2 alpha))
    double s = 0.0, v = 0.0;
    for (int l = threadIdx.x; l < a.P; l += kEnergyThreads) {
      const double u = 0.5 * a.w[l] * (a.rho[l] * a.rho[l] + a.rho[a.P + l] * a.rho[a.P + l]);
      const double kx = kTwoPi * a.mkd[l] / a.L[0], ky = kTwoPi * a.mkd[a.P + l] / a.L[1],
                   kz = kTwoPi * a.mkd[2 * a.P + l] / a.L[2];
      const double k2 = kx * kx + ky * ky + kz * kz;
      s += u;
      v += u * (1.0 - k2 / (2.0 * a.alpha));
    }
    uf = block_sum(s, lds);
    wf = block_sum(v, lds);
  }
  double q2 = 0.0, v2 = 0.0;
#pragma unroll 4
  for (int64_t b = threadIdx.x; b < a.nb_sq; b += kEnergyThreads) {
    const double2 v = ((const double2 *)a.sq_part)[b];
    q2 += v.x;
    v2 += v.y;
  }
  q2 = block_sum(q2, lds);
  v2 = block_sum(v2, lds);
  if (threadIdx.x == 0) {
    a.out[0] = near[0];
    a.out[1] = near[1];
    a.out[2] = a.rho ? a.kc * uf : 0.0;
    a.out[3] = a.rho ? a.self_coef * q2 : 0.0;
    a.out[4] = a.half_mass * v2;
    a.out[5] = near[2];
    a.out[6] = near[3];
    a.out[7] = a.rho ? a.kc * wf : 0.0;
  }
}

static int64_t energy_near_blocks(int64_t n, int lanes) {
  const int64_t nb = (n * lanes + kEnergyThreads - 1) / kEnergyThreads;
  return nb < kEnergyNearBlocks ? nb : kEnergyNearBlocks;
}

int energy_part_len(int64_t n_max) { return (int)(4 * energy_near_blocks(n_max, 64) + 2 * kEnergySqBlocks); }

void launch_energy(const PairParams &pp, double lj4, int64_t n, const Sorted &s,
                   const int32_t *cell_start, bool near, const double *q, const double *vx, const double *vy,
                   const double *vz, double *part, EnergyFinal fin, hipStream_t st) {
  int64_t nb_near = 0;
  if (near && n > 0) {
    const bool narrow = energy_narrow(pp, n);
    const int lanes = energy_lanes(narrow, n);
    nb_near = energy_near_blocks(n, lanes);
    EnergyNear a{};
    a.pp = pp;
    a.lj4 = lj4;
    a.two_sqrt_a_pi = 2.0 * std::sqrt(pp.alpha / kPi);
    a.n = n;
    a.xq = s.xq;
    a.pk = s.pk;
    a.pk_scale = s.pk_scale;
    a.t2_q = pack_reach2(std::sqrt(pp.rq2), s.pk_scale);
    a.t2_lj = pack_reach2(std::sqrt(pp.rlj2), s.pk_scale);
    a.queue_lj = narrow;
    a.cell_start = cell_start;
    a.part = part;
    const auto kernel = lanes == 64 ? k_energy_near<64> : lanes == 32 ? k_energy_near<32> : k_energy_near_queue;
    kernel<<<(unsigned)nb_near, kEnergyThreads, 0, st>>>(a);
  }
  double *sq_part = part + 4 * nb_near;
  int64_t nb_sq = (n + kEnergyThreads - 1) / kEnergyThreads;
  if (nb_sq > kEnergySqBlocks) nb_sq = kEnergySqBlocks;
  if (nb_sq < 1) nb_sq = 1;
  k_energy_sq<<<(unsigned)nb_sq, kEnergyThreads, 0, st>>>(n, q, vx, vy, vz, sq_part);
  fin.near_part = near ? part : nullptr;
  fin.nb_near = nb_near;
  fin.sq_part = sq_part;
  fin.nb_sq = nb_sq;
  k_energy_final<<<1, kEnergyThreads, 0, st>>>(fin);
}

}  // namespace rbe
