// Fourier part of the RBE force (Sec. 2.1, Eq. 5, 7, 9; Sec. 2.3.1):
// structure factors rho(k_l) = sum_j q_j exp(i k_l . r_j) over the charged
// particles, then F_i = -kc q_i sum_l w_l k_l Im(exp(-i k_l . r_i) rho_l)
// (kc the Coulomb prefactor, 1 in reduced units).
//
// Phase: k_l . r_j = 2 pi t with t = m_l . s_j (s = r/L, the fractional
// coordinate). Whole turns are removed in FP64 (exactly) before the sine and
// cosine, so the trigonometric argument is a fraction of a turn whatever the
// box size.
//
// Structure factor: thread = mode, particles walked in a wave-uniform loop
// (the chunk's (s, q) records staged in LDS), one partial sum per particle
// chunk and mode; up to 128 modes the waves of a block share the records
// (FP64). A wave left with fewer than 64 modes (P not a multiple of 64)
// spreads each mode over several lanes that split the chunk's particles and
// adds their sums with a fixed butterfly. The chunk partials are summed in
// FP64 in a fixed order by a second kernel.
//
// Gather: thread = particle, modes walked in a wave-uniform loop with the
// per-mode coefficients (m, w Im rho, w Re rho) in scalar registers; for few
// particles the waves of a block share the modes.
//
// Tables with columns (an Ewald lattice given by the caller, FP64): up to nine
// modes consecutive in m_z share one sine and cosine (k_rho_runs,
// k_gather_runs).
//
// FP32C form: the turn reduction stays FP64; the hardware turn-argument
// sine/cosine (v_sin_f32 / v_cos_f32 compute sin(2 pi x), cos(2 pi x)) run on
// the FP32 fraction; sums are FP32: blocks of 8 terms summed plainly, the
// block sums added with Kahan compensation.
#include <type_traits>

#include "fourier_device.h"

namespace rbe {

constexpr int kModesPerBlock = 256;
// Terms summed in plain FP32 before their sum joins the Kahan-compensated
// total (FP32C kernels).
constexpr int kSumBlock = 8;

void fill_turn_table(double2 *host, int n) {
  const long double two_pi = 6.283185307179586476925286766559005768L;
  for (int k = 0; k < n; ++k) {
    const long double a = two_pi * (long double)k / (long double)n;
    host[k] = make_double2((double)sinl(a), (double)cosl(a));
  }
}

__global__ void k_modes_to_double(int P, const int32_t *__restrict__ m, double *__restrict__ mkd) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l < 3 * P) mkd[l] = (double)m[l];
}

void launch_modes_to_double(int P, const int32_t *m, double *mkd, hipStream_t st) {
  k_modes_to_double<<<(3 * P + 255) / 256, 256, 0, st>>>(P, m, mkd);
}

// ---------------------------------------------------------------------------
// structure factor partial sums
// ---------------------------------------------------------------------------
// A wave holds 64 consecutive modes. The last wave of a mode set whose size
// is not a multiple of 64 holds a < 64: its lanes then split as rep lanes per
// mode (rep the largest power of two with rep a <= 64), each taking every
// rep-th particle of the chunk, and the rep partial sums of a mode are added
// by a fixed butterfly, so that wave does 1/rep of the trips instead of all.
__device__ inline int wave_rep(int a) {
  int rep = 1;
  while (2 * rep * a <= 64) rep *= 2;
  return rep;
}

__global__ void __launch_bounds__(kModesPerBlock) k_rho_partial_f64(const int32_t *__restrict__ nq_ptr, int P,
                                                                     int nchunk_max,
                                                                     const double4 *__restrict__ sq,
                                                                     const double *__restrict__ mkd,
                                                                     const double2 *__restrict__ turn_tab,
                                                                     double2 *__restrict__ part,
                                                                     const int32_t *__restrict__ run_count) {
  if (run_count && *run_count > 0) return;  // the segments' kernel has the table
  static_assert(kModesPerBlock == kTurnTable, "one table entry per thread");
  __shared__ double2 tab[kTurnTable];
  __shared__ double4 rec[kModesPerBlock];  // the chunk's records, staged a round at a time
  __shared__ double2 shares[kModesPerBlock];
  const int64_t nq = *nq_ptr;
  int nchunks;
  const int chunk = rho_layout(nq, P, nchunk_max, &nchunks);
  if ((int)blockIdx.x >= nchunks) return;  // uniform over the block
  tab[threadIdx.x] = turn_tab[threadIdx.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // waves that share a mode set (1, 2 or 4: what P leaves of the block's four),
  // each taking a run of every round's records
  const int sets = blockIdx.y == 0 && P <= 128 ? (P + 63) / 64 : 4, split = 4 / sets;
  const int share = wave / sets;
  const int l0 = blockIdx.y * kModesPerBlock + wave % sets * 64;  // first mode of this wave
  const int a = max(0, min(64, P - l0));  // modes of this wave (0: it only stages records)
  const int64_t j0 = (int64_t)blockIdx.x * chunk;
  const int64_t j1 = min(nq, j0 + chunk);
  // a == 64: one mode per lane; fewer: rep lanes per mode, each taking every
  // rep-th record, added by a fixed butterfly
  const int rep = a == 64 ? 1 : (a > 0 ? wave_rep(a) : 64);
  const int mi = lane / rep, ph = lane % rep;
  const bool active = mi < a;
  const int l = l0 + (active ? mi : 0);
  double mx = 0.0, my = 0.0, mz = 0.0;
  if (a > 0) {
    mx = kTurnTable * mkd[l];
    my = kTurnTable * mkd[P + l];
    mz = kTurnTable * mkd[2 * P + l];
  }
  double re = 0.0, im = 0.0;
  for (int64_t b = j0; b < j1; b += kModesPerBlock) {
    const int cnt = (int)min((int64_t)kModesPerBlock, j1 - b);
    __syncthreads();  // the table is written; the previous round is no longer read
    if ((int)threadIdx.x < cnt) rec[threadIdx.x] = sq[b + threadIdx.x];
    __syncthreads();
    if (a == 0) continue;
    const int run = (cnt + split - 1) / split, end = min(cnt, (share + 1) * run);
#pragma unroll 4
    for (int u = share * run + ph; u < end; u += rep) {
      const double4 r = rec[u];
      double sn, cs;
      sincos_phase_f64(phase_dot(mx, my, mz, r.x, r.y, r.z), tab, &sn, &cs);
      re = fma(r.w, cs, re);
      im = fma(r.w, sn, im);
    }
  }
  if (split > 1) {
    shares[threadIdx.x] = make_double2(re, im);
    __syncthreads();
    if (share) return;
    for (int k = 1; k < split; ++k) {
      re += shares[threadIdx.x + k * sets * 64].x;
      im += shares[threadIdx.x + k * sets * 64].y;
    }
  }
  if (a == 0) return;
  for (int o = rep >> 1; o > 0; o >>= 1) {
    re += __shfl_xor(re, o, 64);
    im += __shfl_xor(im, o, 64);
  }
  if (active && ph == 0) part[(int64_t)blockIdx.x * P + l] = make_double2(re, im);
}

// Record: x, y, z as doubles, the FP32 charge in the low word of w.
__device__ inline float rec_q(const double4 &r) { return __int_as_float(__double2loint(r.w)); }

__global__ void __launch_bounds__(kModesPerBlock) k_rho_partial_f32c(const int32_t *__restrict__ nq_ptr, int P,
                                                                      int nchunk_max,
                                                                      const double4 *__restrict__ sq,
                                                                      const double *__restrict__ mkd,
                                                                      double2 *__restrict__ part) {
  __shared__ double4 rec[kModesPerBlock];
  const int64_t nq = *nq_ptr;
  int nchunks;
  const int chunk = rho_layout(nq, P, nchunk_max, &nchunks);
  if ((int)blockIdx.x >= nchunks) return;  // uniform over the block
  const int lane = threadIdx.x & 63;
  const int l0 = blockIdx.y * kModesPerBlock + (threadIdx.x & ~63);
  // a wave past the last mode still stages records for the others
  const int a = max(0, min(64, P - l0));
  const int64_t j0 = (int64_t)blockIdx.x * chunk;
  const int64_t j1 = min(nq, j0 + chunk);
  const int rep = a == 64 ? 1 : (a > 0 ? wave_rep(a) : 64);
  const int mi = lane / rep, ph = lane % rep;
  const bool active = mi < a;
  const int l = l0 + (active ? mi : 0);
  double mx = 0.0, my = 0.0, mz = 0.0;
  if (a > 0) {
    mx = mkd[l];
    my = mkd[P + l];
    mz = mkd[2 * P + l];
  }
  float re = 0.f, re_c = 0.f, im = 0.f, im_c = 0.f;
  auto term = [&](const double4 &r, float &br, float &bi) {
    const float t = turn_f32(mx, my, mz, r.x, r.y, r.z);
    const float q = rec_q(r);
    br = fmaf(q, __builtin_amdgcn_cosf(t), br);
    bi = fmaf(q, __builtin_amdgcn_sinf(t), bi);
  };
  for (int64_t b = j0; b < j1; b += kModesPerBlock) {
    const int cnt = (int)min((int64_t)kModesPerBlock, j1 - b);
    __syncthreads();  // the previous round's records are no longer read
    if ((int)threadIdx.x < cnt) {
      const double4 s = sq[b + threadIdx.x];
      rec[threadIdx.x] = make_double4(s.x, s.y, s.z, __hiloint2double(0, __float_as_int((float)s.w)));
    }
    __syncthreads();
    if (a == 0) continue;
    if (rep == 1) {
      // blocks of kSumBlock terms summed in FP32, each block sum added to
      // the chunk's sum with Kahan compensation
      int u = 0;
      for (; u + kSumBlock <= cnt; u += kSumBlock) {
        double4 r[kSumBlock];  // all loads issued before the arithmetic
#pragma unroll
        for (int v = 0; v < kSumBlock; ++v) r[v] = rec[u + v];
        float br = 0.f, bi = 0.f;
#pragma unroll
        for (int v = 0; v < kSumBlock; ++v) term(r[v], br, bi);
        kahan_add(re, re_c, br);
        kahan_add(im, im_c, bi);
      }
      float br = 0.f, bi = 0.f;
      for (; u < cnt; ++u) term(rec[u], br, bi);
      kahan_add(re, re_c, br);
      kahan_add(im, im_c, bi);
    } else {
      for (int u = ph; u < cnt; u += rep) {
        const double4 r = rec[u];
        const float t = turn_f32(mx, my, mz, r.x, r.y, r.z);
        kahan_fma(re, re_c, rec_q(r), __builtin_amdgcn_cosf(t));
        kahan_fma(im, im_c, rec_q(r), __builtin_amdgcn_sinf(t));
      }
    }
  }
  if (a == 0) return;
  double dre = (double)re - (double)re_c, dim = (double)im - (double)im_c;
  for (int o = rep >> 1; o > 0; o >>= 1) {
    dre += __shfl_xor(dre, o, 64);
    dim += __shfl_xor(dim, o, 64);
  }
  if (active && ph == 0) part[(int64_t)blockIdx.x * P + l] = make_double2(dre, dim);
}

// rho_l = sum over chunks (fixed order: thread-strided FP64 sums, a fixed
// butterfly in each wave, then the waves in index order). Also forms the
// gather coefficients of each mode.
__device__ inline void put_rho(int l, int P, double re, double im, const double *__restrict__ mkd,
                               const double *__restrict__ w, double kc, double *__restrict__ rho,
                               GatherMode *__restrict__ modes, double *__restrict__ rho_out) {
  rho[l] = re;
  rho[P + l] = im;
  if (rho_out) {
    rho_out[l] = re;
    rho_out[P + l] = im;
  }
  GatherMode gm;
  gm.mx = mkd[l];
  gm.my = mkd[P + l];
  gm.mz = mkd[2 * P + l];
  const double wl = kc * w[l];
  gm.a = wl * im;
  gm.b = wl * re;
  gather_floats(gm);
  modes[l] = gm;
}
constexpr int kRhoFinalThreads = 256;
__global__ void __launch_bounds__(kRhoFinalThreads) k_rho_final(const int32_t *__restrict__ nq_ptr, int nchunk_max, int P,
                                                                const double2 *__restrict__ part,
                                                                const double *__restrict__ mkd,
                                                                const double *__restrict__ w, double kc,
                                                                double *__restrict__ rho,
                                                                GatherMode *__restrict__ modes,
                                                                double *__restrict__ rho_out,
                                                                const int32_t *__restrict__ run_count) {
  if (run_count && *run_count > 0) return;
  __shared__ double2 wsum[kRhoFinalThreads / 64];
  int nchunks;
  (void)rho_layout(*nq_ptr, P, nchunk_max, &nchunks);
  const int l = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double re = 0.0, im = 0.0;
#pragma unroll 4
  for (int c = threadIdx.x; c < nchunks; c += kRhoFinalThreads) {
    const double2 v = part[(int64_t)c * P + l];
    re += v.x;
    im += v.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    re += __shfl_xor(re, o, 64);
    im += __shfl_xor(im, o, 64);
  }
  if (lane == 0) wsum[wave] = make_double2(re, im);
  __syncthreads();
  if (threadIdx.x == 0) {
    re = 0.0;
    im = 0.0;
    for (int k = 0; k < kRhoFinalThreads / 64; ++k) {
      re += wsum[k].x;
      im += wsum[k].y;
    }
    put_rho(l, P, re, im, mkd, w, kc, rho, modes, rho_out);
  }
}

// The same sums, in the same order, with a thread per mode where at most
// kRhoFlat chunks are possible (many modes of few particles: an Ewald lattice):
// a block per mode spends its time on being launched, 92,000 modes of 6 chunks
// 98 us, now 7.6.
constexpr int kRhoFlat = 16;
__global__ void __launch_bounds__(256) k_rho_final_flat(const int32_t *__restrict__ nq_ptr, int nchunk_max, int P,
                                                        const double2 *__restrict__ part,
                                                        const double *__restrict__ mkd, const double *__restrict__ w,
                                                        double kc, double *__restrict__ rho,
                                                        GatherMode *__restrict__ modes, double *__restrict__ rho_out,
                                                        const int32_t *__restrict__ run_count) {
  if (run_count && *run_count > 0) return;
  const int l = blockIdx.x * 256 + threadIdx.x;
  if (l >= P) return;
  int nchunks;
  (void)rho_layout(*nq_ptr, P, nchunk_max, &nchunks);
  double2 v[kRhoFlat];
#pragma unroll
  for (int c = 0; c < kRhoFlat; ++c) v[c] = c < nchunks ? part[(int64_t)c * P + l] : make_double2(0.0, 0.0);
#pragma unroll
  for (int o = kRhoFlat / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int c = 0; c < o; ++c) {
      v[c].x += v[c + o].x;
      v[c].y += v[c + o].y;
    }
  }
  put_rho(l, P, v[0].x, v[0].y, mkd, w, kc, rho, modes, rho_out);
}


// ---------------------------------------------------------------------------
// tables with columns: segments of modes (kernels.h, ModeRuns)
// ---------------------------------------------------------------------------
// A segment starts at mode l unless l - 1 is its predecessor in m_z and the
// boundary of two segments does not lie between them.
__device__ inline int run_place(int mz) {
  const int r = mz % kRunLen;
  return r < 0 ? r + kRunLen : r;
}
__device__ inline bool run_head(int P, const int32_t *__restrict__ m, int l) {
  if (l >= P) return false;
  if (l == 0 || m[l] != m[l - 1] || m[P + l] != m[P + l - 1]) return true;
  return (int64_t)m[2 * P + l] != (int64_t)m[2 * P + l - 1] + 1 || run_place(m[2 * P + l]) == 0;
}
// Segments that start in each block's kRunsThreads modes; then, with the sums
// over the blocks before, their records.
__global__ void __launch_bounds__(kRunsThreads) k_run_heads(int P, const int32_t *__restrict__ m, ModeRuns R) {
  const int c = __syncthreads_count(run_head(P, m, blockIdx.x * kRunsThreads + threadIdx.x));
  if (threadIdx.x == 0) R.heads[blockIdx.x] = c;
}
__global__ void __launch_bounds__(kRunsThreads) k_run_segments(int P, const int32_t *__restrict__ m, ModeRuns R) {
  __shared__ int wsum[kRunsThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l = blockIdx.x * kRunsThreads + tid;
  const bool head = run_head(P, m, l);
  const uint64_t heads = __builtin_amdgcn_ballot_w64(head);
  if (lane == 0) wsum[wave] = __popcll(heads);
  __syncthreads();
  int at = 0, total = 0;
  for (int b = 0; b < (int)gridDim.x; ++b) {
    if (b < (int)blockIdx.x) at += R.heads[b];
    total += R.heads[b];
  }
  for (int k = 0; k < wave; ++k) at += wsum[k];
  at += __popcll(heads & ((1ull << lane) - 1ull));
  const bool fits = total <= R.cap;
  if (head && fits) {
    const int mz = m[2 * P + l];
    R.first[at] = l;
    double *r = R.rec + (int64_t)at * kRunRec;
    r[0] = (double)m[l];
    r[1] = (double)m[P + l];
    r[2] = (double)mz + (kRunHalf - run_place(mz));
    r[3] = (double)run_place(mz);
  }
  if (l == 0) {
    if (fits) R.first[total] = P;
    *R.count = fits ? total : 0;
  }
}

void launch_mode_runs(int P, const int32_t *m, const ModeRuns &runs, hipStream_t st) {
  const unsigned nb = (unsigned)((P + kRunsThreads - 1) / kRunsThreads);
  k_run_heads<<<nb, kRunsThreads, 0, st>>>(P, m, runs);
  k_run_segments<<<nb, kRunsThreads, 0, st>>>(P, m, runs);
}

// Blocks of kRunBlockSegs segments times chunks of particles: as many chunks
// as kRunBlocks holds, of at least 16 particles.
__device__ inline int run_chunks(int64_t nq, int nsb, int *len) {
  const int64_t most = max(1, kRunBlocks / nsb);
  const int64_t nc = min(most, max((int64_t)1, (nq + 15) / 16));
  *len = (int)((nq + nc - 1) / nc);
  return (int)nc;
}
static int run_grid(int cap) { return std::max(kRunBlocks, (cap + kRunBlockSegs - 1) / kRunBlockSegs); }

// exp(2 pi i u s_z), u = 1..kRunHalf, of a particle: (cos, sin) of a power.
__device__ inline double2 run_power(int u, double sz, const double2 *tab) {
  double2 z;
  sincos_phase_f64((double)u * (kTurnTable * sz), tab, &z.y, &z.x);
  return z;
}

// Partial sums of the segments: a lane has two of them, the block's records
// and powers are staged in LDS (half of a wave's time at one segment a lane
// would go to reading them). Of a pair of modes u off the centre only the four
// real products with the power are summed; the modes' sums are their sums and
// differences, formed once at the end: 2 FP64 operations a mode and particle
// and 18 a segment for its centre, 4.1 where the general kernel has 19.
// Bound by FP64 issue and the LDS reads alike: 4,000 ions and the 92,000 modes
// of their Ewald lattice 82 us, 320 by the general kernel. Twice the blocks
// (more chunks) save 5 us here and cost 7 in the final sums.
__global__ void __launch_bounds__(kRunBlockSegs / 2) __attribute__((amdgpu_waves_per_eu(4)))
k_rho_runs(const int32_t *__restrict__ nq_ptr, const int32_t *__restrict__ count, const double *__restrict__ seg,
           const double4 *__restrict__ sq, const double2 *__restrict__ turn_tab, double2 *__restrict__ part) {
  constexpr int T = kRunBlockSegs / 2, kStage = T / 2;
  static_assert(T == kTurnTable && kRunHalf == 4, "one table entry per thread, two threads a record");
  __shared__ double2 tab[kTurnTable];
  __shared__ double4 rec[kStage];
  __shared__ double2 pow[kStage][kRunHalf];
  const int nseg = *count;
  if (nseg <= 0) return;  // uniform over the grid
  const int nsb = (nseg + kRunBlockSegs - 1) / kRunBlockSegs;
  const int64_t nq = *nq_ptr;
  int len;
  const int nc = run_chunks(nq, nsb, &len);
  const int chunk = blockIdx.x / nsb, sb = blockIdx.x % nsb;
  if (chunk >= nc) return;  // uniform over the block
  const int tid = threadIdx.x;
  tab[tid] = turn_tab[tid];
  double mx[2], my[2], mz[2], c0[2], s0[2], cc[2][kRunHalf], ss[2][kRunHalf], sc[2][kRunHalf], cs[2][kRunHalf];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int sg = min(sb * kRunBlockSegs + v * T + tid, nseg - 1);
    const double *r = seg + (int64_t)sg * kRunRec;
    mx[v] = kTurnTable * r[0];
    my[v] = kTurnTable * r[1];
    mz[v] = kTurnTable * r[2];
    c0[v] = s0[v] = 0.0;
#pragma unroll
    for (int u = 0; u < kRunHalf; ++u) cc[v][u] = ss[v][u] = sc[v][u] = cs[v][u] = 0.0;
  }
  const int64_t j0 = (int64_t)chunk * len, j1 = min(nq, j0 + len);
  for (int64_t b = j0; b < j1; b += kStage) {
    const int cnt = (int)min((int64_t)kStage, j1 - b);
    __syncthreads();  // the table is written; the previous round is no longer read
    if ((tid >> 1) < cnt) {
      const double4 r = sq[b + (tid >> 1)];
      const int u = (tid & 1) * 2;
      if (u == 0) rec[tid >> 1] = r;
      pow[tid >> 1][u] = run_power(u + 1, r.z, tab);
      pow[tid >> 1][u + 1] = run_power(u + 2, r.z, tab);
    }
    __syncthreads();
    for (int k = 0; k < cnt; ++k) {
      const double4 r = rec[k];
      double2 z[kRunHalf];
#pragma unroll
      for (int u = 0; u < kRunHalf; ++u) z[u] = pow[k][u];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        double sn, c;
        sincos_phase_f64(phase_dot(mx[v], my[v], mz[v], r.x, r.y, r.z), tab, &sn, &c);
        const double qc = r.w * c, qs = r.w * sn;
        c0[v] += qc;
        s0[v] += qs;
#pragma unroll
        for (int u = 0; u < kRunHalf; ++u) {
          cc[v][u] = fma(qc, z[u].x, cc[v][u]);
          ss[v][u] = fma(qs, z[u].y, ss[v][u]);
          sc[v][u] = fma(qs, z[u].x, sc[v][u]);
          cs[v][u] = fma(qc, z[u].y, cs[v][u]);
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int sg = sb * kRunBlockSegs + v * T + tid;
    if (sg >= nseg) continue;
    double2 *out = part + (int64_t)chunk * kRunLen * nseg + sg;
    out[0] = make_double2(c0[v], s0[v]);
#pragma unroll
    for (int u = 0; u < kRunHalf; ++u) {
      out[(int64_t)(2 * u + 1) * nseg] = make_double2(cc[v][u], ss[v][u]);
      out[(int64_t)(2 * u + 2) * nseg] = make_double2(sc[v][u], cs[v][u]);
    }
  }
}

// One thread per segment and its centre (k = 0) or pair (k = u): the chunks'
// sums in order, the structure factors of the modes that exist, and the
// segment's gather coefficients (zero for the modes it lacks).
__global__ void __launch_bounds__(256) k_rho_runs_final(const int32_t *__restrict__ nq_ptr, int P,
                                                        const int32_t *__restrict__ count,
                                                        const int32_t *__restrict__ first,
                                                        const double2 *__restrict__ part,
                                                        const double *__restrict__ w, double kc,
                                                        double *__restrict__ seg, double *__restrict__ rho,
                                                        double *__restrict__ rho_out) {
  const int nseg = *count;
  const int64_t it = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (it >= (int64_t)nseg * (kRunHalf + 1)) return;
  const int u = (int)(it / nseg), sg = (int)(it % nseg);
  int len;
  const int nc = run_chunks(*nq_ptr, (nseg + kRunBlockSegs - 1) / kRunBlockSegs, &len);
  double *r = seg + (int64_t)sg * kRunRec;
  const int off = (int)r[3];  // the segment's first mode is at this place of its kRunLen
  const int f = first[sg], cnt = first[sg + 1] - f;
  double2 A = make_double2(0.0, 0.0), B = A;
  const int ka = u ? 2 * u - 1 : 0;
  const double2 *pa = part + (int64_t)ka * nseg + sg;
#pragma unroll 4
  for (int c = 0; c < nc; ++c) {
    const double2 va = pa[(int64_t)c * kRunLen * nseg];
    A.x += va.x;
    A.y += va.y;
    if (u) {
      const double2 vb = pa[((int64_t)c * kRunLen + 1) * nseg];
      B.x += vb.x;
      B.y += vb.y;
    }
  }
  // structure factor of the segment's mode at place k, and its coefficients
  auto put = [&](int k, double re, double im) {
    if (k < off || k >= off + cnt) return make_double2(0.0, 0.0);
    const int l = f + k - off;
    rho[l] = re;
    rho[P + l] = im;
    if (rho_out) {
      rho_out[l] = re;
      rho_out[P + l] = im;
    }
    const double wl = kc * w[l];
    return make_double2(wl * im, wl * re);
  };
  if (u == 0) {
    const double2 g = put(kRunHalf, A.x, A.y);
    r[4] = g.x;
    r[5] = g.y;
  } else {
    const double2 g = put(kRunHalf + u, A.x - A.y, B.x + B.y), h = put(kRunHalf - u, A.x + A.y, B.x - B.y);
    r += 8 + 4 * (u - 1);
    r[0] = g.x + h.x;
    r[1] = g.y - h.y;
    r[2] = g.x - h.x;
    r[3] = g.y + h.y;
  }
}

void launch_rho_partial(int prec, const int32_t *nq, int64_t nq_max, int P, const double4 *sq,
                        const FourierBuffers &fb, hipStream_t st) {
  const ModeRuns &R = fb.runs;
  if (R.cap)
    k_rho_runs<<<(unsigned)run_grid(R.cap), kRunBlockSegs / 2, 0, st>>>(nq, R.count, R.rec, sq, fb.turn_tab, R.part);
  const int nchunks = rho_max_chunks(nq_max, P, fb.nchunk_max);
  dim3 grid((unsigned)nchunks, (unsigned)((P + kModesPerBlock - 1) / kModesPerBlock));
  if (prec == RBE_FP32C)
    k_rho_partial_f32c<<<grid, kModesPerBlock, 0, st>>>(nq, P, fb.nchunk_max, sq, fb.mkd, fb.part);
  else
    k_rho_partial_f64<<<grid, kModesPerBlock, 0, st>>>(nq, P, fb.nchunk_max, sq, fb.mkd, fb.turn_tab, fb.part,
                                                         R.cap ? R.count : nullptr);
}

void launch_rho_final(const int32_t *nq, int64_t nq_max, int P, const FourierBuffers &fb, const double *w, double kc,
                      double *rho_out, hipStream_t st) {
  const ModeRuns &R = fb.runs;
  if (R.cap)
    k_rho_runs_final<<<(unsigned)((R.cap * (int64_t)(kRunHalf + 1) + 255) / 256), 256, 0, st>>>(
        nq, P, R.count, R.first, R.part, w, kc, R.rec, fb.rho, rho_out);
  const int32_t *rc = R.cap ? R.count : nullptr;
  if (rho_max_chunks(nq_max, P, fb.nchunk_max) <= kRhoFlat)
    k_rho_final_flat<<<(P + 255) / 256, 256, 0, st>>>(nq, fb.nchunk_max, P, fb.part, fb.mkd, w, kc, fb.rho, fb.modes,
                                                      rho_out, rc);
  else
    k_rho_final<<<P, kRhoFinalThreads, 0, st>>>(nq, fb.nchunk_max, P, fb.part, fb.mkd, w, kc, fb.rho, fb.modes,
                                                rho_out, rc);
}

// ---------------------------------------------------------------------------
// force gather (adds F^F into f for the charged range)
// ---------------------------------------------------------------------------
// Mode groups: blockIdx.y = g sums the modes [g M, min(P, (g + 1) M)); with
// one group the force is applied here, with several the group's sums go to
// gpart[g * stride + i] and k_gather_reduce adds the groups in order.
__global__ void __launch_bounds__(kTurnTable) k_gather_f64(const int32_t *__restrict__ nq_ptr, int P, int M,
                                                           const double4 *__restrict__ sq,
                                                           const GatherMode *__restrict__ modes,
                                                           const double2 *__restrict__ turn_tab, double kx,
                                                           double ky, double kz, double *__restrict__ fx,
                                                           double *__restrict__ fy, double *__restrict__ fz,
                                                           double4 *__restrict__ gpart, int64_t stride,
                                                           const int32_t *__restrict__ run_count) {
  if (run_count && *run_count > 0) return;
  __shared__ double2 tab[kTurnTable];
  const int64_t nq = *nq_ptr;
  if ((int64_t)blockIdx.x * blockDim.x >= nq) return;  // uniform over the block
  tab[threadIdx.x] = turn_tab[threadIdx.x];
  __syncthreads();
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nq) return;
  const double4 s = sq[i];
  const double sx = kTurnTable * s.x, sy = kTurnTable * s.y, sz = kTurnTable * s.z;
  double gx = 0.0, gy = 0.0, gz = 0.0;
  const int lb = blockIdx.y * M, le = min(P, lb + M);
#pragma unroll 4
  for (int l = lb; l < le; ++l) {
    const GatherMode gm = modes[l];
    double sn, cs;
    sincos_phase_f64(phase_dot(gm.mx, gm.my, gm.mz, sx, sy, sz), tab, &sn, &cs);
    const double g = gm.a * cs - gm.b * sn;  // w Im(exp(-i theta) rho)
    gx = fma(g, gm.mx, gx);
    gy = fma(g, gm.my, gy);
    gz = fma(g, gm.mz, gz);
  }
  if (gpart) {
    gpart[blockIdx.y * stride + i] = make_double4(gx, gy, gz, 0.0);
    return;
  }
  const double q = s.w;
  fx[i] -= q * kx * gx;
  fy[i] -= q * ky * gy;
  fz[i] -= q * kz * gz;
}

// The same sums over segments: with A_u = a_u + i b_u and Z = exp(2 pi i
// s_z), the segment's sum of g is Re(e S), S = sum_u A_u Z^u, and that of u g
// is Re(e W), W = sum_u u A_u Z^u, e the centre's exp(i k . r). The powers are
// the particle's own, the pairs' coefficients come added and subtracted: 4
// FP64 operations a mode and 25 a segment, 6.8 a mode where the general kernel
// has 22. Two particles a lane, so that a segment's scalar loads (three cache
// lines, waited for in full) serve 128 particles; the four waves of a block
// take a quarter of the group's segments each, and their sums are added in
// order. Bound by FP64 issue: 4,000 ions, 92,000 modes 122 us, 199 with one
// particle a lane, 440 by the general kernel.
constexpr int kRunGather = 128;  // particles per block
__global__ void __launch_bounds__(256) k_gather_runs(const int32_t *__restrict__ nq_ptr,
                                                     const int32_t *__restrict__ count,
                                                     const double *__restrict__ seg, const double4 *__restrict__ sq,
                                                     const double2 *__restrict__ turn_tab, double kx, double ky,
                                                     double kz, double *__restrict__ fx, double *__restrict__ fy,
                                                     double *__restrict__ fz, double4 *__restrict__ gpart,
                                                     int64_t stride) {
  static_assert(kTurnTable == 256, "one table entry per thread");
  __shared__ double2 tab[kTurnTable];
  __shared__ double sums[4][3][kRunGather];
  const int64_t nq = *nq_ptr, i0 = blockIdx.x * (int64_t)kRunGather;
  const int nseg = *count;
  if (nseg <= 0 || i0 >= nq) return;  // uniform over the block
  tab[threadIdx.x] = turn_tab[threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double s[2][3], gx[2], gy[2], gz[2];
  double2 z[2][kRunHalf], uz[2][kRunHalf];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const double4 r = sq[min(i0 + 64 * v + lane, nq - 1)];
    s[v][0] = kTurnTable * r.x;
    s[v][1] = kTurnTable * r.y;
    s[v][2] = kTurnTable * r.z;
#pragma unroll
    for (int u = 0; u < kRunHalf; ++u) {
      z[v][u] = run_power(u + 1, r.z, tab);
      uz[v][u] = make_double2((u + 1) * z[v][u].x, (u + 1) * z[v][u].y);
    }
    gx[v] = gy[v] = gz[v] = 0.0;
  }
  const int parts = 4 * gridDim.y, M = (nseg + parts - 1) / parts;
  const int lb = (blockIdx.y * 4 + wave) * M, le = min(nseg, lb + M);
  for (int l = lb; l < le; ++l) {
    struct Rec {
      double v[kRunRec];
    };
    const Rec r = ((const Rec *)seg)[l];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      double sn, cs;
      sincos_phase_f64(phase_dot(r.v[0], r.v[1], r.v[2], s[v][0], s[v][1], s[v][2]), tab, &sn, &cs);
      double sr = r.v[4], si = r.v[5], wr = 0.0, wi = 0.0;
#pragma unroll
      for (int u = 0; u < kRunHalf; ++u) {
        const double pa = r.v[8 + 4 * u], mb = r.v[9 + 4 * u], ma = r.v[10 + 4 * u], pb = r.v[11 + 4 * u];
        sr = fma(pa, z[v][u].x, sr);
        sr = fma(-mb, z[v][u].y, sr);
        si = fma(ma, z[v][u].y, si);
        si = fma(pb, z[v][u].x, si);
        wr = fma(ma, uz[v][u].x, wr);
        wr = fma(-pb, uz[v][u].y, wr);
        wi = fma(pa, uz[v][u].y, wi);
        wi = fma(mb, uz[v][u].x, wi);
      }
      const double g = fma(sr, cs, -(si * sn));
      gx[v] = fma(g, r.v[0], gx[v]);
      gy[v] = fma(g, r.v[1], gy[v]);
      gz[v] = fma(g, r.v[2], gz[v]);
      gz[v] = fma(wr, cs, gz[v]);
      gz[v] = fma(-wi, sn, gz[v]);
    }
  }
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    sums[wave][0][64 * v + lane] = gx[v];
    sums[wave][1][64 * v + lane] = gy[v];
    sums[wave][2][64 * v + lane] = gz[v];
  }
  __syncthreads();
  const int64_t i = i0 + threadIdx.x;
  if (threadIdx.x >= kRunGather || i >= nq) return;
  double g[3];
#pragma unroll
  for (int d = 0; d < 3; ++d)
    g[d] = ((sums[0][d][threadIdx.x] + sums[1][d][threadIdx.x]) + sums[2][d][threadIdx.x]) + sums[3][d][threadIdx.x];
  if (gpart) {
    gpart[blockIdx.y * stride + i] = make_double4(g[0], g[1], g[2], 0.0);
    return;
  }
  const double q = sq[i].w;
  fx[i] -= q * kx * g[0];
  fy[i] -= q * ky * g[1];
  fz[i] -= q * kz * g[2];
}

// Two charged particles per thread (i and i + 256 of the block's 512); every
// lane reads the same mode at a time (wave-uniform scalar loads, which
// deliver a record once per wave), and each mode read serves both particles.
// Staging the modes in LDS instead measured slower: the broadcast LDS reads
// cost more than the load latency they hide.
constexpr int kGatherThreads = 256;
constexpr int kGatherPerBlock = 2 * kGatherThreads;
__global__ void __launch_bounds__(kGatherThreads) k_gather_f32c(const int32_t *__restrict__ nq_ptr, int P, int M,
                                                                const double4 *__restrict__ sq,
                                                                const GatherMode *__restrict__ modes, double kx,
                                                                double ky, double kz, double *__restrict__ fx,
                                                                double *__restrict__ fy, double *__restrict__ fz,
                                                                double4 *__restrict__ gpart, int64_t stride) {
  const int64_t nq = *nq_ptr;
  const int64_t i = blockIdx.x * (int64_t)kGatherPerBlock + threadIdx.x, i2 = i + kGatherThreads;
  if (i >= nq) return;
  const bool two = i2 < nq;
  const double4 s = sq[i], s2 = two ? sq[i2] : s;
  float gx = 0.f, gy = 0.f, gz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
  float hx = 0.f, hy = 0.f, hz = 0.f, dx = 0.f, dy = 0.f, dz = 0.f;
  auto term = [&](int l, float &bx, float &by, float &bz, float &ex, float &ey, float &ez) {
    const GatherMode gm = modes[l];
    const float t = turn_f32(gm.mx, gm.my, gm.mz, s.x, s.y, s.z);
    const float t2 = turn_f32(gm.mx, gm.my, gm.mz, s2.x, s2.y, s2.z);
    const float g = fmaf(gm.af, __builtin_amdgcn_cosf(t), -gm.bf * __builtin_amdgcn_sinf(t));
    const float g2 = fmaf(gm.af, __builtin_amdgcn_cosf(t2), -gm.bf * __builtin_amdgcn_sinf(t2));
    bx = fmaf(g, gm.mxf, bx);
    by = fmaf(g, gm.myf, by);
    bz = fmaf(g, gm.mzf, bz);
    ex = fmaf(g2, gm.mxf, ex);
    ey = fmaf(g2, gm.myf, ey);
    ez = fmaf(g2, gm.mzf, ez);
  };
  // blocks of kSumBlock modes summed in FP32, each block sum added with
  // Kahan compensation (a group's first mode is a multiple of kSumBlock, so
  // the blocks run over the modes in order and only the last one is short)
  const int lb = blockIdx.y * M, le = min(P, lb + M);
  int l = lb;
  for (; l + kSumBlock <= le; l += kSumBlock) {
    float bx = 0.f, by = 0.f, bz = 0.f, ex = 0.f, ey = 0.f, ez = 0.f;
#pragma unroll
    for (int u = 0; u < kSumBlock; ++u) term(l + u, bx, by, bz, ex, ey, ez);
    kahan_add(gx, cx, bx);
    kahan_add(gy, cy, by);
    kahan_add(gz, cz, bz);
    kahan_add(hx, dx, ex);
    kahan_add(hy, dy, ey);
    kahan_add(hz, dz, ez);
  }
  {
    float bx = 0.f, by = 0.f, bz = 0.f, ex = 0.f, ey = 0.f, ez = 0.f;
    for (; l < le; ++l) term(l, bx, by, bz, ex, ey, ez);
    kahan_add(gx, cx, bx);
    kahan_add(gy, cy, by);
    kahan_add(gz, cz, bz);
    kahan_add(hx, dx, ex);
    kahan_add(hy, dy, ey);
    kahan_add(hz, dz, ez);
  }
  auto put = [&](int64_t k, const double4 &sk, float ax, float acx, float ay, float acy, float az, float acz) {
    const double sx = (double)ax - (double)acx, sy = (double)ay - (double)acy, sz = (double)az - (double)acz;
    if (gpart) {
      gpart[blockIdx.y * stride + k] = make_double4(sx, sy, sz, 0.0);
      return;
    }
    const double q = sk.w;
    fx[k] -= q * kx * sx;
    fy[k] -= q * ky * sy;
    fz[k] -= q * kz * sz;
  };
  put(i, s, gx, cx, gy, cy, gz, cz);
  if (two) put(i2, s2, hx, dx, hy, dy, hz, dz);
}

// Few particles: the W waves of a block share 64 of them, each taking every
// W-th block of kSumBlock modes, and the waves' sums are added in order (FP64)
// or, of W such blocks at a time, each block's with Kahan compensation in the
// order of the modes (FP32C: the same bits as a lane that sums them one after
// another). A lane on its own waits for 100 modes' loads and chains one after
// another: 2,000 to 10,000 particles, 100 modes, FP64 21 -> 6.5 us, FP32C 32 ->
// 5.6; 4,000 and 92,000 modes, FP32C 490 -> 292.
template <bool F32, int W>
__global__ void __launch_bounds__(64 * W) k_gather_waves(const int32_t *__restrict__ nq_ptr, int P, int M,
                                                         const double4 *__restrict__ sq,
                                                         const GatherMode *__restrict__ modes,
                                                         const double2 *__restrict__ turn_tab, double kx, double ky,
                                                         double kz, double *__restrict__ fx, double *__restrict__ fy,
                                                         double *__restrict__ fz, double4 *__restrict__ gpart,
                                                         int64_t stride, const int32_t *__restrict__ run_count) {
  if (run_count && *run_count > 0) return;
  using T = std::conditional_t<F32, float, double>;
  __shared__ double2 tab[F32 ? 1 : kTurnTable];
  __shared__ T sums[W][3][64];
  const int64_t nq = *nq_ptr, i0 = blockIdx.x * (int64_t)64;
  if (i0 >= nq) return;  // uniform over the block
  if (!F32) {
    for (int k = threadIdx.x; k < kTurnTable; k += 64 * W) tab[k] = turn_tab[k];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double4 s = sq[min(i0 + lane, nq - 1)];
  const double sx = kTurnTable * s.x, sy = kTurnTable * s.y, sz = kTurnTable * s.z;
  const int first = blockIdx.y * M, end = min(P, first + M);
  const int nb = (end - first) / kSumBlock + 1;  // blocks of modes; the last may be empty
  T g[3] = {};
  float sum = 0.f, comp = 0.f;  // FP32C: component wave of the lane's particle
  for (int b0 = 0; b0 < nb; b0 += W) {
    const int lb = first + (b0 + wave) * kSumBlock, le = min(end, lb + kSumBlock);
    if (F32) g[0] = g[1] = g[2] = 0;
#pragma unroll 4
    for (int l = lb; l < le; ++l) {
      const GatherMode gm = modes[l];
      if constexpr (F32) {
        const float t = turn_f32(gm.mx, gm.my, gm.mz, s.x, s.y, s.z);
        const float h = fmaf(gm.af, __builtin_amdgcn_cosf(t), -gm.bf * __builtin_amdgcn_sinf(t));
        g[0] = fmaf(h, gm.mxf, g[0]);
        g[1] = fmaf(h, gm.myf, g[1]);
        g[2] = fmaf(h, gm.mzf, g[2]);
      } else {
        double sn, cs;
        sincos_phase_f64(phase_dot(gm.mx, gm.my, gm.mz, sx, sy, sz), tab, &sn, &cs);
        const double h = gm.a * cs - gm.b * sn;
        g[0] = fma(h, gm.mx, g[0]);
        g[1] = fma(h, gm.my, g[1]);
        g[2] = fma(h, gm.mz, g[2]);
      }
    }
    if (F32) {
      for (int d = 0; d < 3; ++d) sums[wave][d][lane] = g[d];
      __syncthreads();
      if (wave < 3)
        for (int k = 0; k < W && b0 + k < nb; ++k) kahan_add(sum, comp, (float)sums[k][wave][lane]);
      __syncthreads();
    }
  }
  if (!F32) {
    for (int d = 0; d < 3; ++d) sums[wave][d][lane] = g[d];
    __syncthreads();
  }
  const int64_t i = i0 + lane;
  if (wave >= 3 || i >= nq) return;
  double v;
  if (F32) {
    v = (double)sum - (double)comp;
  } else {
    v = 0.0;
    for (int k = 0; k < W; ++k) v += (double)sums[k][wave][lane];
  }
  if (gpart) {
    ((double *)&gpart[blockIdx.y * stride + i])[wave] = v;
    return;
  }
  double *f = wave == 0 ? fx : wave == 1 ? fy : fz;
  f[i] -= s.w * (wave == 0 ? kx : wave == 1 ? ky : kz) * v;
}

// The groups' sums of each charged particle added in group order (FP64),
// then applied like the single-group gather.
__global__ void __launch_bounds__(256) k_gather_reduce(const int32_t *__restrict__ nq_ptr, int groups,
                                                       int run_groups, const int32_t *__restrict__ run_count,
                                                       int64_t stride,
                                                       const double4 *__restrict__ gpart,
                                                       const double4 *__restrict__ sq, double kx, double ky,
                                                       double kz, double *__restrict__ fx, double *__restrict__ fy,
                                                       double *__restrict__ fz) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= *nq_ptr) return;
  const int G = run_count && *run_count > 0 ? run_groups : groups;
  double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll 4
  for (int g = 0; g < G; ++g) {
    const double4 v = gpart[g * stride + i];
    gx += v.x;
    gy += v.y;
    gz += v.z;
  }
  const double q = sq[i].w;
  fx[i] -= q * kx * gx;
  fy[i] -= q * ky * gy;
  fz[i] -= q * kz * gz;
}

// Mode groups of the gather: one unless the charged range alone gives too few
// blocks to fill the GPU (a small system with many modes, such as the full
// Ewald lattice), then enough groups of M modes (a multiple of the staging
// round) for about 1024 blocks, within the partial-sum buffer.
static int gather_split(int64_t nq_max, int P, const FourierBuffers &fb, int *M) {
  const int64_t pb = (nq_max + 255) / 256;
  *M = P;
  if (!fb.gpart || pb >= 512 || P < 4 * kGatherThreads) return 1;
  int64_t G = (1024 + pb - 1) / pb;
  while (G > 1 && G * pb * 256 > kGatherPartMax) --G;
  const int64_t m = ((P + G - 1) / G + kGatherThreads - 1) / kGatherThreads * kGatherThreads;
  *M = (int)m;
  return (int)((P + m - 1) / m);
}

// Particles up to which the waves of a block share them (k_gather_waves),
// against the other form in us: 100 modes FP64 20,000: 7, 21; 130,000: 20, 23;
// 200,000: 27, 26; 300,000: 38, 31; FP32C 20,000: 8, 32; 200,000: 28, 33;
// 300,000: 40, 37; 500 modes FP64 200,000: 90, 108; FP32C 200,000: 101, 134;
// 300,000: 148, 137.
constexpr int64_t kGatherWavesMost64 = 196608, kGatherWavesMost32 = 262144;
void launch_fourier_gather(int prec, const int32_t *nq, int64_t nq_max, int P, const double4 *sq,
                           const FourierBuffers &fb, const Grid &g, double *fx, double *fy, double *fz,
                           hipStream_t st) {
  if (nq_max <= 0) return;
  const unsigned blocks = (unsigned)((nq_max + 255) / 256);
  const double kx = kTwoPi / g.L[0], ky = kTwoPi / g.L[1], kz = kTwoPi / g.L[2];
  int M;
  const int G = gather_split(nq_max, P, fb, &M);
  double4 *gp = G > 1 ? fb.gpart : nullptr;
  const int64_t stride = (int64_t)blocks * 256;
  // segments: groups for about 1024 blocks, if the particles alone are fewer,
  // of at least eight segments a wave
  const ModeRuns &R = fb.runs;
  const int32_t *rc = R.cap ? R.count : nullptr;
  const int64_t rb = (nq_max + kRunGather - 1) / kRunGather;
  const int64_t rg = gp ? std::max<int64_t>(1, std::min({1024 / rb, kGatherPartMax / stride,
                                                         (int64_t)P / (32 * kRunLen)}))
                        : 1;
  if (R.cap)
    k_gather_runs<<<dim3((unsigned)rb, (unsigned)rg), 256, 0, st>>>(nq, R.count, R.rec, sq, fb.turn_tab, kx, ky, kz,
                                                                    fx, fy, fz, gp, stride);
  const bool f32 = prec == RBE_FP32C;
  if (nq_max <= (f32 ? kGatherWavesMost32 : kGatherWavesMost64)) {
    const auto kernel = f32 ? k_gather_waves<true, 16> : k_gather_waves<false, 16>;
    kernel<<<dim3((unsigned)((nq_max + 63) / 64), (unsigned)G), 1024, 0, st>>>(
        nq, P, M, sq, fb.modes, fb.turn_tab, kx, ky, kz, fx, fy, fz, gp, stride, rc);
  } else if (f32) {
    k_gather_f32c<<<dim3((unsigned)((nq_max + kGatherPerBlock - 1) / kGatherPerBlock), (unsigned)G), kGatherThreads,
                    0, st>>>(nq, P, M, sq, fb.modes, kx, ky, kz, fx, fy, fz, gp, stride);
  } else {
    k_gather_f64<<<dim3(blocks, (unsigned)G), kTurnTable, 0, st>>>(nq, P, M, sq, fb.modes, fb.turn_tab, kx, ky, kz, fx,
                                                                   fy, fz, gp, stride, rc);
  }
  if (G > 1) k_gather_reduce<<<blocks, 256, 0, st>>>(nq, G, (int)rg, rc, stride, gp, sq, kx, ky, kz, fx, fy, fz);
}

}  // namespace rbe
