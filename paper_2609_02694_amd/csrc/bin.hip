// Cell binning: stable counting sort of particles by (species, cell), and
// the reorder of the particle arrays into that order (Sec. 2.2: linked-cell
// reassignment and cell-wise reordering).
//
// key = s * C + (c_z n_y + c_y) n_x + c_x with s = 0 for charged and 1 for
// neutral particles. Charged particles therefore occupy one contiguous range
// [0, start[C]) in cell order, which the Fourier kernels walk directly.
//
// Steps: keys + histogram (integer atomics give exact counts) -> exclusive
// scan -> provisional scatter (atomic slot order, not deterministic) ->
// stable placement: each bucket's entries (input indices) are put in
// increasing order, so a particle's final slot is start[key] + the number of
// bucket members with a smaller input index. The output is a pure function
// of the input, whatever order the atomics took.
//
// The input of a step is the previous step's cell order, so equal keys come
// in runs. A wave takes one atomic per run (its length) and hands out the
// slots of the run in input order; a bucket is then usually already in order
// and its placement a copy (checked per bucket; short buckets out of order are
// sorted by insertion, long ones by counting). Small systems run all steps in
// one block (k_bin_block).
#include <algorithm>

#include "rbe_internal.h"
#include "kernels.h"

namespace rbe {

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_fill_i32<<<(unsigned)blocks, 256, 0, st>>>(p, n, v);
}

__global__ void k_fill_f64(double *p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_f64(double *p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_fill_f64<<<(unsigned)blocks, 256, 0, st>>>(p, n, v);
}

// ---------------------------------------------------------------------------
// keys + histogram
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_bin_keys(int64_t n, const double *__restrict__ x, const double *__restrict__ y,
                                                  const double *__restrict__ z, const double *__restrict__ q, Grid g,
                                                  int32_t *__restrict__ key, int32_t *__restrict__ slot,
                                                  int32_t *__restrict__ count) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool active = i < n;
  int k = -1 - (int)(threadIdx.x & 63);  // lanes past the end: a key no other lane has
  if (active) {
    const int cx = cell_coord(wrap_coord(x[i], g.L[0]), g.inv_h[0], g.nx);
    const int cy = cell_coord(wrap_coord(y[i], g.L[1]), g.inv_h[1], g.ny);
    const int cz = cell_coord(wrap_coord(z[i], g.L[2]), g.inv_h[2], g.nz);
    k = (q[i] == 0.0 ? g.ncell : 0) + (cz * g.ny + cy) * g.nx + cx;
    key[i] = k;
  }
  const int sl = run_slot(k, active, count);  // every lane of the wave takes part in the vote
  if (active) slot[i] = sl;
}

// ---------------------------------------------------------------------------
// exclusive scan of int32 counts (three phases)
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;
// Tiles up to which each block adds the sums before its own itself (at most
// four loads a thread: under a microsecond, where a launch takes 4.6).
constexpr int64_t kScanTotals = 1024;

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ inline int block_exclusive_scan(int v, int *lds_waves, int *out_excl) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) lds_waves[wave] = incl;
  __syncthreads();
  int wave_off = 0, total = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) {
    const int s = lds_waves[w];
    if (w < wave) wave_off += s;
    total += s;
  }
  __syncthreads();
  *out_excl = wave_off + incl - v;
  return total;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_tiles(const int32_t *__restrict__ cnt, int64_t n,
                                                              int32_t *__restrict__ tile_sum) {
  __shared__ int lds[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) s += cnt[base + k];
  int excl;
  const int total = block_exclusive_scan(s, lds, &excl);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_top(int32_t *__restrict__ tile_sum, int64_t ntiles,
                                                            int32_t *__restrict__ grand_total) {
  __shared__ int lds[kScanThreads / 64];
  int carry = 0;
  for (int64_t b = 0; b < ntiles; b += kScanThreads) {
    const int64_t i = b + threadIdx.x;
    const int v = i < ntiles ? tile_sum[i] : 0;
    int excl;
    const int total = block_exclusive_scan(v, lds, &excl);
    if (i < ntiles) tile_sum[i] = carry + excl;
    carry += total;
  }
  if (threadIdx.x == 0) *grand_total = carry;
}

// TOTALS: tile_off holds the tiles' sums, not yet their offsets: each block adds
// those before its own (and the last one the total), a launch less.
template <bool TOTALS>
__global__ void __launch_bounds__(kScanThreads) k_scan_apply(const int32_t *__restrict__ cnt, int64_t n,
                                                              const int32_t *__restrict__ tile_off,
                                                              int32_t *__restrict__ start) {
  __shared__ int lds[kScanThreads / 64];
  int off = 0;
  if (TOTALS) {
    int before = 0, excl;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanThreads) before += tile_off[t];
    off = block_exclusive_scan(before, lds, &excl);
  } else {
    off = tile_off[blockIdx.x];
  }
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int v[kScanItems];
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? cnt[base + k] : 0;
    s += v[k];
  }
  int excl;
  const int total = block_exclusive_scan(s, lds, &excl);
  if (TOTALS && threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) start[n] = off + total;
  int run = off + excl;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) start[base + k] = run;
    run += v[k];
  }
}

int64_t scan_tiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

// start[0..n] = exclusive scan of cnt[0..n); start[n] = total. tmp needs scan_tiles(n) ints.
void launch_exclusive_scan(const int32_t *cnt, int64_t n, int32_t *start, int32_t *tmp, hipStream_t st) {
  const int64_t nt = scan_tiles(n);
  k_scan_tiles<<<(unsigned)nt, kScanThreads, 0, st>>>(cnt, n, tmp);
  if (nt <= kScanTotals) {
    k_scan_apply<true><<<(unsigned)nt, kScanThreads, 0, st>>>(cnt, n, tmp, start);
  } else {
    k_scan_top<<<1, kScanThreads, 0, st>>>(tmp, nt, start + n);
    k_scan_apply<false><<<(unsigned)nt, kScanThreads, 0, st>>>(cnt, n, tmp, start);
  }
}

// ---------------------------------------------------------------------------
// provisional scatter and stable placement
// ---------------------------------------------------------------------------
// count: cleared here for the keys pass of a following step (nullptr: none
// follows).
__global__ void __launch_bounds__(256) k_scatter_prov(int64_t n, const int32_t *__restrict__ key,
                                                      const int32_t *__restrict__ slot,
                                                      const int32_t *__restrict__ start, int32_t *__restrict__ tmp,
                                                      int32_t *__restrict__ count, int64_t nkeys) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (count)
    for (int64_t k = i; k < nkeys; k += (int64_t)gridDim.x * blockDim.x) count[k] = 0;
  if (i >= n) return;
  tmp[start[key[i]] + slot[i]] = (int32_t)i;
}

// Blocks [0, nb): one thread per bucket. Blocks from nb on (grids of few cells):
// one thread per particle of a bucket longer than kPlaceAlone, whose place is
// the count of the members with a smaller input index. A lone thread sorting
// hundreds of entries by insertion is bound by the latency of its moves, as many
// as the disorder that the atomics happened to leave: binning 12,000 particles in
// random order into 64 cells took 19.0 ms, now 50 us, 332,000 into 17,576 570 us,
// now 105.
constexpr int kPlaceAlone = 8;
// Particles a key from which on the second kind of block is launched: buckets
// are twice as long where one species fills the grid, longer where the density
// varies.
constexpr int kPlaceMean = 2;
__global__ void __launch_bounds__(256) k_place_buckets(int64_t nkeys, int64_t n, unsigned nb,
                                                       const int32_t *__restrict__ key,
                                                       const int32_t *__restrict__ start,
                                                       const int32_t *__restrict__ tmp, int32_t *__restrict__ perm) {
  if (blockIdx.x < nb) {
    const int64_t k = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (k >= nkeys) return;
    const int lo = start[k], hi = start[k + 1];
    if (gridDim.x == nb || hi - lo <= kPlaceAlone) place_bucket(lo, hi, tmp, perm);
    return;
  }
  const int64_t t = (blockIdx.x - nb) * (int64_t)256 + threadIdx.x;
  if (t >= n) return;
  const int32_t i = tmp[t];
  const int k = key[i], lo = start[k], hi = start[k + 1];
  if (hi - lo <= kPlaceAlone) return;
  int r = lo;
#pragma unroll 8
  for (int u = lo; u < hi; ++u) r += tmp[u] < i;
  perm[r] = i;
}

// ---------------------------------------------------------------------------
// small systems: one block
// ---------------------------------------------------------------------------
// The whole sort (POS: with its keys pass) in one block. What it replaces is
// six launches of 4.6 us each for a few thousand particles; it is bound by the
// latency of its own phases: a step's binning 28 -> 5.7 us at 2,000
// particles. The histogram and the starts stay in memory (the L2): in LDS they
// would limit the grid.
constexpr int kBlockBinThreads = 1024, kBlockBinEach = 8;  // 8,192 particles
// The block's accesses to the histogram, all of them atomics that the L2
// executes, are done before any that follow (a fence of the device's scope
// would write the L2 back: 3 us).
__device__ inline void histogram_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}
template <bool POS>
__global__ void __launch_bounds__(kBlockBinThreads) k_bin_block(int n, int nkeys, const double *__restrict__ x,
                                                                const double *__restrict__ y,
                                                                const double *__restrict__ z,
                                                                const double *__restrict__ q, Grid g,
                                                                const int32_t *__restrict__ key_in, int32_t *count,
                                                                int32_t *start, int32_t *__restrict__ perm) {
  constexpr int T = kBlockBinThreads, E = kBlockBinEach;
  __shared__ int32_t tmp[T * E];
  __shared__ int waves[T / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = tid; k < nkeys; k += T) __hip_atomic_store(&count[k], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int key[E], slot[E];
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const int i = u * T + tid;
    key[u] = -1 - lane;  // lanes past the end: a key no other lane has
    if (i < n) {
      if (POS) {
        const int cx = cell_coord(wrap_coord(x[i], g.L[0]), g.inv_h[0], g.nx);
        const int cy = cell_coord(wrap_coord(y[i], g.L[1]), g.inv_h[1], g.ny);
        const int cz = cell_coord(wrap_coord(z[i], g.L[2]), g.inv_h[2], g.nz);
        key[u] = (q[i] == 0.0 ? g.ncell : 0) + (cz * g.ny + cy) * g.nx + cx;
      } else {
        key[u] = key_in[i];
      }
    }
  }
  histogram_sync();  // it is clear
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (u * T < n) slot[u] = run_slot(key[u], u * T + tid < n, count);
  histogram_sync();  // and complete
  int carry = 0;
  for (int base = 0; base < nkeys; base += T * E) {
    const int k0 = base + tid * E;
    int v[E], s = 0;
#pragma unroll
    for (int u = 0; u < E; ++u) {
      v[u] = k0 + u < nkeys ? __hip_atomic_load(&count[k0 + u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
      s += v[u];
    }
    int incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) waves[wave] = incl;
    __syncthreads();
    int run = carry + incl - s;
    for (int w = 0; w < T / 64; ++w) {
      if (w < wave) run += waves[w];
      carry += waves[w];
    }
#pragma unroll
    for (int u = 0; u < E; ++u) {
      if (k0 + u < nkeys) start[k0 + u] = run;
      run += v[u];
    }
    __syncthreads();  // waves is read before the next round writes it
  }
  if (tid == 0) start[nkeys] = carry;
  __syncthreads();
  int lo[E], hi[E];
#pragma unroll
  for (int u = 0; u < E; ++u) {
    lo[u] = hi[u] = 0;
    if (u * T + tid < n) {
      lo[u] = start[key[u]];
      hi[u] = start[key[u] + 1];
    }
  }
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (u * T + tid < n) tmp[lo[u] + slot[u]] = u * T + tid;
  __syncthreads();
  // a particle's place: the members of its bucket with a smaller input index
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const int i = u * T + tid;
    if (i >= n) continue;
    int r = lo[u];
    for (int t = lo[u]; t < hi[u]; ++t) r += tmp[t] < i;
    perm[r] = i;
  }
}

// One block's time grows with the keys (its clearing and scan) and with the
// particles, of random order most (an atomic each, where cell order makes
// runs); the launches' hardly does, but each costs the caller its submission.
// Block against launches in us, kernels alone and (a whole call): a step's
// passes from given keys 500 particles and 8,192 keys 11.4, 12.6; and 14,400:
// 17.4, 13.0; 4,000 and 8,192: 14.3, 12.4; 8,000 and 3,456: 15.1, 15.6 (two
// steps 1,000 and 13,824: 81, 99; and 32,768: 112, 100; 8,000 and 4,096: 83,
// 95; and 13,824: 96, 94). All passes, particles in random order 2,000 and
// 8,192: 17.1, 19.0; 4,000 and 3,456: 18.5, 20.9; 8,000 and 8,192: 35.6, 22.1
// (a force call 2,000 and 13,824: 36, 40; and 32,768: 51, 40; 4,000 and 4,096:
// 39, 42; and 13,824: 45, 41; 6,000 and 4,096: 47, 46).
// A particle's place is a count over its bucket in both, of long buckets faster
// by the launches (8,000 and 128 keys: 184, 36; 2,000: 19, 23).
static bool bin_in_block(int64_t n, int64_t nkeys, bool keys_given) {
  return n <= kBlockBinThreads * kBlockBinEach && nkeys + (keys_given ? n : 3 * n) <= (keys_given ? 13000 : 21000) &&
         n * n <= 180000 * nkeys;
}

void launch_bin_clear(const BinBuffers &b, int64_t nkeys, int64_t n, hipStream_t st) {
  if (!bin_in_block(n, nkeys, true)) launch_fill_i32(b.count, nkeys, 0, st);
}

BinKeyOut bin_keys_out(const BinBuffers &b, int64_t nkeys, int64_t n, const double *q) {
  return BinKeyOut{q, b.key, b.slot, bin_in_block(n, nkeys, true) ? nullptr : b.count};
}

// Keys that a thread of the scatter clears at most: on a grid of many more
// cells than particles the launch is as wide as a fill of the histogram (300
// particles and 16 million keys, cleared by two blocks: a binning 916 us,
// without the clearing 145).
constexpr int64_t kClearEach = 16;

static void launch_bin_passes(const BinBuffers &b, int64_t nkeys, int64_t n, int32_t *cell_start, int32_t *perm,
                              bool more, hipStream_t st) {
  launch_exclusive_scan(b.count, nkeys, cell_start, b.scan_tmp, st);
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (more) blocks = std::max(blocks, std::min<int64_t>(8192, nkeys / (256 * kClearEach)));
  k_scatter_prov<<<(unsigned)blocks, 256, 0, st>>>(n, b.key, b.slot, cell_start, b.tmp, more ? b.count : nullptr,
                                                   nkeys);
  const unsigned nb = (unsigned)((nkeys + 255) / 256);
  const unsigned pb = n > kPlaceMean * nkeys ? (unsigned)((n + 255) / 256) : 0u;
  k_place_buckets<<<nb + pb, 256, 0, st>>>(nkeys, n, nb, b.key, cell_start, b.tmp, perm);
}

void launch_bin_place(const BinBuffers &b, int64_t nkeys, int64_t n, int32_t *cell_start, int32_t *perm, bool more,
                      hipStream_t st) {
  if (bin_in_block(n, nkeys, true))
    k_bin_block<false><<<1, kBlockBinThreads, 0, st>>>((int)n, (int)nkeys, nullptr, nullptr, nullptr, nullptr, Grid{},
                                                       b.key, b.count, cell_start, perm);
  else
    launch_bin_passes(b, nkeys, n, cell_start, perm, more, st);
}

void launch_bin(const BinBuffers &b, const Grid &g, int64_t n, const double *x, const double *y, const double *z,
                const double *q, int32_t *cell_start, int32_t *perm, hipStream_t st) {
  const int64_t nkeys = 2 * (int64_t)g.ncell;
  if (bin_in_block(n, nkeys, false)) {
    k_bin_block<true><<<1, kBlockBinThreads, 0, st>>>((int)n, (int)nkeys, x, y, z, q, g, nullptr, b.count, cell_start,
                                                      perm);
    return;
  }
  launch_fill_i32(b.count, nkeys, 0, st);
  if (n > 0) {
    const unsigned blocks = (unsigned)((n + 255) / 256);
    k_bin_keys<<<blocks, 256, 0, st>>>(n, x, y, z, q, g, b.key, b.slot, b.count);
  }
  launch_bin_passes(b, nkeys, n, cell_start, perm, false, st);
}

}  // namespace rbe
