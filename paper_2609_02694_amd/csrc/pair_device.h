// Device building blocks of the near-field kernels (internal): pair
// scalars of Eq. 8 in FP64 and FP32, compensated accumulation, and the
// stencil traversals of the cell list.
#pragma once
#include "kernels.h"

namespace rbe {

// Coefficients of the FP64 polynomials below, highest degree first.
#define RBE_ERFCX_COEFS \
    1.63618628481317543e-08, -4.60928758649811430e-08, -6.88442333452307132e-08, \
    4.40190654889049080e-07, -4.46917185831068957e-07, -1.14063358111397811e-06, \
    3.75537844601685302e-06, -1.41703053499259700e-06, -1.39602653735770222e-05, \
    2.75867068654632672e-05, 2.75241444094816018e-05, -1.74362281120596591e-04, \
    4.35557661104548185e-05, 9.81977137355043118e-04, -8.47143262890503600e-04, \
    -6.99746174546772310e-03, 3.73289240473987467e-03, 7.89785810158994406e-02, \
    2.41658194242463487e-01, 4.27185847413955655e-01, 2.55395676310504194e-01
#define RBE_EXP_COEFS \
    1.1470745597729725e-11, 1.6059043836821613e-10, 2.08767569878681e-09, 2.505210838544172e-08, \
    2.755731922398589e-07, 2.7557319223985893e-06, 2.48015873015873e-05, 0.0001984126984126984, \
    0.001388888888888889, 0.008333333333333333, 0.041666666666666664, 0.16666666666666666, 0.5, 1.0, \
    1.0
constexpr double kErfcxCoef[] = {RBE_ERFCX_COEFS};
constexpr double kExpCoef[] = {RBE_EXP_COEFS};
constexpr int kErfcxTerms = (int)(sizeof(kErfcxCoef) / sizeof(double));
constexpr int kExpTerms = (int)(sizeof(kExpCoef) / sizeof(double));
// The same coefficients in constant memory, for kernels that evaluate the
// pair scalar in a branch most trips of a neighbour walk skip: read there
// with scalar loads at an opaque offset, so the compiler cannot keep the
// whole table in vector registers for the walk (it did, costing a wave of
// occupancy).
static __constant__ double kErfcxTable[kErfcxTerms] = {RBE_ERFCX_COEFS};
static __constant__ double kExpTable[kExpTerms] = {RBE_EXP_COEFS};
__device__ inline int opaque_zero() {
  int z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return z;
}
// d = a b + c as one v_fma_f64 with c in vector (fma_vv) or scalar (fma_vs)
// registers; plain fma() here becomes v_fmac with the addend copied into the
// destination first, two or three instructions per polynomial step.
__device__ inline double fma_vv(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ inline double fma_vs(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}
// Horner evaluation of a coefficient list at x (TABLE: from constant memory).
template <bool TABLE, int N>
__device__ inline double horner_f64(const double (&coef)[N], const double *table, double x) {
  if constexpr (TABLE) {
    const double *t = table + opaque_zero();
    double c[N];
#pragma unroll
    for (int k = 0; k < N; ++k) c[k] = t[k];  // issued together, merged into wide scalar loads
    double r = c[0];
#pragma unroll
    for (int k = 1; k < N; ++k) r = fma_vs(r, x, c[k]);
    return r;
  } else {
    double r = coef[0];
#pragma unroll
    for (int k = 1; k < N; ++k) r = fma_vv(r, x, coef[k]);
    return r;
  }
}

// FP64 erfc(x) = exp(-x^2) R(x) with R(x) = erfc(x) e^{x^2} a degree-20
// polynomial in s = 2/(1 + x/2) - 1 (fit over x in [0, 8] by fit_erfcx.py,
// relative error below 7.2e-15); e = exp(-x^2) is passed in.
__device__ inline double rcp_f64(double a);
template <bool TABLE>
__device__ inline double erfc_scaled_f64(double x) {
  const double s = fma(2.0, rcp_f64(fma(0.5, x, 1.0)), -1.0);
  return horner_f64<TABLE>(kErfcxCoef, kErfcxTable, s);
}

// FP64 building blocks of the pair scalar: hardware reciprocal and
// reciprocal-square-root estimates refined by two Newton steps each (the
// error of the estimate squares at every step: a few ulp after two), and
// exp(x) for x <= 0 by x = k ln2 + t, |t| <= ln2/2 (ln2 split into a head
// with 21 trailing zero bits, so k * head is exact, and a tail), the Taylor
// series of e^t to degree 14 (remainder below 1e-17) and a scaling by 2^k.
__device__ inline double rcp_f64(double a) {
  double y = __builtin_amdgcn_rcp(a);
  double e = fma(-a, y, 1.0);
  y = fma(y, e, y);
  e = fma(-a, y, 1.0);
  return fma(y, e, y);
}
__device__ inline double rsqrt_f64(double a) {
  double y = __builtin_amdgcn_rsq(a);
  // y <- y + y (1 - a y^2) / 2
  double e = fma(-a * y, y, 1.0);
  y = fma(0.5 * y, e, y);
  e = fma(-a * y, y, 1.0);
  return fma(0.5 * y, e, y);
}
template <bool TABLE>
__device__ inline double exp_nonpos_f64(double x) {
  const double k = rint(x * 1.4426950408889634);
  double t = fma(-k, 0.6931471803691238, x);
  t = fma(-k, 1.9082149292705877e-10, t);
  return ldexp(horner_f64<TABLE>(kExpCoef, kExpTable, t), (int)k);
}

template <bool TABLE = false>
__device__ inline double pair_scalar_f64(const PairParams &pp, double r2, double qi, double qj) {
  const double rinv = rsqrt_f64(r2);
  const double inv_r2 = rinv * rinv;
  double f = 0.0;
  if (pp.do_coul && r2 <= pp.rc2 && qi != 0.0 && qj != 0.0) {
    const double r = r2 * rinv;
    const double e = exp_nonpos_f64<TABLE>(-pp.alpha * r2);
    const double R = erfc_scaled_f64<TABLE>(pp.sqrt_alpha * r);
    // G = erfc(x)/r^3 + 2 sqrt(a) e/(sqrt(pi) r^2) = e/r^2 (R/r + 2 sqrt(a)/sqrt(pi))
    const double G = e * inv_r2 * fma(R, rinv, pp.two_sqrt_alpha_over_sqrt_pi);
    f = pp.kc * qi * qj * G;
  }
  if (pp.do_lj && r2 <= pp.rlj2) {
    const double s2 = pp.sig2 * inv_r2;
    const double s6 = s2 * s2 * s2;
    f = fma(pp.eps24 * (2.0 * s6 * s6 - s6), inv_r2, f);
  }
  return f;
}

// FP32 form of the pair scalar: erfc(x) = exp(-x^2) R(x), R(x) = erfc(x) e^{x^2}
// as a degree-9 polynomial in t = 1/(1 + x/2) (fit over x in [0, 8] by
// fit_erfcx.py; relative error of the FP32 evaluation below 3.3e-7). The
// exponential exp(-alpha r^2) is shared with the second term of G.

__device__ inline float erfcx_poly(float t) {
  float r = -5.023304369e-02f;
  r = fmaf(r, t, 2.383836403e-01f);
  r = fmaf(r, t, -3.831243495e-01f);
  r = fmaf(r, t, 1.457629880e-01f);
  r = fmaf(r, t, 7.766769416e-02f);
  r = fmaf(r, t, 1.499599762e-01f);
  r = fmaf(r, t, 2.601579210e-01f);
  r = fmaf(r, t, 2.789792283e-01f);
  r = fmaf(r, t, 2.824637353e-01f);
  r = fmaf(r, t, -1.781403551e-05f);
  return r;
}

__device__ inline float pair_scalar_f32(const PairParams &pp, const PairF32 &pf, double r2d, float qiqj) {
  const float r2 = (float)r2d;
  const float rinv = __builtin_amdgcn_rsqf(r2);
  const float rinv2 = rinv * rinv;
  float f = 0.f;
  if (pp.do_coul && r2d <= pp.rc2 && qiqj != 0.f) {
    const float r = r2 * rinv;
    const float x = pf.sqrt_alpha * r;
    const float e = __builtin_amdgcn_exp2f(pf.neg_alpha_log2e * r2);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
    const float erfc_x = e * erfcx_poly(t);
    const float G = fmaf(erfc_x * rinv, rinv2, pf.two_sqrt_alpha_over_sqrt_pi * e * rinv2);
    f = pf.kc * qiqj * G;
  }
  if (pp.do_lj && r2d <= pp.rlj2) {
    const float s2 = pf.sig2 * rinv2;
    const float s6 = s2 * s2 * s2;
    f = fmaf(pf.eps24 * fmaf(2.0f, s6 * s6, -s6), rinv2, f);
  }
  return f;
}

__device__ inline double pair_scalar_lj_f64(const PairParams &pp, double r2) {
  if (!(pp.do_lj && r2 <= pp.rlj2)) return 0.0;
  const double inv_r2 = rcp_f64(r2);
  const double s2 = pp.sig2 * inv_r2;
  const double s6 = s2 * s2 * s2;
  return pp.eps24 * (2.0 * s6 * s6 - s6) * inv_r2;
}

__device__ inline float pair_scalar_lj_f32(const PairParams &pp, const PairF32 &pf, double r2d) {
  if (!(pp.do_lj && r2d <= pp.rlj2)) return 0.f;
  const float rinv2 = __builtin_amdgcn_rcpf((float)r2d);
  const float s2 = pf.sig2 * rinv2;
  const float s6 = s2 * s2 * s2;
  return pf.eps24 * fmaf(2.0f, s6 * s6, -s6) * rinv2;
}

// Kahan-compensated FP32 accumulation of a 3-vector.
struct Kahan3 {
  float s[3] = {0.f, 0.f, 0.f}, c[3] = {0.f, 0.f, 0.f};
  __device__ inline void add(int k, float v) {
#pragma clang fp contract(off)
    const float y = v - c[k];
    const float t = s[k] + y;
    c[k] = (t - s[k]) - y;
    s[k] = t;
  }
  // s += a b with the product fused into the compensation step
  __device__ inline void add_prod(int k, float a, float b) {
#pragma clang fp contract(off)
    const float y = fmaf(a, b, -c[k]);
    const float t = s[k] + y;
    c[k] = (t - s[k]) - y;
    s[k] = t;
  }
  __device__ inline double get(int k) const { return (double)s[k] - (double)c[k]; }
};

__device__ inline double sq_dist(double dx, double dy, double dz) {
#pragma clang fp contract(off)
  return dx * dx + dy * dy + dz * dz;
}

__device__ inline double min_image(double a, double L) {
#pragma clang fp contract(off)
  return a - L * rint(a / L);
}

// Calls fn(jofs + j, p_j, shx, shy, shz) for the records j0..j1-1 of xq;
// jofs separates the index ranges of natives (0) and ghosts (n). Four fixed
// slots: slot k holds record j + k and is reloaded with j + k + 4 right after
// use, so each load has three candidates of work to complete behind it. The
// lookahead reads up to kScanPad - 1 records past j1: every array scanned
// here is allocated with kScanPad records of padding, so those loads stay
// inside the allocation (their values are never used), and the addresses are
// plain increments.
template <class Fn>
__device__ inline void scan_range(const double4 *__restrict__ xq, int j0, int j1, double shx, double shy, double shz,
                                  Fn &&fn, int jofs = 0) {
  if (j0 >= j1) return;
  const double4 *p = xq + j0;
  double4 r0 = p[0], r1 = p[1], r2 = p[2], r3 = p[3];
  j0 += jofs;
  j1 += jofs;
#pragma unroll 1
  for (int j = j0; j < j1; j += 4) {
    fn(j, r0, shx, shy, shz);
    r0 = p[4];
    if (j + 1 < j1) fn(j + 1, r1, shx, shy, shz);
    r1 = p[5];
    if (j + 2 < j1) fn(j + 2, r2, shx, shy, shz);
    r2 = p[6];
    if (j + 3 < j1) fn(j + 3, r3, shx, shy, shz);
    r3 = p[7];
    p += 4;
  }
}

// Rows of a walk: each stencil row is trimmed to the x-cells the reach sphere
// can touch. The gap g from (y, z) to the row's y/z cell slabs bounds the x
// extent by sqrt(r^2 - g^2), and rows with g > r are skipped. All of it in
// FP32, in the frame of the particle's own cell (coordinates of the size of
// the reach, whatever the box): the squared reach is enlarged by 2^-18 and
// the gaps and the extent by 2^-18 of the reach and the largest cell edge,
// tens of times the rounding of these few operations and of the binning, so
// no cell inside the reach is left out; every pair is classified exactly
// afterwards. (In FP64, with its square root, the set-up of a row cost as
// many issue cycles as several candidates.)
struct RowFrame {
  float ux, uy, uz;        // offset of the particle in its cell
  float hy, hz, inv_hx;
  float r2, margin;
  __device__ inline RowFrame(const Grid &g, double x, double y, double z, int cx, int cy, int cz, double reach2) {
    ux = (float)(x - (double)cx * g.h[0]);
    uy = (float)(y - (double)cy * g.h[1]);
    uz = (float)(z - (double)cz * g.h[2]);
    hy = (float)g.h[1];
    hz = (float)g.h[2];
    inv_hx = (float)g.inv_h[0];
    r2 = (float)reach2 * (1.0f + 0x1p-18f);
    margin = 0x1p-18f * (__builtin_amdgcn_sqrtf(r2) + fmaxf((float)g.h[0], fmaxf(hy, hz)));
  }
  // Distance from an offset u to the slab of the cell o cells away, less the margin, at least 0.
  __device__ inline float gap(float u, int o, float h) const {
    const float lo = (float)o * h;
    return fmaxf(fmaxf(lo - u, u - (lo + h)) - margin, 0.0f);
  }
  // x-cell offsets [*a, *b] (within [-s, s]) of a row at gaps whose squares sum to g2; false if out of reach.
  __device__ inline bool range(float g2, int s, int *a, int *b) const {
    const float rem = r2 - g2;
    if (rem < 0.0f) return false;
    const float ext = __builtin_amdgcn_sqrtf(rem) + margin;
    *a = max(-s, (int)floorf((ux - ext) * inv_hx));
    *b = min(s, (int)floorf((ux + ext) * inv_hx));
    return *a <= *b;
  }
  // Whether the enlarged reach may be what a row at g2 owes its place to (the
  // enlargements above, summed, are under half of this band).
  __device__ inline bool doubtful(float g2) const { return r2 - g2 < 8.0f * margin * __builtin_amdgcn_sqrtf(r2); }
};

// Distance from p to the slab of unwrapped cell c, less 1e-9 (the rounding of
// the binning), at least 0.
__device__ inline double slab_gap(double p, int c, double h) {
#pragma clang fp contract(off)
  const double lo = (double)c * h, hi = lo + h;
  const double d = lo - p > 0.0 ? lo - p : (p - hi > 0.0 ? p - hi : 0.0);
  return d > 1e-9 ? d - 1e-9 : 0.0;
}
// The rows a walk closes are part of an FP32C result (closing an empty row can
// move a Kahan sum's rounding), so a doubtful row is decided in FP64: whether
// unwrapped row (cy, cz) is out of the squared reach of (y, z).
__device__ inline bool row_beyond(const Grid &g, double y, double z, int cy, int cz, double reach2) {
#pragma clang fp contract(off)
  const double gy = slab_gap(y, cy, g.h[1]), gz = slab_gap(z, cz, g.h[2]);
  return reach2 - (gy * gy + gz * gz) < 0.0;
}

// Cell in [0, n) of an unwrapped cell index a in [-n, 2 n), and the boxes it
// lies off. (A cutoff is at most half the box, so a stencil radius is at most
// n and the neighbours of a cell of the grid lie in that range.)
__device__ inline int wrap_cell(int a, int n, int *q) {
  *q = a < 0 ? -1 : (a >= n ? 1 : 0);
  return a - *q * n;
}

// Periodic traversal: every particle j of species block `blk` (keys cell_base
// + blk C + cell) in the (2 s.x + 1)(2 s.y + 1)(2 s.z + 1) cells around
// (cx, cy, cz), the cell of (x, y, z), that the squared reach r2 can touch,
// each met once per periodic image; (shx, shy, shz) is the image shift of j
// (its image lies at r_j + shift).
// row_end() is called after each stencil row (the FP32C accumulators close a
// row's plain partial sum there).
struct NoRowEnd {
  __device__ inline void operator()() const {}
};
template <class Fn, class RowEnd = NoRowEnd>
__device__ inline void for_stencil(const Grid &g, const int32_t *__restrict__ cell_start,
                                   const double4 *__restrict__ xq, int blk, int cx, int cy, int cz, const Sten &s,
                                   double x, double y, double z, double r2, Fn &&fn, int64_t cell_base = 0,
                                   RowEnd row_end = RowEnd()) {
  const int32_t *cs = cell_start + cell_base + (int64_t)blk * g.ncell;
  const RowFrame F(g, x, y, z, cx, cy, cz, r2);
  for (int oz = -s.z; oz <= s.z; ++oz) {
    const float gz = F.gap(F.uz, oz, F.hz);
    if (gz * gz > F.r2) continue;
    int qz;
    const int wz = wrap_cell(cz + oz, g.nz, &qz);
    const double shz = (double)qz * g.L[2];
    for (int oy = -s.y; oy <= s.y; ++oy) {
      const float gy = F.gap(F.uy, oy, F.hy);
      int a, a_end;
      const float g2 = fmaf(gy, gy, gz * gz);
      if (!F.range(g2, s.x, &a, &a_end)) continue;
      if (F.doubtful(g2) && row_beyond(g, y, z, cy + oy, cz + oz, r2)) continue;
      a += cx;
      a_end += cx;
      int qy;
      const int wy = wrap_cell(cy + oy, g.ny, &qy);
      const double shy = (double)qy * g.L[1];
      const int32_t *row = cs + (wz * g.ny + wy) * g.nx;
      do {
        int qx;
        const int wa = wrap_cell(a, g.nx, &qx);
        const int b = min(a_end, (qx + 1) * g.nx - 1);
        scan_range(xq, row[wa], row[b - qx * g.nx + 1], (double)qx * g.L[0], shy, shz, fn);
        a = b + 1;
      } while (a <= a_end);
      row_end();
    }
  }
}

// Ghost-shell traversal (no periodic images): the natives of the stencil
// rows that lie inside the native grid, then the ghosts of the same rows of
// the padded grid, each row trimmed to the reach. (cx, cy, cz) is a native
// cell. Ghosts reach fn with indices offset by nnat.
template <class Fn, class RowEnd>
__device__ inline void for_stencil_ghost(const Grid &g, const int32_t *__restrict__ cell_start,
                                         const double4 *__restrict__ xq,
                                         const int32_t *__restrict__ gcell_start, const double4 *__restrict__ gxq,
                                         int nnat, int blk, int cx, int cy, int cz, const Sten &s, double px,
                                         double py, double pz, double r2, Fn &&fn, RowEnd row_end) {
  const int32_t *cs = cell_start + (int64_t)blk * g.ncell;
  const int32_t *gs = gcell_start + (int64_t)blk * g.pncell;
  const RowFrame F(g, px, py, pz, cx, cy, cz, r2);
  for (int oz = -s.z; oz <= s.z; ++oz) {
    const float gz = F.gap(F.uz, oz, F.hz);
    if (gz * gz > F.r2) continue;
    const int z = cz + oz;
    for (int oy = -s.y; oy <= s.y; ++oy) {
      const float gy = F.gap(F.uy, oy, F.hy);
      int xa, xb;
      const float g2 = fmaf(gy, gy, gz * gz);
      if (!F.range(g2, s.x, &xa, &xb)) continue;
      if (F.doubtful(g2) && row_beyond(g, py, pz, cy + oy, cz + oz, r2)) continue;
      xa += cx;
      xb += cx;
      const int y = cy + oy;
      const bool inner = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
      if (inner) {
        const int na = max(xa, 0), nb = min(xb, g.nx - 1);
        if (na <= nb) {
          const int32_t *row = cs + (z * g.ny + y) * g.nx;
          scan_range(xq, row[na], row[nb + 1], 0.0, 0.0, 0.0, fn);
        }
      }
      // the padded cells over the native grid hold no ghosts: a row range
      // inside it has none to scan
      if (!inner || xa < 0 || xb >= g.nx) {
        const int32_t *prow = gs + ((z + g.goff[2]) * g.pny + (y + g.goff[1])) * g.pnx + g.goff[0];
        scan_range(gxq, prow[xa], prow[xb + 1], 0.0, 0.0, 0.0, fn, nnat);
      }
      row_end();
    }
  }
}

// ---------------------------------------------------------------------------
// Group walks: G consecutive lanes per particle
// ---------------------------------------------------------------------------
// Sum over the G lanes of a group (fixed order; the lanes of a group together).
template <int G>
__device__ inline double group_sum(double v) {
#pragma unroll
  for (int o = 1; o < G; o <<= 1) v += __shfl_xor(v, o, G);
  return v;
}
// The lanes of this lane's group for which v holds, as bits 0..G-1.
template <int G>
__device__ inline uint64_t group_ballot(bool v) {
  const uint64_t b = __builtin_amdgcn_ballot_w64(v);
  if (G == 64) return b;
  return (b >> (threadIdx.x & 63 & ~(G - 1))) & ((1ull << (G & 63)) - 1ull);
}

// Bits of `who` (a group ballot) below this lane's place in its group.
template <int G>
__device__ inline int bits_below(uint64_t who) {
  if (G == 64) return __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0));
  return __popc((uint32_t)who & ((1u << (threadIdx.x & (G - 1))) - 1u));
}

// Particles of one species block to meet: its stencil and squared reach.
struct Block {
  Sten s;
  double r2;
  __device__ inline int rows() const { return s.y < 0 ? 0 : (2 * s.y + 1) * (2 * s.z + 1); }
};
__device__ inline Block no_block() { return Block{Sten{0, -1, 0}, 0.0}; }

// Candidates listed at a time, and the group's table of listed rows in LDS:
// the first record of a row less its place in the list, its image shifts and
// species block, and one bit per place, set if a row starts at the place after.
template <int G>
constexpr int kGroupList = 8 * G;
template <int G>
struct GroupRows {
  int base[G], code[G];
  alignas(8) uint32_t starts[kGroupList<G> / 32];
};

// The signed 10-bit field of v that starts at bit `at`.
__device__ inline int bits10(int v, int at) { return (int)((uint32_t)v << (22 - at)) >> 22; }
// Orders the LDS accesses of a wave's lanes before and after it (a wave's LDS
// operations execute in order; this holds the compiler to it).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A group's walk of its particle's stencil rows (block A's, then block B's,
// each z-major), G rows at a time, one to a lane. The rows' candidates are
// put end to end by a prefix sum of their counts, and the lanes then take G
// consecutive ones each trip, whatever rows they come from: a lane finds its
// row by counting the start bits up to its own place. So all lanes stay busy
// however short or uneven the rows are, and the walk's length is that of the
// particle's whole neighbourhood divided by G, not of its longest row.
// The whole group calls fetch(j, ghost) for record j of the natives or of the
// ghosts (ghost: the same for all), for AHEAD (1 or 2) trips at a time so that
// their loads are in flight together, then visit(ok, k, j, code, ghost,
// shifted, fetched) for each: the row's code has its species block in bit 0, then its image
// shifts (row_shift; shifted: some row of the piece has one); k is the place in
// the listed chunk of kGroupList<G> (ok false: nothing there, and j the last
// record listed).
// listed(first, len) follows each chunk: this lane's row holds the places
// [first, first + len) of it (len may be 0). rows_end(reached) follows each
// round of G rows: the lanes whose rows the particle's reach touches.
// GHOST: no periodic images, but the ghost arrays.
template <int G, bool GHOST, int AHEAD, class Fetch, class Visit, class Listed, class RowsEnd>
__device__ inline void group_list(const Grid &g, const int32_t *__restrict__ cell_start,
                                  const int32_t *__restrict__ gcell_start, const double4 &pi, const Block &A,
                                  const Block &B, GroupRows<G> &T, Fetch &&fetch, Visit &&visit,
                                  Listed &&listed, RowsEnd &&rows_end) {
  constexpr int CH = kGroupList<G>;
  const int sub = threadIdx.x & (G - 1);
  const int cx = cell_coord(pi.x, g.inv_h[0], g.nx), cy = cell_coord(pi.y, g.inv_h[1], g.ny),
            cz = cell_coord(pi.z, g.inv_h[2], g.nz);
  const int ra = A.rows(), rows = ra + B.rows();
  for (int r0 = 0; r0 < rows; r0 += G) {
    // this lane's row: its unwrapped x-cells [a, a_end], none if out of reach
    int row = r0 + sub, a = 1, a_end = 0, y = 0, z = 0, blk = 0;
    if (row < rows) {
      blk = row >= ra;
      const Sten s = blk ? B.s : A.s;
      if (blk) row -= ra;
      const RowFrame F(g, pi.x, pi.y, pi.z, cx, cy, cz, blk ? B.r2 : A.r2);
      const int ny = 2 * s.y + 1;
      int oz = (int)(((float)row + 0.5f) / (float)ny);  // row / ny: the quotient is at least 0.5/ny off an integer
      const int oy = row - oz * ny - s.y;
      oz -= s.z;
      const float gz = F.gap(F.uz, oz, F.hz), gy = F.gap(F.uy, oy, F.hy);
      const float g2 = fmaf(gy, gy, gz * gz);
      if (F.range(g2, s.x, &a, &a_end) &&
          !(F.doubtful(g2) && row_beyond(g, pi.y, pi.z, cy + oy, cz + oz, blk ? B.r2 : A.r2))) {
        a += cx;
        a_end += cx;
      } else {
        a = 1;
        a_end = 0;
      }
      y = cy + oy;
      z = cz + oz;
    }
    // a row's records lie in one piece, or in several: the pieces of a row that
    // crosses the box edge, the natives and the ghosts of one at the edge
    bool more = a <= a_end;
    const uint64_t reached = group_ballot<G>(more);
    for (int pass = 0; group_ballot<G>(more); ++pass) {
      int j0 = 0, len = 0, code = 0;
      if (more) {
        if (GHOST) {
          if (pass == 0) {
            const bool inner = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
            const int na = max(a, 0), nb = min(a_end, g.nx - 1);
            if (inner && na <= nb) {
              const int32_t *t = cell_start + (int64_t)blk * g.ncell + (z * g.ny + y) * g.nx;
              j0 = t[na];
              len = t[nb + 1] - j0;
            }
            // the padded cells over the native grid hold no ghosts
            more = !inner || a < 0 || a_end >= g.nx;
          } else {
            const int32_t *t = gcell_start + (int64_t)blk * g.pncell +
                               ((z + g.goff[2]) * g.pny + (y + g.goff[1])) * g.pnx + g.goff[0];
            j0 = t[a];
            len = t[a_end + 1] - j0;
            more = false;
          }
        } else {
          int qx, qy, qz;
          const int wz = wrap_cell(z, g.nz, &qz), wy = wrap_cell(y, g.ny, &qy);
          const int32_t *t = cell_start + (int64_t)blk * g.ncell + (wz * g.ny + wy) * g.nx;
          const int wa = wrap_cell(a, g.nx, &qx);
          const int b = min(a_end, (qx + 1) * g.nx - 1);
          j0 = t[wa];
          len = t[b - qx * g.nx + 1] - j0;
          a = b + 1;
          more = a <= a_end;
          code = ((qx & 1023) << 20) | ((qy & 1023) << 10) | (qz & 1023);
        }
      }
      int end = len;  // inclusive prefix sum over the group
#pragma unroll
      for (int o = 1; o < G; o <<= 1) {
        const int t = __shfl_up(end, o, G);
        if (sub >= o) end += t;
      }
      const int start = end - len, total = __shfl(end, G - 1, G);
      if (total == 0) {
        listed(0, 0);
        continue;
      }
      const uint64_t some = group_ballot<G>(len > 0);
      const bool shifted = !GHOST && group_ballot<G>(code != 0) != 0;
      if (len > 0) {
        const int rank = bits_below<G>(some);
        T.base[rank] = j0 - start;
        T.code[rank] = code << 1 | blk;
      }
      for (int c0 = 0; c0 < total; c0 += CH) {
        if (sub < CH / 32) T.starts[sub] = 0;
        wave_sync();
        if (len > 0 && start > c0 && start <= c0 + CH)
          atomicOr(&T.starts[(start - 1 - c0) >> 5], 1u << ((start - 1 - c0) & 31));
        wave_sync();
        // the row of the chunk's first place; a trip's row adds the starts before its place
        int row0 = __popcll(group_ballot<G>(len > 0 && start <= c0)) - 1;
        const int cnt = min(CH, total - c0);
        struct Place {
          int k, j, code;
          bool ok;
        };
        auto place = [&](int k0) {
          uint64_t bits;
          if (G == 64) bits = *(const uint64_t *)&T.starts[k0 >> 5];
          else bits = (T.starts[k0 >> 5] >> (k0 & 31)) & (uint32_t)((1ull << (G & 63)) - 1ull);
          Place q;
          q.k = k0 + sub;
          q.ok = q.k < cnt;
          const int r = row0 + bits_below<G>(bits);
          row0 += __popcll(bits);
          q.j = T.base[r] + c0 + min(q.k, cnt - 1);
          q.code = T.code[r];
          return q;
        };
        for (int k0 = 0; k0 < cnt; k0 += AHEAD * G) {
          const bool ghost = GHOST && pass;
          const Place a0 = place(k0);
          const auto f0 = fetch(a0.j, ghost);
          if (AHEAD == 2 && k0 + G < cnt) {
            const Place a1 = place(k0 + G);
            const auto f1 = fetch(a1.j, ghost);
            visit(a0.ok, a0.k, a0.j, a0.code, ghost, shifted, f0);
            visit(a1.ok, a1.k, a1.j, a1.code, ghost, shifted, f1);
          } else {
            visit(a0.ok, a0.k, a0.j, a0.code, ghost, shifted, f0);
          }
        }
        wave_sync();
        const int first = max(start - c0, 0);
        listed(first, max(0, min(end - c0, cnt) - first));
        wave_sync();
      }
    }
    rows_end(reached);
  }
}

// Image shift (boxes) of a listed row's code along an axis.
__device__ inline double row_shift(int code, int axis) { return (double)bits10(code, 21 - 10 * axis); }

// The walk on FP64 records: visit(ok, k, blk, j, p_j, dx, dy, dz, r^2), ghosts
// indexed from nnat on.
template <int G, bool GHOST, class Visit, class Listed, class RowsEnd>
__device__ inline void group_walk(const Grid &g, const int32_t *__restrict__ cell_start,
                                  const double4 *__restrict__ xq, const int32_t *__restrict__ gcell_start,
                                  const double4 *__restrict__ gxq, int nnat, const double4 &pi, const Block &A,
                                  const Block &B, GroupRows<G> &T, Visit &&visit, Listed &&listed,
                                  RowsEnd &&rows_end) {
  group_list<G, GHOST, 1>(
      g, cell_start, gcell_start, pi, A, B, T, [&](int j, bool ghost) { return ghost ? gxq[j] : xq[j]; },
      [&](bool ok, int k, int j, int code, bool ghost, bool shifted, const double4 &p) {
        double dx = pi.x - p.x, dy = pi.y - p.y, dz = pi.z - p.z;
        if (shifted) {
          dx -= row_shift(code, 0) * g.L[0];
          dy -= row_shift(code, 1) * g.L[1];
          dz -= row_shift(code, 2) * g.L[2];
        }
        visit(ok, k, code & 1, ghost ? nnat + j : j, p, dx, dy, dz, sq_dist(dx, dy, dz));
      },
      listed, rows_end);
}

// Pairs of a group walk that passed their test, kept in LDS until a lane of
// the group has one each: about half of the lanes hold a pair in a trip, which
// tells where a term costs many times its test (the energies' library error
// function; the forces' terms gain less than the registers cost). The whole
// group calls put_hits for every trip (in: this lane has the pair v) and
// take_hits at the end; eval(v) then runs for G pairs at a time, together with
// the other group of the wave, whose pairs are taken as they are.
template <int G, class Pair>
struct GroupHits {
  Pair list[2 * G];  // `pending` of them, fewer than G between trips
};
template <int G, class Pair, class Eval>
__device__ inline void take_hits(GroupHits<G, Pair> &H, int &pending, Eval &&eval) {
  const int sub = threadIdx.x & (G - 1), k = min(pending, G);
  wave_sync();
  if (sub < k) eval(H.list[pending - k + sub]);
  pending -= k;
  wave_sync();
}
template <int G, class Pair, class Eval>
__device__ inline void put_hits(GroupHits<G, Pair> &H, int &pending, bool in, const Pair &v, Eval &&eval) {
  const uint64_t who = group_ballot<G>(in);
  if (in) H.list[pending + bits_below<G>(who)] = v;
  pending += __popcll(who);
  if (__builtin_amdgcn_ballot_w64(pending >= G)) take_hits<G>(H, pending, eval);
}

// Ordered sums of the FP32C form in a group walk: the terms of a chunk are
// left in LDS by the lanes that evaluated them, each row's are then added in
// order by the lane of that row, and the rows' sums by every lane (flush_rows):
// the same bits as one thread walking the rows one after another.
template <int G>
struct GroupTerms {
  float4 t[kGroupList<G>];  // pair scalar and displacement
};

// Accumulator of the per-particle force in the two precision forms.
// add<true> evaluates Coulomb + LJ, add<false> LJ only (j neutral); TABLE
// selects the constant-memory polynomial coefficients (FP64 form).
template <bool F32>
struct ForceAcc;
template <>
struct ForceAcc<false> {
  double v[3] = {0.0, 0.0, 0.0};
  template <bool COUL, bool TABLE = false>
  __device__ inline void add(const PairParams &pp, const PairF32 &, double r2, double qi, double qj, double dx,
                             double dy, double dz) {
    const double sc = COUL ? pair_scalar_f64<TABLE>(pp, r2, qi, qj) : pair_scalar_lj_f64(pp, r2);
    v[0] = fma(sc, dx, v[0]);
    v[1] = fma(sc, dy, v[1]);
    v[2] = fma(sc, dz, v[2]);
  }
  __device__ inline double get(int k) const { return v[k]; }
  // the sum over the lanes of a group
  template <int G>
  __device__ inline double total(int k) const {
    return group_sum<G>(v[k]);
  }
};
template <>
struct ForceAcc<true> {
  Kahan3 k;
  float p[3] = {0.f, 0.f, 0.f};  // the current row's plain partial sums (add_row)
  // the thread-form walks: a row's terms summed plainly in FP32, the row sum
  // added with Kahan compensation at flush_row
  template <bool COUL, bool TABLE = false>
  __device__ inline void add_row(const PairParams &pp, const PairF32 &pf, double r2, double qi, double qj, double dx,
                                 double dy, double dz) {
    const float sc = COUL ? pair_scalar_f32(pp, pf, r2, (float)(qi * qj)) : pair_scalar_lj_f32(pp, pf, r2);
    p[0] = fmaf(sc, (float)dx, p[0]);
    p[1] = fmaf(sc, (float)dy, p[1]);
    p[2] = fmaf(sc, (float)dz, p[2]);
  }
  __device__ inline void flush_row() {
    for (int c = 0; c < 3; ++c) {
      k.add(c, p[c]);
      p[c] = 0.f;
    }
  }
  // a row's terms of one chunk of a group walk, in order
  __device__ inline void add_terms(const float4 *t, int n) {
#pragma unroll 4
    for (int u = 0; u < n; ++u) {
      const float4 v = t[u];
      p[0] = fmaf(v.x, v.y, p[0]);
      p[1] = fmaf(v.x, v.z, p[1]);
      p[2] = fmaf(v.x, v.w, p[2]);
    }
  }
  // the sums of the group's rows in `rows` (bits), in order (every lane holds the total)
  template <int G>
  __device__ inline void flush_rows(uint64_t rows) {
    for (; rows; rows &= rows - 1)
      for (int c = 0; c < 3; ++c) k.add(c, __shfl(p[c], __ffsll((long long)rows) - 1, G));
    for (int c = 0; c < 3; ++c) p[c] = 0.f;
  }
  template <int G>
  __device__ inline double total(int c) const {
    return k.get(c);
  }
  template <bool COUL, bool TABLE = false>
  __device__ inline void add(const PairParams &pp, const PairF32 &pf, double r2, double qi, double qj, double dx,
                             double dy, double dz) {
    const float sc = COUL ? pair_scalar_f32(pp, pf, r2, (float)(qi * qj)) : pair_scalar_lj_f32(pp, pf, r2);
    k.add_prod(0, sc, (float)dx);
    k.add_prod(1, sc, (float)dy);
    k.add_prod(2, sc, (float)dz);
  }
  __device__ inline double get(int c) const { return k.get(c); }
};

// ---------------------------------------------------------------------------
// Queue walks: one lane per particle, candidates filtered on packed positions
// ---------------------------------------------------------------------------
// A thread-form walk that tests its candidates in two steps. The first reads
// 8 packed bytes per candidate (pack_position) and compares integer distances
// with a reach no pair inside the cutoff exceeds; the candidates that pass go
// to the lane's queue in LDS. The second takes a queue entry per lane, loads
// its FP64 record, classifies it exactly and evaluates it. What this buys: a
// lane's load of a 32-byte record keeps the CU's 64 bytes per clock return
// path busy for half a clock, so four SIMDs testing FP64 records wait on it
// (128 SIMD cycles per candidate and wave) whatever the arithmetic costs, and
// a pair term evaluated as soon as any lane holds a pair runs with a quarter
// to half of the lanes. The filter needs a quarter of the bytes and six
// integer instructions; the queues let the pair terms run with nearly all
// lanes, however the pairs are spread over the rows.
constexpr int kQueueCap = 32;       // entries per lane (a ring)
constexpr int kQueueThreads = 256;  // block size: entry e of a lane at [e * kQueueThreads]
constexpr int kCodeBits = 6;        // image shifts of an entry, two bits per axis
constexpr int kIndexBits = 32 - kCodeBits;

// A lane's ring of entries: byte offsets into the block's queue (slot e of
// lane t at 4 (e kQueueThreads + t)), so that a push is a store and a step of
// the offset.
struct HitQueue {
  char *lds;  // the block's queue
  uint32_t head, tail;
  uint32_t now = 0;  // image code of the piece being scanned
  static constexpr uint32_t kStep = 4 * kQueueThreads, kMask = kQueueCap * kStep - 1;
  __device__ inline HitQueue(uint32_t *queue) : lds((char *)queue), head(4 * threadIdx.x), tail(head) {}
  __device__ inline uint32_t pending() const { return (tail - head) & kMask; }  // in bytes: entries times kStep
  __device__ inline bool nearly_full() const { return pending() > (kQueueCap - 5) * kStep; }
  __device__ inline void push(uint32_t e) {
    *(uint32_t *)(lds + tail) = e;
    tail = (tail + kStep) & kMask;
  }
  __device__ inline uint32_t pop() {
    const uint32_t e = *(uint32_t *)(lds + head);
    head = (head + kStep) & kMask;
    return e;
  }
};
// Squared distance of two packed positions in grid units (each difference a
// signed 16-bit integer), at most 2^31 - 1. The clamp is there for far pairs;
// it also takes the three-operand form of the dot product, which needs no
// register cleared first.
__device__ inline uint32_t packed_dist2(uint32_t axy, uint32_t az, uint32_t bxy, uint32_t bz) {
  typedef short s2 __attribute__((ext_vector_type(2)));
  const s2 dxy = __builtin_bit_cast(s2, axy) - __builtin_bit_cast(s2, bxy);
  const s2 dz = __builtin_bit_cast(s2, az) - __builtin_bit_cast(s2, bz);
  return (uint32_t)__builtin_amdgcn_sdot2(dz, dz, __builtin_amdgcn_sdot2(dxy, dxy, 0, true), true);
}
// Shift of one axis (boxes) from a code's two bits.
__device__ inline double code_shift(uint32_t code, int axis) { return (double)((int)((code >> (2 * axis)) & 3u) - 1); }
constexpr uint32_t kNoShift = 0x15u;  // 1 on every axis

// Lanes of the wave for which v holds, as a scalar.
__device__ inline int wave_count(bool v) {
  return __builtin_amdgcn_readfirstlane(__popcll(__builtin_amdgcn_ballot_w64(v)));
}
// Largest v over the wave, as a scalar.
__device__ inline int wave_max(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return __builtin_amdgcn_readfirstlane(v);
}

// One species block of a queue walk, by the whole wave (lanes with active
// false take part without candidates): the rows of stencil s out to the
// squared reach r2 around pi, whose candidates within the integer squared
// reach t2 are queued. drain(all) empties the queues of the wave, all of them
// or only as far as it pays; it is called when a queue might overflow, and
// (`coded` false: entries have no room for the image code) with all = true at
// the end of every piece of a row, whose code is then the queue's `now`.
// gs, gpk: the ghost arrays (GHOST), entries indexed from nnat on.
template <bool GHOST, class Tested, class Drain>
__device__ inline void queue_walk(const Grid &g, const int32_t *__restrict__ cs, const uint2 *__restrict__ pk,
                                  const int32_t *__restrict__ gs, const uint2 *__restrict__ gpk, int nnat,
                                  bool active, const double4 &pi, const Sten &s, double r2, uint32_t t2,
                                  double scale, bool coded, HitQueue &Q, Tested &&tested, Drain &&drain) {
  typedef uint32_t quad __attribute__((ext_vector_type(4), aligned(8)));  // two packed records
  const int cx = cell_coord(pi.x, g.inv_h[0], g.nx), cy = cell_coord(pi.y, g.inv_h[1], g.ny),
            cz = cell_coord(pi.z, g.inv_h[2], g.nz);
  const RowFrame F(g, pi.x, pi.y, pi.z, cx, cy, cz, r2);
  const uint2 home = pack_position(pi.x, pi.y, pi.z, scale);
  const int my = wave_max(active ? s.y : 0), mz = wave_max(active ? s.z : 0);
  for (int oz = -mz; oz <= mz; ++oz) {
    const float gz = F.gap(F.uz, oz, F.hz);
    if (wave_count(active && gz * gz <= F.r2) == 0) continue;
    for (int oy = -my; oy <= my; ++oy) {
      const float gy = F.gap(F.uy, oy, F.hy);
      int a = 1, a_end = 0;
      const bool in = active && abs(oz) <= s.z && abs(oy) <= s.y && F.range(fmaf(gy, gy, gz * gz), s.x, &a, &a_end);
      if (wave_count(in) == 0) continue;
      const int y = cy + oy, z = cz + oz;
      a += cx;
      a_end += cx;
      bool more = in;
      for (int pass = 0;; ++pass) {
        int j0 = 0, len = 0;
        const uint2 *rec = pk;
        uint2 own = home;
        uint32_t code = GHOST ? 0u : kNoShift;
        if (more) {
          if (GHOST) {
            const bool inner = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
            if (pass == 0) {
              const int na = max(a, 0), nb = min(a_end, g.nx - 1);
              if (inner && na <= nb) {
                const int32_t *t = cs + (z * g.ny + y) * g.nx;
                j0 = t[na];
                len = t[nb + 1] - j0;
              }
              more = !inner || a < 0 || a_end >= g.nx;  // the padded cells over the native grid hold no ghosts
            } else {
              const int32_t *t = gs + ((z + g.goff[2]) * g.pny + (y + g.goff[1])) * g.pnx + g.goff[0];
              j0 = t[a];
              len = t[a_end + 1] - j0;
              more = false;
            }
          } else {
            int qx, qy, qz;
            const int wz = wrap_cell(z, g.nz, &qz), wy = wrap_cell(y, g.ny, &qy);
            const int32_t *t = cs + (wz * g.ny + wy) * g.nx;
            const int wa = wrap_cell(a, g.nx, &qx);
            const int b = min(a_end, (qx + 1) * g.nx - 1);
            j0 = t[wa];
            len = t[b - qx * g.nx + 1] - j0;
            a = b + 1;
            more = a <= a_end;
            code = (uint32_t)(qx + 1) | (uint32_t)(qy + 1) << 2 | (uint32_t)(qz + 1) << 4;
          }
        }
        if (GHOST) {
          if (pass) rec = gpk;
        } else if (wave_count(code != kNoShift)) {
          own = pack_position(pi.x - code_shift(code, 0) * g.L[0], pi.y - code_shift(code, 1) * g.L[1],
                              pi.z - code_shift(code, 2) * g.L[2], scale);
        }
        tested(len);
        Q.now = code;
        const uint32_t tag = GHOST ? (pass ? (uint32_t)nnat : 0u) : (coded ? code << kIndexBits : 0u);
        rec += j0;
        quad n0{}, n1{};
        if (len > 0) {
          n0 = *(const quad *)rec;
          n1 = *(const quad *)(rec + 2);
        }
        for (int k = 0, going = wave_count(k < len); going; k += 4) {
          if (k < len) {
            // four candidates, the next four requested before them (up to 7
            // records past the end are read: padding)
            const uint32_t xy[4] = {n0.x, n0.z, n1.x, n1.z}, zz[4] = {n0.y, n0.w, n1.y, n1.w};
            n0 = *(const quad *)(rec + k + 4);
            n1 = *(const quad *)(rec + k + 6);
            const uint32_t e = (uint32_t)(j0 + k) + tag;
            const int rest = len - k;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if ((packed_dist2(own.x, own.y, xy[u], zz[u]) <= t2) & (rest > u)) Q.push(e + u);
            }
          }
          going = wave_count(k + 4 < len);
          const bool piece = !GHOST && !coded && going == 0;  // its code is not in the entries
          if (piece || wave_count(Q.nearly_full())) drain(piece);
        }
        if (wave_count(more) == 0) break;
      }
    }
  }
}

// The steps of a drain: one(e) for an entry of every lane that has one, until
// all queues are empty (all), or until none is close to overflowing and fewer
// than three quarters of the lanes would take part.
template <class One>
__device__ inline void drain_queue(HitQueue &Q, bool all, One &&one) {
  for (;;) {
    const bool any = Q.pending() != 0;
    if (wave_count(any) < (all || wave_count(Q.nearly_full()) ? 1 : 48)) return;
    if (any) one(Q.pop());
  }
}

// Particles of a part up to which a group of lanes shares one (group walk) in
// its plain sums; above, one thread each (queue walk, FP32C: thread form). One
// thread each leaves the chip nearly idle below a few hundred thousand
// particles: its time is then that of one particle's walk. Measured on one
// MI355X, thread form against 64 and 32 lanes, in us: charged FP64 (r = 6, 8)
// 1,000 particles 393, 11, 22; 25,000: 410, 86, 88; 100,000: 536, 312, 295 (10 %
// charged, 80,000: 294, 224, 187 and ten times that many 1280, -, 1850). Neutral
// FP64 (LJ only) 45,000: 77, 77, 54; 100,000: 82, 151, 98. FP32C 25,000: 283, 91,
// 81; 100,000: 318, 322, 265; 80,000 of a sparse kind: 150, 239, 160.
// With few particles in the reach a wave has little to share, and the lines
// lie lower (mean: particles within the reach of one). The kernel alone, one
// thread against 32 lanes: FP64 charged, mean 1 20,000: 22, 19; 48,000: 23, 42;
// mean 4 48,000: 30, 45; mean 16 100,000: 54, 99; neutral, mean 2 48,000: 33,
// 43; FP32C mean 1 20,000: 18, 18; mean 4: 24, 20. A whole force call FP64
// charged, mean 20 60,000: 109, 98; 120,000: 131, 160; mean 100 120,000: 237,
// 229; 200,000: 325, 362; FP32C mean 10 40,000: 90, 95; mean 40 60,000: 114, 109.
inline int64_t group_most(bool f32, bool charged, double mean) {
  if (mean < (charged && !f32 ? 12.0 : 24.0)) return 32768;
  return charged && !f32 && mean >= 48.0 ? 262144 : 65536;
}
// Mean number of particles within r of one of the n in the grid's box.
inline double mean_within(const Grid &g, int64_t n, double r) {
  return (double)n / (g.L[0] * g.L[1] * g.L[2]) * (4.0 / 3.0) * kPi * r * r * r;
}
// Blocks of a group launch over up to `most` particles (each block takes a
// run of consecutive ones; enough for several waves per SIMD, and few enough
// that a launch whose part turns out empty or large ends in about 4 us).
inline unsigned group_blocks(int64_t most, int lanes) {
  const int64_t nb = (most * lanes + 255) / 256;
  return (unsigned)(nb < 4096 ? nb : 4096);
}

// Plain sums of particle i by its group: charged i against the charged block
// out to max(r_coul, r_lj) and the neutral block out to r_lj, neutral i
// against both out to r_lj; coulomb: the screened Coulomb terms alone.
// tested(coul, other, r^2) is called for every candidate (other: it is not i).
template <bool F32, bool GHOST, int G, class Tested>
__device__ inline void group_sums(const PairParams &pp, const PairF32 &pf, const Grid &g, const Sten &s_coul,
                                  const Sten &s_lj, const int32_t *__restrict__ cell_start,
                                  const double4 *__restrict__ xq, const int32_t *__restrict__ gcell_start,
                                  const double4 *__restrict__ gxq, int nnat, int i, const double4 &pi, bool coulomb,
                                  GroupRows<G> &rows, float4 *terms, ForceAcc<F32> &acc, Tested &&tested) {
  const double qi = pi.w;
  const bool charged = qi != 0.0;
  const Block near_lj = pp.do_lj ? Block{s_lj, pp.rlj2} : no_block();
  const Block A = coulomb ? Block{s_coul, pp.rc2}
                  : !charged ? near_lj
                  : pp.do_coul || pp.do_lj ? Block{s_coul, pp.rq2}
                                           : no_block();
  const Block B = coulomb ? no_block() : near_lj;
  group_walk<G, GHOST>(
      g, cell_start, xq, gcell_start, gxq, nnat, pi, A, B, rows,
      [&](bool ok, int k, int blk, int j, const double4 &pj, double dx, double dy, double dz, double r2) {
        const bool coul = charged && blk == 0;  // every other pairing: LJ only
        const bool in = ok & (j != i) & (r2 <= (coul ? A.r2 : pp.rlj2));
        if (ok) tested(coul, j != i, r2);
        if constexpr (F32) {
          float sc = 0.f;
          if (in) sc = coul ? pair_scalar_f32(pp, pf, r2, (float)(qi * pj.w)) : pair_scalar_lj_f32(pp, pf, r2);
          terms[k] = in ? make_float4(sc, (float)dx, (float)dy, (float)dz) : make_float4(0.f, 0.f, 0.f, 0.f);
        } else if (in) {
          if (coul) acc.template add<true>(pp, pf, r2, qi, pj.w, dx, dy, dz);
          else acc.template add<false>(pp, pf, r2, qi, pj.w, dx, dy, dz);
        }
      },
      [&](int first, int len) {
        if constexpr (F32) acc.add_terms(terms + first, len);
      },
      [&](uint64_t reached) {
        if constexpr (F32) acc.template flush_rows<G>(reached);
      });
}

}  // namespace rbe

namespace rbe {

// ---------------------------------------------------------------------------
// Cluster traversal (8 x 8 lanes per wave)
// ---------------------------------------------------------------------------
// A wave computes the near field of a cluster of up to kCI consecutive
// particles of the cell order. Lane l plays i = cluster[l / kCJ] against the
// j-stream offset l % kCJ: the wave walks one shared sequence of candidate
// records kCJ at a time, so a load instruction touches kCJ consecutive
// records (two cache lines) and every lane runs the same loop. Particles of a
// cluster that lie in different cell rows (or species blocks, or replicas)
// are handled one row group after another; a group walks the union of its
// particles' stencils: the stencil rows around (cy, cz) with x running from
// min(cx) - s to max(cx) + s.
constexpr int kCI = 8;
constexpr int kCJ = 8;

// Buffer resource over `bytes` bytes at p (gfx9 raw buffer, no stride):
// loads that start past the end return zeros instead of touching memory.
__device__ inline __amdgpu_buffer_rsrc_t bounded_rsrc(const void *p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, bytes, 0x00020000);
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ inline double dword_pair(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// Record k of a segment (zeros past its end).
__device__ inline double4 load_record(__amdgpu_buffer_rsrc_t r, int k) {
  const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(r, k * 32, 0, 0);
  const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(r, k * 32 + 16, 0, 0);
  return make_double4(dword_pair(a.x, a.y), dword_pair(a.z, a.w), dword_pair(c.x, c.y), dword_pair(c.z, c.w));
}

// fn(ok, j, p_j, id_j, shx, shy, shz) for the records j0..j1-1 taken by this
// lane (j = jofs + j0 + b, jofs + j0 + b + kCJ, ...: jofs separates the index
// ranges of different arrays, natives 0 and ghosts n; ok = false on trips
// where this lane's record is past j1), one record prefetched ahead, then tick() once per trip with
// the whole wave. The trip count depends only on j0, j1, so the loop is the
// same for the wave; the segment is read through bounded buffer loads, so the
// lookahead needs no clamping.
template <bool WITH_ID, class Fn, class Tick>
__device__ inline void scan_cluster(const double4 *__restrict__ xq, const int32_t *__restrict__ ids, int j0, int j1,
                                    int b, double shx, double shy, double shz, Fn &&fn, Tick &&tick, int jofs = 0) {
  j0 = __builtin_amdgcn_readfirstlane(j0);  // uniform by construction; tell the compiler
  j1 = __builtin_amdgcn_readfirstlane(j1);
  if (j0 >= j1) return;
  const int cnt = j1 - j0;
  const __amdgpu_buffer_rsrc_t rx = bounded_rsrc(xq + j0, cnt * (int)sizeof(double4));
  const __amdgpu_buffer_rsrc_t ri = bounded_rsrc(WITH_ID ? ids + j0 : ids, WITH_ID ? cnt * 4 : 0);
  auto load_id = [&](int k) { return WITH_ID ? (int)__builtin_amdgcn_raw_buffer_load_b32(ri, k * 4, 0, 0) : 0; };
  int k = b;
  double4 r0 = load_record(rx, k);
  int d0 = load_id(k);
#pragma unroll 1
  for (int base = 0;; base += 2 * kCJ) {
    const double4 r1 = load_record(rx, k + kCJ);
    const int d1 = load_id(k + kCJ);
    fn(k < cnt, jofs + j0 + k, r0, d0, shx, shy, shz);
    tick();
    if (base + kCJ >= cnt) break;
    r0 = load_record(rx, k + 2 * kCJ);
    d0 = load_id(k + 2 * kCJ);
    fn(k + kCJ < cnt, jofs + j0 + k + kCJ, r1, d1, shx, shy, shz);
    tick();
    if (base + 2 * kCJ >= cnt) break;
    k += 2 * kCJ;
  }
}

// Row tables of a cluster walk: lane t of the wave resolves stencil row
// r0 + t (rows ordered z-major) into the cell-table bounds of its segments,
// so the cell-table loads of up to 64 rows are in flight together instead of
// one dependent pair per row; the walk then takes each row's bounds from its
// lane (wave-uniform reads).
struct RowSegs {
  int j0a, j1a, j0b, j1b;  // up to two segments of the row
  int qxa, qxb, qy, qz;    // their image shifts in boxes
};
__device__ inline RowSegs row_segs_at(const RowSegs &v, int k) {
  RowSegs u;
  u.j0a = __builtin_amdgcn_readlane(v.j0a, k);
  u.j1a = __builtin_amdgcn_readlane(v.j1a, k);
  u.j0b = __builtin_amdgcn_readlane(v.j0b, k);
  u.j1b = __builtin_amdgcn_readlane(v.j1b, k);
  u.qxa = __builtin_amdgcn_readlane(v.qxa, k);
  u.qxb = __builtin_amdgcn_readlane(v.qxb, k);
  u.qy = __builtin_amdgcn_readlane(v.qy, k);
  u.qz = __builtin_amdgcn_readlane(v.qz, k);
  return u;
}

// Periodic walk of species block `blk` (keys base + blk * C + cell) for a row
// group: rows (cy + oy, cz + oz), |oy| <= s.y, |oz| <= s.z, x from xa - s.x
// to xb + s.x, each row split where it crosses the periodic boundary (a cell
// met twice is met with two different image shifts, so no image is counted
// twice).
template <bool WITH_ID, class Fn, class Tick>
__device__ inline void cluster_walk(const Grid &g, const int32_t *__restrict__ cell_start,
                                    const double4 *__restrict__ xq, const int32_t *__restrict__ ids, int64_t base,
                                    int xa, int xb, int cy, int cz, const Sten &s, int b, Fn &&fn,
                                    Tick &&tick) {
  const int x0 = xa - s.x, x1 = xb + s.x;
  if (x1 - x0 + 1 > g.nx) {
    // the range wraps more than once (boxes of few cells): row by row
    for (int oz = -s.z; oz <= s.z; ++oz) {
      const int az = cz + oz;
      const int qz = floor_div(az, g.nz);
      const double shz = (double)qz * g.L[2];
      for (int oy = -s.y; oy <= s.y; ++oy) {
        const int ay = cy + oy;
        const int qy = floor_div(ay, g.ny);
        const double shy = (double)qy * g.L[1];
        const int64_t row = base + (int64_t)((az - qz * g.nz) * g.ny + (ay - qy * g.ny)) * g.nx;
        int x = x0;
        while (x <= x1) {
          const int qx = floor_div(x, g.nx);
          const int xe = min(x1, (qx + 1) * g.nx - 1);
          const int j0 = cell_start[row + (x - qx * g.nx)];
          const int j1 = cell_start[row + (xe - qx * g.nx) + 1];
          scan_cluster<WITH_ID>(xq, ids, j0, j1, b, (double)qx * g.L[0], shy, shz, fn, tick);
          x = xe + 1;
        }
      }
    }
    return;
  }
  const int lane = threadIdx.x & 63;
  const int nyr = 2 * s.y + 1, nrows = nyr * (2 * s.z + 1);
  for (int r0 = 0; r0 < nrows; r0 += 64) {
    RowSegs v{0, 0, 0, 0, 0, 0, 0, 0};
    const int r = r0 + lane;
    if (r < nrows) {
      const int az = cz + r / nyr - s.z, ay = cy + r % nyr - s.y;
      v.qz = floor_div(az, g.nz);
      v.qy = floor_div(ay, g.ny);
      const int64_t row = base + (int64_t)((az - v.qz * g.nz) * g.ny + (ay - v.qy * g.ny)) * g.nx;
      v.qxa = floor_div(x0, g.nx);
      const int ea = min(x1, (v.qxa + 1) * g.nx - 1);
      v.j0a = cell_start[row + (x0 - v.qxa * g.nx)];
      v.j1a = cell_start[row + (ea - v.qxa * g.nx) + 1];
      if (ea < x1) {  // wraps once: the rest lies in the next image
        v.qxb = v.qxa + 1;
        v.j0b = cell_start[row];
        v.j1b = cell_start[row + (x1 - v.qxb * g.nx) + 1];
      }
    }
    const int nr = min(64, nrows - r0);
    for (int k = 0; k < nr; ++k) {
      const RowSegs u = row_segs_at(v, k);
      const double shy = (double)u.qy * g.L[1], shz = (double)u.qz * g.L[2];
      scan_cluster<WITH_ID>(xq, ids, u.j0a, u.j1a, b, (double)u.qxa * g.L[0], shy, shz, fn, tick);
      scan_cluster<WITH_ID>(xq, ids, u.j0b, u.j1b, b, (double)u.qxb * g.L[0], shy, shz, fn, tick);
    }
  }
}

// Ghost-shell walk (no periodic images): the native part of each stencil row
// clipped to the native grid, then the same row of the padded ghost grid
// (row tables as in the periodic walk: segment a native, segment b ghost).
// Ghost records are passed to fn with indices offset by nnat, so no ghost
// index equals a native one.
template <bool WITH_ID, class Fn, class Tick>
__device__ inline void cluster_walk_ghost(const Grid &g, const int32_t *__restrict__ cell_start,
                                          const double4 *__restrict__ xq, const int32_t *__restrict__ ids,
                                          const int32_t *__restrict__ gcell_start, const double4 *__restrict__ gxq,
                                          const int32_t *__restrict__ gid, int nnat, int blk, int xa, int xb,
                                          int cy, int cz, const Sten &s, int b, Fn &&fn, Tick &&tick) {
  const int64_t base = (int64_t)blk * g.ncell;
  const int64_t pbase = (int64_t)blk * g.pncell;
  const int na = max(xa - s.x, 0), nb = min(xb + s.x, g.nx - 1);
  const int lane = threadIdx.x & 63;
  const int nyr = 2 * s.y + 1, nrows = nyr * (2 * s.z + 1);
  for (int r0 = 0; r0 < nrows; r0 += 64) {
    RowSegs v{0, 0, 0, 0, 0, 0, 0, 0};
    const int r = r0 + lane;
    if (r < nrows) {
      const int z = cz + r / nyr - s.z, y = cy + r % nyr - s.y;
      if (z >= 0 && z < g.nz && y >= 0 && y < g.ny) {
        const int64_t row = base + (int64_t)(z * g.ny + y) * g.nx;
        v.j0a = cell_start[row + na];
        v.j1a = cell_start[row + nb + 1];
      }
      const int64_t prow = pbase + (int64_t)((z + g.goff[2]) * g.pny + (y + g.goff[1])) * g.pnx + g.goff[0];
      v.j0b = gcell_start[prow + xa - s.x];
      v.j1b = gcell_start[prow + xb + s.x + 1];
    }
    const int nr = min(64, nrows - r0);
    for (int k = 0; k < nr; ++k) {
      const RowSegs u = row_segs_at(v, k);
      scan_cluster<WITH_ID>(xq, ids, u.j0a, u.j1a, b, 0.0, 0.0, 0.0, fn, tick);
      scan_cluster<WITH_ID>(gxq, gid, u.j0b, u.j1b, b, 0.0, 0.0, 0.0, fn, tick, nnat);
    }
  }
}

// Row groups of a cluster wave. `valid`: this lane's i exists; rowkey: a
// value shared exactly by the particles of one cell row (and species block,
// and replica). Calls gfn(in, leader, xa, xb) once per distinct row, where
// `in` says whether this lane's i belongs to the group, `leader` is a lane of
// the group and [xa, xb] the group's x-cell range (all wave-uniform).
template <class GroupFn>
__device__ inline void for_each_row_group(bool valid, int64_t rowkey, int cx, GroupFn &&gfn) {
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(valid && (lane % kCJ) == 0);
  while (todo) {
    const int leader = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
    const int64_t R = __shfl(rowkey, leader, 64);
    const bool in = valid && rowkey == R;
    int xa = in ? cx : 0x7FFFFFFF, xb = in ? cx : -0x7FFFFFFF;
#pragma unroll
    for (int o = kCJ; o < 64; o <<= 1) {
      xa = min(xa, __shfl_xor(xa, o, 64));
      xb = max(xb, __shfl_xor(xb, o, 64));
    }
    xa = __builtin_amdgcn_readfirstlane(xa);
    xb = __builtin_amdgcn_readfirstlane(xb);
    gfn(in, leader, xa, xb);
    todo &= ~__ballot(in && (lane % kCJ) == 0);
  }
}

// Sum over the kCJ lanes that share an i (fixed order: deterministic).
__device__ inline double sum_j_lanes(double v) {
#pragma unroll
  for (int o = 1; o < kCJ; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline int sum_j_lanes(int v) {
#pragma unroll
  for (int o = 1; o < kCJ; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace rbe
