// Smallest eigenpair of a small Hermitian matrix (n <= 64) held in
// double-double, by one workgroup of C = 2 .. 8 waves, n <= 8 C: the solver of
// the forms whose Gram is double-double (FP64, MIXED).  The steps are those
// of eigsmall.h -- Householder tridiagonalisation, Sturm multisection,
// X = (T - sigma I)^{-1}, inverse iteration, Newton refinement against the
// double-double matrix -- laid out for latency:
//
//  * Thread (r, q) = (tid / 8, tid mod 8) holds the entries (r, q + 8 i), i < C,
//    of the matrix and of the accumulated unitary Q in registers; eight
//    neighbouring lanes share a row, so a product with a vector is C
//    multiply-adds and three lane exchanges, and only vectors pass through
//    LDS (two barriers per reflector).
//  * Q is accumulated beside the reduction (its product and update fill the
//    latency of the matrix's own), so W = Q D is applied afterwards as one
//    product instead of n - 2 reflectors with a wave sum each.
//  * The Sturm counts use the leading principal minors' two-term recurrence
//    p_k = (a_k - t) p_{k-1} - b_{k-1}^2 p_{k-2} (one dependent FMA per step
//    and no reciprocal), rescaled by a power of two every eight steps (T has a
//    norm near 1 and b^2 is kept above 2^-200, so eight steps shrink the pair by
//    2^-800 at most); the number of sign changes is the number of eigenvalues
//    below t.  The
//    bracket starts at [0, min a_k] (Rayleigh; the matrix is positive
//    semidefinite) instead of the Gershgorin interval, with a graded first
//    round: a pair of noiseless frames' smallest eigenvalues sit at rounding
//    level (64x64 FP64, both solves: 77 -> 73.6 us a call; 719x1277 164.5 ->
//    159.5; noisy pairs within 1 us).
//
// Measured against the one-wave solver (launch times, one frame): sample
// solves of order 10 / 20 / 32: 37 / 68 / 126 -> 18 / 29 / 41 us; scale solves
// of order 10 / 22 / 34: 37 / 76 / 146 -> 22 / 36 / 76 us (their setup and
// assembly on every wave included).
//
// What bounds it: the dependent chain of a reflector (two barriers, three
// LDS round trips, a wave sum, a reciprocal root and a reciprocal), not
// arithmetic.  The loops are kept free of branches on lanes: vectors are
// zero-padded to 64 entries in LDS and read without masks, dead rows and
// columns are transformed along (they hold the exact zeros of the reduced
// matrix up to rounding and are not read again), and lanes that own nothing
// store to a dump slot.  Every sum is formed in an order that depends on n
// alone (padding adds exact zeros), with explicit FMAs, so the result does
// not depend on C.  A reflector takes ~1500 cycles at C = 2 .. 4 (6 cycles per
// instruction: about 220 .. 280 of them and the two LDS round trips); from C = 5
// on two waves share a SIMD and it takes up to twice as long.
//
// Many solves in a launch are bound by instructions instead, so what one wave
// can do the others leave alone: the bisection, the factors and X are the first
// wave's, and a wave whose rows are reduced takes part in Q only.  On every wave
// / so, FP64 calls of one frame with kernels of 18 and 17 184 / 170 us, 21 and 20
// 240 / 202 (six waves instead of eight), 32 and 32 325 / 303; of 400 frames of
// 48x40 4.91 / 4.50 ms, 7.89 / 6.41, 15.5 / 14.7 (18 and 17 then 4.15 by
// many_solves in recover.hip; the one-wave solver took 4.18, 6.83, 39.3).
#pragma once

#include "eigsmall.h"

namespace cbp {

constexpr int BLK_MAX_WAVES = 8;

// Powers of two that the norm of block_eig's matrix lies between (2^-464 is
// 2e-140, 2^511 is 7e153); beyond them it returns a NaN vector, which the
// callers turn into zero kernels and diagnostic flags.
constexpr int BLK_MIN_EXP = -464, BLK_MAX_EXP = 511;

// ---------------------------------------------------------------- explicit-FMA complex helpers
__device__ inline c64 cfma(c64 a, c64 b, c64 s) {      // s + a b
  return {fma(a.re, b.re, fma(-a.im, b.im, s.re)), fma(a.re, b.im, fma(a.im, b.re, s.im))};
}
__device__ inline c64 cfms_bc(c64 a, c64 b, c64 s) {   // s - a conj(b)
  return {fma(-a.re, b.re, fma(-a.im, b.im, s.re)), fma(a.re, b.im, fma(-a.im, b.re, s.im))};
}
__device__ inline c64 crfms(double g, c64 a, c64 s) {  // s - g a
  return {fma(-g, a.re, s.re), fma(-g, a.im, s.im)};
}
// (a struct-valued ?: may select between addresses, which would put both
// values in scratch memory)
__device__ inline c64 csel(bool c, c64 a, c64 b) { return {c ? a.re : b.re, c ? a.im : b.im}; }
__device__ inline double cnorm2(c64 a) { return fma(a.re, a.re, a.im * a.im); }
__device__ inline double cdotr(c64 a, c64 b) { return fma(a.re, b.re, a.im * b.im); }   // Re(conj(a) b)

// Sum over the eight lanes of a row (in every lane of the row).
__device__ inline double sum8(double v) {
  v += dpp_z<0xB1>(v);     // quad_perm [1,0,3,2]
  v += dpp_z<0x4E>(v);     // quad_perm [2,3,0,1]
  v += dpp_z<0x141>(v);    // row_half_mirror
  return v;
}
__device__ inline c64 sum8(c64 v) { return {sum8(v.re), sum8(v.im)}; }

// Sum over the wave's eight rows of a value equal in the lanes of a row.
__device__ inline double sum_rows(double v) {
  v += dpp_z<0x128>(v);    // row_ror:8: the two rows of each 16 lanes
  v += dpp_z<0x142>(v);    // row_bcast:15
  v += dpp_z<0x143>(v);    // row_bcast:31
  return readlane_d(v, 63);
}

// The same in double-double.
__device__ inline dd sum_rows(dd v) {
  v = dd_add(v, dpp_dd<0x128>(v));
  v = dd_add(v, dpp_dd<0x142>(v));
  v = dd_add(v, dpp_dd<0x143>(v));
  return {readlane_d(v.hi, 63), readlane_d(v.lo, 63)};
}

// Reciprocal and reciprocal square root: hardware estimate (2^-23 or
// better) and one third-order step (error below 2^-68 before rounding).
__device__ inline double rcp_h(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ inline double rsq_h(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// ---------------------------------------------------------------- workspace (LDS)
struct blk_ws {
  c64* v0;        // 64: vector buffers, zero beyond the rows in use
  c64* v1;        // 64
  c64* x;         // 64: the result
  c64* dump;      // 64: stores of lanes that own nothing
  double2* ab;    // 72: {a_k, b_(k-1)^2} scaled to norm ~1, padded with {4, 0}
  double2* fac;   // 72: LDL^T factors {1 / d_k, b_k / d_k}, zero past the matrix
  double* part;   // 6 x BLK_MAX_WAVES: partial sums of the waves
  c64* M;         // n x (n + 1): W = Q D for its transpose, then X (doubles)
};

constexpr size_t blk_fixed_bytes() {
  return 64 * 4 * sizeof(c64) + (72 + 72) * sizeof(double2) + 6 * BLK_MAX_WAVES * sizeof(double);
}
// (X is held with its rows rounded up to a multiple of eight)
__host__ __device__ inline size_t blk_matrix_bytes(int n) {
  return (size_t)(n < 8 ? 8 : n) * (n + 1) * sizeof(c64);
}

// fixed: blk_fixed_bytes(); matrix: blk_matrix_bytes(n), free for the
// caller's use before the solve (as long as acc does not read it) and after.
__device__ inline blk_ws blk_carve(char* fixed, char* matrix) {
  blk_ws s;
  s.v0 = (c64*)fixed;
  s.v1 = s.v0 + 64;
  s.x = s.v1 + 64;
  s.dump = s.x + 64;
  s.ab = (double2*)(s.dump + 64);
  s.fac = s.ab + 72;
  s.part = (double*)(s.fac + 72);
  s.M = (c64*)matrix;
  return s;
}

// The C waves' partial sums p[0..C) (C <= 8) as a fixed tree over eight slots
// (missing ones are zero).
template <int C>
__device__ inline double wave_parts(const double* p) {
  double v[8];
#pragma unroll
  for (int w = 0; w < 8; ++w) v[w] = w < C ? p[w] : 0.0;
  return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// The same in double-double (high parts in hi, low parts in lo), without the
// missing slots: a zero added to a normalised double-double changes nothing.
template <int C>
__device__ inline dd wave_parts(const double* hi, const double* lo) {
  dd v[C];
#pragma unroll
  for (int w = 0; w < C; ++w) v[w] = {hi[w], lo[w]};
#pragma unroll
  for (int n = 1; n < C; n *= 2)
#pragma unroll
    for (int w = 0; w + n < C; w += 2 * n) v[w] = dd_add(v[w], v[w + n]);
  return v[0];
}

// Sum over the block of a value equal in the eight lanes of each row.  slot:
// the row of s.part used (free again two barriers later), slot and slot2 for a
// double-double.  Contains a barrier.
template <int C>
__device__ inline double block_rows_sum(const blk_ws& s, int slot, double v) {
  double* p = s.part + slot * BLK_MAX_WAVES;
  p[threadIdx.x >> 6] = sum_rows(v);
  __syncthreads();
  return wave_parts<C>(p);
}
template <int C>
__device__ inline dd block_rows_sum(const blk_ws& s, int slot, int slot2, dd v) {
  double* h = s.part + slot * BLK_MAX_WAVES;
  double* l = s.part + slot2 * BLK_MAX_WAVES;
  v = sum_rows(v);
  h[threadIdx.x >> 6] = v.hi;
  l[threadIdx.x >> 6] = v.lo;
  __syncthreads();
  return wave_parts<C>(h, l);
}

// ---------------------------------------------------------------- 2. Sturm counts
// Eigenvalues of the scaled T (ab) below t: sign changes of the leading
// principal minors of T - t I, eight steps per load of the entries (the next
// eight in flight); the padding entries {4, 0} change no sign for t < 4.
__device__ inline int sturm_minors(const double2* ab, int n, double t) {
  double p0 = 1.0, p1 = 1.0;
  unsigned c = 0;
  double2 f[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) f[u] = ab[u];
  for (int k0 = 0; k0 < n; k0 += 8) {
    double2 g[8];
    const double2* nx = ab + min(k0 + 8, 64);
#pragma unroll
    for (int u = 0; u < 8; ++u) g[u] = nx[u];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double m = f[u].y * p0;
      p0 = p1;
      p1 = fma(f[u].x - t, p1, -m);
      c += (unsigned)(__double2hiint(p1) ^ __double2hiint(p0)) >> 31;
    }
    // rescale the pair by a power of two (exact; the signs stay)
    const int e0 = __builtin_amdgcn_frexp_exp(p0), e1 = __builtin_amdgcn_frexp_exp(p1);
    const int e = p1 == 0.0 ? e0 : max(e0, e1);
    p0 = __builtin_amdgcn_ldexp(p0, -e);
    p1 = __builtin_amdgcn_ldexp(p1, -e);
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] = g[u];
  }
  return (int)c;
}

// T (lane l of every wave: a_l and |e_l| = b_l, zero past the matrix) scaled
// by the power of two 2^-*ex to norm in [1/2, 1) into s.ab (squared
// off-diagonals kept above 2^-200: a split T perturbed far below rounding).
// Returns the scaled Gershgorin bounds and norm; the caller synchronises.
__device__ inline void scale_tridiag(const blk_ws& s, int n, double a, double b, int* ex, double* glo_o,
                                     double* ghi_o, double* tn_o) {
  const int l = threadIdx.x & 63;
  // b_(l-1): the previous lane's b
  const double bl = __shfl_up(b, 1);
  const double bp = l > 0 ? bl : 0.0;
  const double glo = wmin(l < n ? a - bp - b : 1.7976931348623157e308);
  const double ghi = wmax(l < n ? a + bp + b : -1.7976931348623157e308);
  const double tn = fmax(fabs(glo), fabs(ghi));
  const int e = (tn > 0.0 && tn < 1.0e300) ? __builtin_amdgcn_frexp_exp(tn) : 0;
  if (threadIdx.x < 64) {
    const double bs = __builtin_amdgcn_ldexp(bp, -e);
    s.ab[l] = l < n ? double2{__builtin_amdgcn_ldexp(a, -e), l > 0 ? fmax(bs * bs, 0x1p-200) : 0.0} : double2{4.0, 0.0};
    if (l < 8) s.ab[64 + l] = double2{4.0, 0.0};
  }
  *ex = e;
  *glo_o = __builtin_amdgcn_ldexp(glo, -e);
  *ghi_o = __builtin_amdgcn_ldexp(ghi, -e);
  *tn_o = __builtin_amdgcn_ldexp(tn, -e);
}

// Bracket of the target-th smallest eigenvalue of the scaled T, each wave by
// itself with 64 probes per round (the first at lo), to a width of 6e-15 tn.
// GRADED (target 1): the first round's probes are graded, 32 of them evenly
// over [hi / 32, hi] and 32 a factor of 2.5 apart below, down to 1.4e-14 hi.  An
// eigenvalue near hi takes the same eight rounds as evenly spaced probes, one at
// the noise floor of a Gram (1e-9) four, and one at rounding level two.
template <bool GRADED = false>
__device__ inline void bisect_minors(const blk_ws& s, int n, int target, double glo, double ghi, double tn,
                                     double* lo_o, double* hi_o) {
  const int l = threadIdx.x & 63;
  const double pad = 2.2e-16 * tn + 1e-300;
  double lo = fmax(glo - pad, -64.0 * pad), hi = ghi + pad;
  if (target == 1) hi = fmin(hi, wmin(s.ab[l].x) + 4.0 * pad);
  if (GRADED) {
    const double h = hi * (1.0 / 32.0);
    auto probe = [&](int j) __attribute__((always_inline)) {
      return j > 31 ? h * (double)(j - 31) : h * (double)__builtin_amdgcn_exp2f(1.3219281f * (float)(j - 31));
    };
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(sturm_minors(s.ab, n, probe(l)) >= 1);
    const int js = mask ? __builtin_ctzll(mask) : 64;
    if (js > 0) lo = probe(min(js, 63) - 1);
    if (js < 64) hi = probe(js);
  }
  for (int it = 0; it < 10; ++it) {
    if (__builtin_amdgcn_ballot_w64(hi - lo > 6e-15 * tn) == 0) break;
    const double h = (hi - lo) * (1.0 / 64.0);
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(sturm_minors(s.ab, n, fma(h, (double)l, lo)) >= target);
    const int js = mask ? __builtin_ctzll(mask) : 64;   // first probe above the eigenvalue
    if (js == 0) {             // below the start of the bracket (an indefinite matrix)
      hi = lo;
      lo = glo - pad;
      continue;
    }
    const double l0 = lo;
    lo = fma(h, (double)(js - 1), l0);
    if (js < 64) hi = fma(h, (double)js, l0);
  }
  *lo_o = lo;
  *hi_o = hi;
}

// Every eigenvalue of T on a log scale (see small_spectrum): the eight lanes
// of row r bisect the (r+1)-th smallest to 1/9 of its bracket per
// round.  Returns it in every lane of the group (r < n), to 15 / 9^9 decades;
// s.ab is the scaled T of scale_tridiag (only ratios of the values are used).
__device__ inline __attribute__((always_inline)) double block_spectrum(const blk_ws& s, int n, double ghi) {
  const int r = (int)threadIdx.x >> 3, q = threadIdx.x & 7;
  const double top = log10(fmax(ghi, 1e-300));
  double lo = top - 15.0, hi = top;
  for (int it = 0; it < 9; ++it) {
    const double h = (hi - lo) * (1.0 / 9.0);
    const bool hit = sturm_minors(s.ab, n, exp10(fma(h, (double)(q + 1), lo))) >= r + 1;
    const unsigned m = (unsigned)(__builtin_amdgcn_ballot_w64(hit) >> (threadIdx.x & 56)) & 0xffu;
    const int js = m ? __builtin_ctz(m) : 8;
    hi = js < 8 ? fma(h, (double)(js + 1), lo) : hi;
    lo = fma(h, (double)js, lo);
  }
  return exp10(0.5 * (lo + hi));
}

// ---------------------------------------------------------------- 1. reduction
// Steps k = o - 1 of the Householder reduction with o >> 3 == I0 (the columns
// of groups i >= I0 are live).  v0 holds column k of the rows >= o, zero
// elsewhere, on entry; el collects e_k in lane k of every wave.  Q: accumulate the
// unitary in w.
template <int C, int I0, bool Q>
__device__ inline __attribute__((always_inline)) void block_reflectors(const blk_ws& s, int n, c64* a, c64* w, c64& el) {
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6, r = tid >> 3, q = tid & 7;
  const int o1 = min(8 * I0 + 8, n - 1);
  // rows below 8 I0 are reduced: their waves (one of them at least live) take
  // part in Q alone, with no share in u^H p
  const bool live_rows = __builtin_amdgcn_readfirstlane(wv) >= I0;
#pragma unroll 1
  for (int o = I0 ? 8 * I0 : 1; o < o1; ++o) {
    __syncthreads();
    const c64 xl = s.v0[l], x0 = s.v0[o];
    c64 ur = s.v0[r], u[C];
#pragma unroll
    for (int i = I0; i < C; ++i) u[i] = s.v0[q + 8 * i];
    const double ax0sq = cnorm2(x0);
    const double r0 = rsq_h(ax0sq > 0.0 ? ax0sq : 1.0);   // 1 / |x_0|, overlapping the sum
    const double tail = wsum(l > o ? cnorm2(xl) : 0.0);
    const bool live = tail > 0.0;                         // else reflector k = I
    const double s2 = ax0sq + tail;
    const double nx = s2 * rsq_h(live ? s2 : 1.0);
    const double ax0 = ax0sq > 0.0 ? ax0sq * r0 : 0.0;
    const c64 ph = csel(ax0sq > 0.0, c64{x0.re * r0, x0.im * r0}, c64{1.0, 0.0});
    const c64 alpha = csel(live, c64{-ph.re * nx, -ph.im * nx}, x0);
    // u = x - alpha e_0, H = I - beta u u^H
    const double beta = live ? rcp_h(fma(nx, ax0, s2)) : 0.0;
    const c64 u0 = {x0.re - alpha.re, x0.im - alpha.im};
    u[I0] = csel(q + 8 * I0 == o, u0, u[I0]);
    ur = csel(r == o, u0, ur);
    el = csel(l == o - 1, alpha, el);
    // p = beta A u, z = beta Q u
    c64 p = {0.0, 0.0}, z = {0.0, 0.0};
#pragma unroll
    for (int i = I0; i < C; ++i) {
      if (live_rows) p = cfma(a[i], u[i], p);
      if (Q) z = cfma(w[i], u[i], z);
    }
    if (live_rows) {
      p = sum8(p);
      p = {beta * p.re, beta * p.im};
      s.v1[r] = p;
      s.part[wv] = sum_rows(cdotr(ur, p));
    } else {
      s.part[wv] = 0.0;
    }
    if (Q) {
      z = sum8(z);
      z = {beta * z.re, beta * z.im};
    }
    __syncthreads();
    if (live_rows) {
      c64 wc[C];
#pragma unroll
      for (int i = I0; i < C; ++i) wc[i] = s.v1[q + 8 * i];
      const double g = 0.5 * beta * wave_parts<C>(s.part);
      const c64 wr = crfms(g, ur, p);
      // A -= u w^H + w u^H, Q -= z u^H; the next column first
#pragma unroll
      for (int i = I0; i < C; ++i) {
        wc[i] = crfms(g, u[i], wc[i]);
        a[i] = cfms_bc(wr, u[i], cfms_bc(ur, wc[i], a[i]));
        if (i == I0) {
          c64* at = q + 8 * I0 == o ? s.v0 + r : s.dump + l;
          *at = csel(r > o, a[I0], c64{0.0, 0.0});
        }
      }
    }
    if (Q) {
#pragma unroll
      for (int i = I0; i < C; ++i) w[i] = cfms_bc(z, u[i], w[i]);
    }
  }
  if constexpr (I0 + 1 < C) block_reflectors<C, I0 + 1, Q>(s, n, a, w, el);
}

// Tridiagonal form of the matrix with entries a (thread (r, q): columns q + 8
// i): its diagonal and complex off-diagonal to the lanes of every wave.
template <int C, bool Q>
__device__ inline __attribute__((always_inline)) void block_tridiag(const blk_ws& s, int n, c64* a, c64* w, c64& el,
                                                                    double& al) {
  const int tid = threadIdx.x, l = tid & 63, r = tid >> 3, q = tid & 7;
  if (tid < 64) {
    s.v0[tid] = {0.0, 0.0};
    s.v1[tid] = {0.0, 0.0};
  }
  __syncthreads();
  if (q == 0) s.v0[r] = csel(r > 0, a[0], c64{0.0, 0.0});
  el = {0.0, 0.0};
  block_reflectors<C, 0, Q>(s, n, a, w, el);
  __syncthreads();
  // v0: column n - 2, whose last entry is e_(n-2)
  if (n > 1 && l == n - 2) el = s.v0[n - 1];
  double* dg = (double*)s.v1;
#pragma unroll
  for (int i = 0; i < C; ++i)
    if (q + 8 * i == r) dg[r] = a[i].re;
  __syncthreads();
  al = l < n ? dg[l] : 0.0;
}

// lambda_min / lambda_max of the Hermitian positive semidefinite matrix with
// entries a (see block_tridiag; scaled as block_eig's), as small_extreme_ratio: the midpoints of
// their brackets, the first wave bisecting one and the second the other.
// Valid in every thread; 0 for a zero matrix.
template <int C>
__device__ inline __attribute__((always_inline)) double block_extreme_ratio(const blk_ws& s, int n, c64* a) {
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
  c64 el;
  double al, glo, ghi, tn, lo, hi;
  block_tridiag<C, false>(s, n, a, a, el, al);
  int ex;
  scale_tridiag(s, n, al, l < n - 1 ? sqrt(cnorm2(el)) : 0.0, &ex, &glo, &ghi, &tn);
  __syncthreads();
  if (wv < 2) {
    bisect_minors(s, n, wv == 0 ? 1 : n, glo, ghi, tn, &lo, &hi);
    if (n == 1) lo = hi = s.ab[0].x;
    s.part[wv] = 0.5 * (lo + hi);
  }
  __syncthreads();
  const double lmin = fmax(s.part[0], 0.0), lmax = s.part[1];
  return lmax > 0.0 ? lmin / lmax : 0.0;
}

// ---------------------------------------------------------------- the solver
// Called by every thread of a workgroup of C waves, 8 C >= n.  acc.get(i, j):
// G in double-double.  Leaves the unit eigenvector in s.x (zero beyond n), the
// number of refinement steps in *steps and T in s.ab with *ghi its scaled
// Gershgorin bound; want_diag as in small_eig (the second eigenvalue in the first
// wave's *lam1 and mu = x^H G x returned, else NaN).  ge: a power of two near G's largest
// entry (frexp's exponent); the reduction takes G 2^-ge, so that its squares
// and reciprocals stay in range down to the roundings of a G that is singular.
template <int C, class Acc>
__device__ inline __attribute__((always_inline)) dd block_eig(const blk_ws& s, const Acc& acc, int n, bool want_diag,
                                                              double* lam1, int* steps, double* ghi,
                                                              int max_refine, int ge) {
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
  const int r = tid >> 3, q = tid & 7;
  *lam1 = __builtin_nan("");
  *steps = 0;
  c64 w[C];
  c64 el;                  // e_l in lane l
  double al_;              // a_l in lane l
  {
    c64 a[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int c = q + 8 * i;
      a[i] = {0.0, 0.0};
      if (r < n && c < n) {
        const cdd v = acc.get(r, c);
        a[i] = {__builtin_amdgcn_ldexp(v.re.hi, -ge), __builtin_amdgcn_ldexp(v.im.hi, -ge)};
      }
      w[i] = {r == c ? 1.0 : 0.0, 0.0};
    }
    block_tridiag<C, true>(s, n, a, w, el, al_);
  }
  const double bl_ = l < n - 1 ? sqrt(cnorm2(el)) : 0.0;
  int ex;
  double glo, tn;
  scale_tridiag(s, n, al_, bl_, &ex, &glo, ghi, &tn);
  const int gx = ge + ex;      // of T against G's own eigenvalues
  if (n == 1) {
    if (tid < 64) s.x[tid] = {tid == 0 ? 1.0 : 0.0, 0.0};
    __syncthreads();
    return want_diag ? acc.get(0, 0).re : dd{__builtin_nan(""), 0.0};
  }
  // W = Q D (D: the diagonal unitary that makes the tridiagonal real: in lane
  // l the product of the unit factors of e_0 .. e_(l-1)), and the rows of W^H
  {
    const double ir = bl_ > 0.0 ? rcp_h(bl_) : 0.0;
    const c64 f = csel(bl_ > 0.0, c64{el.re * ir, el.im * ir}, c64{1.0, 0.0});
    c64 t = {__shfl_up(f.re, 1), __shfl_up(f.im, 1)};
    if (l == 0 || l >= n) t = {1.0, 0.0};
    t = scan_mul_step<0x111, 0xf>(t);
    t = scan_mul_step<0x112, 0xf>(t);
    t = scan_mul_step<0x114, 0xf>(t);
    t = scan_mul_step<0x118, 0xf>(t);
    t = scan_mul_step<0x142, 0xa>(t);
    t = scan_mul_step<0x143, 0xc>(t);
    s.v0[l] = t;     // every wave stores the same values
  }
  __syncthreads();
  const int ldw = n + 1;
  c64 wt[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = q + 8 * i;
    w[i] = cfma(w[i], s.v0[c], c64{0.0, 0.0});
    if (r >= n || c >= n) w[i] = {0.0, 0.0};
    c64* at = (r < n && c < n) ? s.M + (size_t)r * ldw + c : s.dump + l;
    *at = w[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = q + 8 * i;
    const bool in = r < n && c < n;
    const c64 v = s.M[in ? (size_t)c * ldw + r : 0];
    wt[i] = csel(in, conj(v), c64{0.0, 0.0});
  }
  __syncthreads();   // X takes the place of W
  // The first wave alone (the others wait at the barrier after X, where they
  // leave the SIMDs to other workgroups):
  double* X = (double*)s.M;
  if (__builtin_amdgcn_readfirstlane(wv) == 0) {
    // 2. the smallest eigenvalue (and with diagnostics the second)
    double lo0, hi0;
    bisect_minors<true>(s, n, 1, glo, *ghi, tn, &lo0, &hi0);
    if (want_diag) {
      double lo1, hi1;
      bisect_minors(s, n, 2, glo, *ghi, tn, &lo1, &hi1);
      *lam1 = __builtin_amdgcn_ldexp(0.5 * (lo1 + hi1), gx);
    }
    // 3. sigma, the LDL^T factors of T - sigma I (every lane in step, entries
    // eight at a time; lane k keeps pivot k)
    const double sigma = lo0 - 16.0 * n * 2.2e-16 * tn;
    const double pivmin = 1e-300 + 2.2e-16 * 2.2e-16 * tn;
    double2 f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] = s.ab[u];
    double d = 1.0, id = 0.0, idl = 0.0;
#pragma unroll 1
    for (int k0 = 0; k0 < n; k0 += 8) {
      double2 g[8];
      const double2* nx = s.ab + min(k0 + 8, 64);
#pragma unroll
      for (int u = 0; u < 8; ++u) g[u] = nx[u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        d = fma(-f[u].y, id, f[u].x - sigma);      // t_k - b_(k-1)^2 / d_(k-1)
        d = d > pivmin ? d : pivmin;
        id = rcp_h(d);
        idl = l == k0 + u ? id : idl;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) f[u] = g[u];
    }
    const double bs = __builtin_amdgcn_ldexp(bl_, -ex);
    if (l >= n) idl = 0.0;
    s.fac[l] = double2{idl, l + 1 < n ? bs * idl : 0.0};
    wave_sync();
    // X = (T - sigma I)^{-1}, column c in lane c: L y = e_c, then L^T z =
    // D^{-1} y, eight rows at a time (rows past n are zero)
    const int nb = (n + 7) >> 3;
    double* col = l < n ? X + l : (double*)(s.dump + l);
    const int ldc = l < n ? ldw : 0;
    double v = 0.0, lp = 0.0;
#pragma unroll 1
    for (int k0 = 0; k0 < 8 * nb; k0 += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) f[u] = s.fac[k0 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        v = fma(-lp, v, k0 + u == l ? 1.0 : 0.0);
        lp = f[u].y;
        col[(k0 + u) * ldc] = v * f[u].x;
      }
    }
    double z = 0.0;
#pragma unroll 1
    for (int k0 = 8 * nb - 8; k0 >= 0; k0 -= 8) {
      double y[8], lk[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        lk[u] = s.fac[k0 + u].y;
        y[u] = col[(k0 + u) * ldc];
      }
#pragma unroll
      for (int u = 7; u >= 0; --u) {
        z = fma(-lk[u], z, y[u]);
        col[(k0 + u) * ldc] = z;
      }
    }
  }
  __syncthreads();
  double xr[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = q + 8 * i;
    const bool in = r < n && c < n;
    const double v = X[in ? (size_t)r * ldw + c : 0];
    xr[i] = in ? v : 0.0;
  }
  // products with the register matrices: the vector from LDS, entry r in
  // every lane of row r
  auto mat_vec = [&](const c64* m, const c64* v) __attribute__((always_inline)) {
    c64 t = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < C; ++i) t = cfma(m[i], v[q + 8 * i], t);
    return sum8(t);
  };
  // inverse iteration on T from a fixed, generic start vector (real), then x = W y
  {
    double* yb[2] = {(double*)s.v0, (double*)s.v1};
    yb[0][r] = 1.0 + 0.6180339887 * (double)((r * 7) % 11);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SMALL_INVIT; ++it) {
      const double* y = yb[it & 1];
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < C; ++i) t = fma(xr[i], y[q + 8 * i], t);
      yb[~it & 1][r] = sum8(t);
      __syncthreads();
    }
    const double* y = yb[SMALL_INVIT & 1];
    const double yl = y[l];
    const double iy = gx >= BLK_MIN_EXP && gx <= BLK_MAX_EXP ? 1.0 / sqrt(wsum(l < n ? yl * yl : 0.0))
                                                             : __builtin_nan("");
    c64 t = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const double yc = y[q + 8 * i] * iy;
      t = {fma(w[i].re, yc, t.re), fma(w[i].im, yc, t.im)};
    }
    t = sum8(t);
    if (tid >= 8 * C && tid < 64) s.x[tid] = {0.0, 0.0};
    s.x[r] = t;
  }
  __syncthreads();
  // 4. Newton refinement
  dd mu = {__builtin_nan(""), 0.0};
  double dprev = 0.0;
  int it = 0;
  bool done = false;
  for (;; ++it) {
    const c64 x = s.x[r];
    // y = G x in double-double: C entries per thread, the eight partial sums
    // of a row joined by error-free additions
    dot2 ar, ai;
    ar.init();
    ai.init();
    const int rc = min(r, n - 1);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int c = q + 8 * i;
      const cdd gv = acc.get(rc, min(c, n - 1));
      const c64 xj = s.x[c];          // zero for c >= n
      ar.add_prod(gv.re.hi, xj.re); ar.add(gv.re.lo * xj.re);
      ar.add_prod(-gv.im.hi, xj.im); ar.add(-gv.im.lo * xj.im);
      ai.add_prod(gv.re.hi, xj.im); ai.add(gv.re.lo * xj.im);
      ai.add_prod(gv.im.hi, xj.re); ai.add(gv.im.lo * xj.re);
    }
    auto join = [](dot2& d, double ph, double pl) __attribute__((always_inline)) {
      double h, e;
      two_sum(d.p, ph, h, e);
      d.p = h;
      d.s = d.s + (pl + e);
    };
    join(ar, dpp_z<0xB1>(ar.p), dpp_z<0xB1>(ar.s));
    join(ai, dpp_z<0xB1>(ai.p), dpp_z<0xB1>(ai.s));
    join(ar, dpp_z<0x4E>(ar.p), dpp_z<0x4E>(ar.s));
    join(ai, dpp_z<0x4E>(ai.p), dpp_z<0x4E>(ai.s));
    join(ar, dpp_z<0x141>(ar.p), dpp_z<0x141>(ar.s));
    join(ai, dpp_z<0x141>(ai.p), dpp_z<0x141>(ai.s));
    const dd yre = ar.result(), yim = ai.result();
    // mu = x^H y and the residual r = y - mu x in double-double, r then rounded
    dot2 t;
    t.init();
    t.add_prod(x.re, yre.hi); t.add(x.re * yre.lo);
    t.add_prod(x.im, yim.hi); t.add(x.im * yim.lo);
    mu = block_rows_sum<C>(s, 0, 5, t.result());
    if (done || it == max_refine) break;
    auto resid = [&](dd y, double xv) __attribute__((always_inline)) {
      dot2 q;
      q.init();
      q.add_dd(y); q.add_prod(-mu.hi, xv); q.add(-mu.lo * xv);
      return __builtin_amdgcn_ldexp(dd_val(q.result()), -gx);
    };
    const c64 rr = csel(r < n, c64{resid(yre, x.re), resid(yim, x.im)}, c64{0.0, 0.0});
    // correction c = W (T - sigma I)^{-1} W^H r
    s.v0[r] = rr;
    __syncthreads();
    s.v1[r] = mat_vec(wt, s.v0);
    __syncthreads();
    c64 t2 = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const c64 v = s.v1[q + 8 * i];
      t2 = {fma(xr[i], v.re, t2.re), fma(xr[i], v.im, t2.im)};
    }
    s.v0[r] = sum8(t2);
    __syncthreads();
    const c64 cl = mat_vec(w, s.v0);
    // the change of direction: with c = alpha x + c_perp, x - c turns by
    // |c_perp| / |1 - alpha|
    const c64 xn = {x.re - cl.re, x.im - cl.im};
    double* pa = s.part + 1 * BLK_MAX_WAVES;
    pa[wv] = sum_rows(cdotr(x, cl));
    pa[BLK_MAX_WAVES + wv] = sum_rows(fma(x.re, cl.im, -(x.im * cl.re)));
    pa[2 * BLK_MAX_WAVES + wv] = sum_rows(cnorm2(xn));
    __syncthreads();
    const c64 al = {wave_parts<C>(pa), wave_parts<C>(pa + BLK_MAX_WAVES)};
    const double inr = 1.0 / sqrt(wave_parts<C>(pa + 2 * BLK_MAX_WAVES));
    const c64 cp = {fma(-x.re, al.re, fma(x.im, al.im, cl.re)), fma(-x.re, al.im, fma(-x.im, al.re, cl.im))};
    s.x[r] = {xn.re * inr, xn.im * inr};
    // (barrier inside: the new x is visible after it)
    const double dn = sqrt(block_rows_sum<C>(s, 4, cnorm2(cp))) /
                      sqrt(fma(1.0 - al.re, 1.0 - al.re, al.im * al.im));
    // converged when the change of direction, or the next one predicted from
    // the linear rate dn / dprev of the last two, is below 4e-15
    done = !(dn > 4e-15) || (dprev > 0.0 && dn * dn <= 4e-15 * dprev);
    done = __builtin_amdgcn_readfirstlane(done);
    dprev = dn;
    if (done && !want_diag) {
      ++it;
      mu = {__builtin_nan(""), 0.0};
      break;
    }
  }
  *steps = it;
  return mu;
}

}  // namespace cbp
