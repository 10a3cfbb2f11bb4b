// The CBP encoder (Sec. 3, blur kernel selection; Sec. 4 eq. 1 without the
// sensor noise) and the multi-level 8-bit streams (Sec. 3, multi-level
// security).
//
// k_draw_first, k_draw_probe, k_draw_again: draw each frame's kernel pair from
//   the counter-based generator Philox4x64-10 (Salmon, Moraes, Dror and Shaw,
//   SC 2011) -- entry e of kernel s, attempt a, is word e mod 4 of
//   Philox(counter (e / 4, s, a, 0), key (seed, frame)), u = ((w >> 11) + 1/2)
//   2^-53, normalised to sum 1 in entry order -- and redraws (a + 1) while at
//   some sample w_j of either evaluation order the Sylvester system of the two
//   kernel slices, [C_{k2-1}(p) | -C_{k1-1}(q)], has lambda_min / lambda_max
//   of its Gram below 1e-12 (the slices nearly share a root, so the pair is
//   not safely coprime).  Nearly every pair passes at its first draw, so that
//   draw's 2S solves run as one workgroup each; only the frames that failed one
//   go on, one wave per frame.
// k_blur: B_s = L (x) K_s, full linear convolution of every channel with one
//   of the kernels, register-tiled from LDS tiles of the latent.
// k_quantize / k_dequantize: the 8-bit stream of a level without the b
//   least significant bits, q = clamp(rint(255 B), 0, 255) & (255 << b), and
//   the receiver's q / 255.
#include <algorithm>

#include <type_traits>

#include "eigsmall.h"
#include "internal.h"

namespace cbp {

namespace {

constexpr double kSylvMin = 1e-12;
constexpr int kMaxAttempts = 64;

// ---------------------------------------------------------------- Philox4x64-10
struct u64x4 {
  unsigned long long v[4];
};

__device__ inline u64x4 philox4x64(u64x4 c, unsigned long long k0, unsigned long long k1) {
  const unsigned long long M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const unsigned long long W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const unsigned long long hi0 = __umul64hi(M0, c.v[0]), lo0 = M0 * c.v[0];
    const unsigned long long hi1 = __umul64hi(M1, c.v[2]), lo1 = M1 * c.v[2];
    u64x4 o;
    o.v[0] = hi1 ^ c.v[1] ^ k0;
    o.v[1] = lo1;
    o.v[2] = hi0 ^ c.v[3] ^ k1;
    o.v[3] = lo0;
    c = o;
  }
  return c;
}

// u_e of entry e of kernel `stream` (unnormalised, in (0, 1)).
__device__ inline double draw_entry(unsigned long long seed, unsigned long long frame, int stream, int attempt,
                                    int e) {
  u64x4 c;
  c.v[0] = (unsigned long long)(e >> 2);
  c.v[1] = (unsigned long long)stream;
  c.v[2] = (unsigned long long)attempt;
  c.v[3] = 0ull;
  const u64x4 w = philox4x64(c, seed, frame);
  const unsigned long long x = w.v[e & 3];
  return ((double)(x >> 11) + 0.5) * 0x1p-53;
}

// One kernel into K (LDS, k x k) by threads tid of nt: entries in parallel, the
// sum in entry order on thread 0, then the division.  Every thread of the
// workgroup calls it (barriers); !on: a share without a kernel.
__device__ inline void draw_kernel(double* K, int k, unsigned long long seed, unsigned long long frame, int stream,
                                   int attempt, double* sum_slot, int tid, int nt, bool on = true) {
  const int kk = on ? k * k : 0;
  for (int e = tid; e < kk; e += nt) K[e] = draw_entry(seed, frame, stream, attempt, e);
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int e = 0; e < kk; ++e) s += K[e];
    *sum_slot = s;
  }
  __syncthreads();
  const double s = *sum_slot;
  for (int e = tid; e < kk; e += nt) K[e] = K[e] / s;
  __syncthreads();
}

// LDS of a probe: two kernels, two slices, the correlations, a sum slot and
// the reduction workspace of order k1 + k2 - 2.
__host__ __device__ inline size_t draw_lds_bytes(int k1, int k2) {
  const int n = k1 + k2 - 2 > 1 ? k1 + k2 - 2 : 1;
  return (size_t)(k1 * k1 + k2 * k2 + 2) * sizeof(double) + 2 * (size_t)CBP_MAX_K * sizeof(c64) +
         (size_t)(2 * CBP_MAX_N) * sizeof(c64) + small_probe_lds_bytes(n) + 16;
}

struct draw_lds {
  double* K1;
  double* K2;
  double* sum_slot;
  c64* p;
  c64* q;
  c64* rho;   // [rho_pp (k1), rho_qq (k2), rho_pq (k1 + k2 - 1)]
  small_ws w;
};

__device__ inline draw_lds draw_carve(char* base, int k1, int k2) {
  const int n = k1 + k2 - 2;
  draw_lds d;
  d.K1 = (double*)base;
  d.K2 = d.K1 + k1 * k1;
  d.sum_slot = d.K2 + k2 * k2;
  d.p = (c64*)(((size_t)(d.sum_slot + 2) + 15) & ~(size_t)15);
  d.q = d.p + CBP_MAX_K;
  d.rho = d.q + CBP_MAX_K;
  d.w = small_probe_carve((char*)(d.rho + 2 * CBP_MAX_N), n > 1 ? n : 1);
  return d;
}

// The Gram of the Sylvester system of the kernel slices at sample j of a pass
// (pass 0 evaluates along y, a polynomial in x; pass 1 along x) into w.A.
__device__ inline void sylvester_gram(const draw_lds& d, int k1, int k2, int S, int pass, int j) {
  const int l = threadIdx.x, nt = blockDim.x;
  const int n1 = k2 - 1, n2 = k1 - 1, n = n1 + n2;
  if (l < k1 + k2) {
    const bool first = l < k1;
    const int k = first ? k1 : k2, t = first ? l : l - k1;
    const double* K = first ? d.K1 : d.K2;
    c64 acc = {0.0, 0.0};
    for (int r = 0; r < k; ++r) {
      double sn, cs;
      sincospi(-2.0 * (double)((j * r) % S) / (double)S, &sn, &cs);
      const double kv = pass == 0 ? K[r * k + t] : K[t * k + r];
      acc = acc + c64{kv * cs, kv * sn};
    }
    (first ? d.p : d.q)[t] = acc;
  }
  __syncthreads();
  // correlations rho_pp(l) (l < k1), rho_qq(l) (l < k2), rho_pq(l), l in [-(n2 - 1), n1 - 1]
  for (int t = l; t < k1 + k2 + n - 1; t += nt) {
    const c64* x;
    const c64* y;
    int lag, lx, ly;
    if (t < k1) { x = d.p; y = d.p; lag = t; lx = k1; ly = k1; }
    else if (t < k1 + k2) { x = d.q; y = d.q; lag = t - k1; lx = k2; ly = k2; }
    else { x = d.p; y = d.q; lag = t - (k1 + k2) - (n2 - 1); lx = k1; ly = k2; }
    c64 acc = {0.0, 0.0};
    for (int s0 = max(0, -lag); s0 < lx && s0 + lag < ly; ++s0) acc = acc + cmulc(x[s0], y[s0 + lag]);
    d.rho[t] = acc;
  }
  __syncthreads();
  for (int e = l; e < n * n; e += nt) {
    const int r = e / n, c = e - r * n;
    const bool ra = r < n1, ca = c < n1;
    const int pr = ra ? r : r - n1, pc = ca ? c : c - n1;
    c64 v;
    if (ra == ca) {
      // rho_pp has k1 lags, rho_qq k2; longer lags are zero
      const int lag = pr - pc, al = lag < 0 ? -lag : lag;
      v = al < (ra ? k1 : k2) ? d.rho[(ra ? 0 : k1) + al] : c64{0.0, 0.0};
      if (lag < 0) v.im = -v.im;
    } else {
      const int cross = k1 + k2 + (n2 - 1);
      v = ra ? d.rho[cross + pr - pc] : conj(d.rho[cross + pc - pr]);
      v = c64{-v.re, -v.im};
    }
    d.w.A[e] = v;
  }
  __syncthreads();
}

constexpr int DRAW_FAILED = 0x40000000;   // in attempts[f] between the launches

// Attempt 0 of every frame: kernels 2 f + stream - 1 < n2, W waves each, 4 / W to
// a workgroup, bound by the ordered sum of their entries.  W = 1 serves kernels
// of at most 64 entries: a million pairs of 2x2 and 1x1 are bound by the number
// of workgroups.
constexpr int kDrawWave = 8;   // largest kernel of one wave
template <int W>
__global__ __launch_bounds__(256) void k_draw_first(unsigned long long seed, long long frame0, int n2, int k1, int k2,
                                                    double* K1s, double* K2s, int* attempts, double* min_ratio) {
  constexpr int PER = 4 / W, NT = 64 * W;
  __shared__ double K[PER][W == 1 ? kDrawWave * kDrawWave : CBP_MAX_K * CBP_MAX_K];
  __shared__ double sum_slot[PER];
  const int h = (int)threadIdx.x / NT, tid = (int)threadIdx.x - h * NT;
  const int i = (int)blockIdx.x * PER + h, f = i >> 1, s = 1 + (i & 1);
  const bool on = i < n2;
  const int k = s == 1 ? k1 : k2;
  draw_kernel(K[h], k, seed, (unsigned long long)(frame0 + f), s, 0, &sum_slot[h], tid, NT, on);
  if (!on) return;
  double* out = s == 1 ? K1s + (size_t)f * k1 * k1 : K2s + (size_t)f * k2 * k2;
  for (int e = tid; e < k * k; e += NT) out[e] = K[h][e];
  if (s == 1 && tid == 0) {
    attempts[f] = 0;
    if (min_ratio) min_ratio[f] = 1.0;
  }
}

// One workgroup of two waves per (frame, pass, sample): the first reduces the
// Gram to tridiagonal form, then each bisects one extreme eigenvalue.  The
// frame's smallest ratio collects in min_ratio (non-negative doubles order as
// their bits), a ratio at or below the limit marks attempts[f].  Bound by the
// one-wave reduction's chain (its operation order is the ratio's last digits);
// 102 us for 30 pairs of 15x15 / 17x17 kernels, whose 1020 systems took one
// wave per frame 3.4 ms.
__global__ __launch_bounds__(128) void k_draw_probe(int k1, int k2, int S, const double* K1s, const double* K2s,
                                                    int* attempts, double* min_ratio) {
  extern __shared__ __attribute__((aligned(16))) char sm_draw[];
  const int f = blockIdx.x / (2 * S), t = blockIdx.x - f * 2 * S, pass = t / S, j = t - pass * S;
  const int n = k1 + k2 - 2, tid = threadIdx.x;
  draw_lds d = draw_carve(sm_draw, k1, k2);
  for (int e = tid; e < k1 * k1; e += 128) d.K1[e] = K1s[(size_t)f * k1 * k1 + e];
  for (int e = tid; e < k2 * k2; e += 128) d.K2[e] = K2s[(size_t)f * k2 * k2 + e];
  __syncthreads();
  sylvester_gram(d, k1, k2, S, pass, j);
  if (tid < 64) small_tridiag(d.w, n);
  __syncthreads();
  double lo, hi, tn;
  small_bisect(d.w, n, tid < 64 ? 1 : n, &lo, &hi, &tn);
  if ((tid & 63) == 0) d.sum_slot[tid >> 6] = 0.5 * (lo + hi);
  __syncthreads();
  if (tid == 0) {
    const double lmin = fmax(d.sum_slot[0], 0.0), lmax = d.sum_slot[1];
    const double r = lmax > 0.0 ? lmin / lmax : 0.0;
    if (r <= kSylvMin) atomicOr(&attempts[f], DRAW_FAILED);
    if (min_ratio && r < 1.0) atomicMin((unsigned long long*)&min_ratio[f], (unsigned long long)__double_as_longlong(r));
  }
}

// Attempts 1, 2, ... of the frames whose first pair failed, one wave each; a
// workgroup looks `per` <= 64 frames over.
__global__ __launch_bounds__(SMALL_NT) void k_draw_again(unsigned long long seed, long long frame0, int k1, int k2,
                                                          int S, double* K1s, double* K2s, int* attempts,
                                                          double* min_ratio, int nframes, int per) {
  extern __shared__ __attribute__((aligned(16))) char sm_draw[];
  const int l = threadIdx.x, f0 = (int)blockIdx.x * per;
  const bool mine = l < per && f0 + l < nframes;
  unsigned long long failed = __builtin_amdgcn_ballot_w64(mine && (attempts[mine ? f0 + l : f0] & DRAW_FAILED));
  for (; failed; failed &= failed - 1) {
    const int f = f0 + __builtin_ctzll(failed);
    const unsigned long long frame = (unsigned long long)(frame0 + f);
    draw_lds d = draw_carve(sm_draw, k1, k2);
    const int n = k1 + k2 - 2;
    int found = -1;
    double worst = 1.0;
    for (int a = 1; a < kMaxAttempts && found < 0; ++a) {
      draw_kernel(d.K1, k1, seed, frame, 1, a, d.sum_slot, l, SMALL_NT);
      draw_kernel(d.K2, k2, seed, frame, 2, a, d.sum_slot, l, SMALL_NT);
      worst = 1.0;
      for (int pass = 0; pass < 2; ++pass)
        for (int j = 0; j < S; ++j) {
          sylvester_gram(d, k1, k2, S, pass, j);
          const double r = small_extreme_ratio(d.w, n);
          worst = fmin(worst, r);
          __syncthreads();
        }
      if (worst > kSylvMin) found = a;
    }
    for (int e = l; e < k1 * k1; e += SMALL_NT) K1s[(size_t)f * k1 * k1 + e] = d.K1[e];
    for (int e = l; e < k2 * k2; e += SMALL_NT) K2s[(size_t)f * k2 * k2 + e] = d.K2[e];
    if (l == 0) {
      attempts[f] = found;
      if (min_ratio) min_ratio[f] = worst;
    }
    __syncthreads();   // the next frame's draw fills the same LDS
  }
}

// ---------------------------------------------------------------- blur
// B_s[y][x] = sum_{a,b} L[y-a][x-b] K_s[a][b].  A workgroup of 256 threads
// makes a 64 x 64 tile of one stream's channel from the latent's tile and
// halo in LDS; a thread makes 4 rows x 4 adjacent columns.  For each kernel
// row a it holds the row's K taps in registers (one broadcast read per four)
// and, per output row, the K + 3 latent values its four columns need (16-byte
// reads), so an LDS read serves 4 K FMAs / ((K + 3) / 4) -- about 14 of them --
// and the kernel is bound by the vector FP32 FMAs (78 TFLOP/s without packed
// instructions).  K is a template argument: the taps and the window are
// registers.  1080p RGB, 15x15 and 17x17: 642 us (one tap at a time, 10
// TFLOP/s) -> 105 us (61).
constexpr int kTX = 64, kTY = 64, kBR = 4;

template <typename T>
struct blur_args {
  const T* L;
  int64_t lp, lcs;
  int m, n, nch;
  const double* K;
  T* B;
  int64_t bp, bcs;
  int k, ntx, nty;
};

// Row stride of the LDS tile (elements): the width rounded up to 16 bytes.
template <typename T, int K>
constexpr int blur_ld() { return (kTX + K - 1 + 3) & ~3; }

// LDS of a tile: the latent's rows and the taps (padded to whole reads).
template <typename T, int K>
constexpr int blur_lds() { return ((kTY + K - 1) * blur_ld<T, K>() + K * ((K + 3) & ~3)) * (int)sizeof(T); }

template <typename T, int K>
__device__ inline void blur_tile(const blur_args<T>& g, int item, char* sm) {
  constexpr int LD = blur_ld<T, K>(), TH = kTY + K - 1, TW = kTX + K - 1, KP = (K + 3) & ~3;
  constexpr int V = 16 / (int)sizeof(T);                  // elements per 16-byte read
  constexpr int NV = (K + 3 + V - 1) / V;                 // reads of a window of K + 3
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  T* tile = (T*)sm;
  T* Ks = tile + TH * LD;
  const int tid = threadIdx.x;
  const int tx0 = item % g.ntx, rest = item / g.ntx;
  const int ty0 = rest % g.nty, ch = rest / g.nty;
  const int y0 = ty0 * kTY, x0 = tx0 * kTX;
  // taps of kernel row a in the order of the window: Ks[a][t] = K[a][K - 1 - t]
  for (int e = tid; e < K * KP; e += 256) {
    const int a = e / KP, t = e - a * KP;
    Ks[e] = t < K ? (T)g.K[a * K + K - 1 - t] : T(0);
  }
  const T* Lc = g.L + (int64_t)ch * g.lcs;
  // the tile, four rows at a time (a wave per row), zero outside the latent
  {
    const int c = tid & 63, x = x0 - (K - 1) + c;
    const bool in0 = x >= 0 && x < g.n, in1 = c + 64 < TW && x + 64 < g.n;   // x + 64 >= 0
#pragma unroll 4
    for (int i = tid >> 6; i < TH; i += 4) {
      const int y = y0 - (K - 1) + i;
      const bool iny = y >= 0 && y < g.m;
      const T* row = Lc + (int64_t)y * g.lp + x;
      const T v0 = iny && in0 ? row[0] : T(0), v1 = iny && in1 ? row[64] : T(0);
      tile[i * LD + c] = v0;
      if (c + 64 < LD) tile[i * LD + c + 64] = v1;
    }
  }
  __syncthreads();
  const int tx = (tid & 15) * 4, ty = (tid >> 4) * kBR;
  T acc[kBR][4];
#pragma unroll
  for (int r = 0; r < kBR; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = T(0);
#pragma unroll 1
  for (int a = 0; a < K; ++a) {
    T k[KP];
#pragma unroll
    for (int v = 0; v < KP / V; ++v) {
      const vec q = *(const vec*)(Ks + a * KP + v * V);
#pragma unroll
      for (int u = 0; u < V; ++u) k[v * V + u] = q[u];
    }
#pragma unroll
    for (int r = 0; r < kBR; ++r) {
      const T* row = tile + (ty + r + K - 1 - a) * LD + tx;
      T w[NV * V];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const vec q = *(const vec*)(row + v * V);
#pragma unroll
        for (int u = 0; u < V; ++u) w[v * V + u] = q[u];
      }
#pragma unroll
      for (int t = 0; t < K; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] += k[t] * w[c + t];
    }
  }
  const int H = g.m + K - 1, W = g.n + K - 1;
  T* Bc = g.B + (int64_t)ch * g.bcs;
#pragma unroll
  for (int r = 0; r < kBR; ++r) {
    const int y = y0 + ty + r;
    if (y < H)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (x0 + tx + c < W) Bc[(int64_t)y * g.bp + x0 + tx + c] = acc[r][c];
  }
}

template <typename T, int K>
__global__ __launch_bounds__(256) void k_blur(blur_args<T> g) {
  __shared__ __attribute__((aligned(16))) char sm[blur_lds<T, K>()];
  blur_tile<T, K>(g, (int)blockIdx.x, sm);
}

// Both streams in one launch, for kernels of at most kBlurPair: their tiles
// are short, and on small frames the second launch costs more than the
// tiles (64x64, 3x3 / 5x5: 14.1 us in two launches, 11.7 in one), while the
// registers of the largest instance still leave three waves per SIMD.  Larger
// ones are bound by their tiles also on small frames: calls of 16x16 to 240x320
// FP32 with 8 / 8, 8 / 9, 9 / 11, 15 / 17, 21 / 19 taps take 15.5, 18, 18 to 21, 29
// to 33, 39 to 43 us (20, 24, 34, 72, 107 one tap at a time in one launch).
constexpr int kBlurPair = 8;

template <typename T, int K>
__device__ inline __attribute__((always_inline)) void blur_any(const blur_args<T>& g, int item, char* sm) {
  if (g.k == K) blur_tile<T, K>(g, item, sm);
  else if constexpr (K > 1) blur_any<T, K - 1>(g, item, sm);
}

template <typename T>
__global__ __launch_bounds__(256) void k_blur_pair(blur_args<T> g1, blur_args<T> g2) {
  __shared__ __attribute__((aligned(16))) char sm[blur_lds<T, kBlurPair>()];
  const int n1 = g1.ntx * g1.nty * g1.nch, b = (int)blockIdx.x;
  if (b < n1) blur_any<T, kBlurPair>(g1, b, sm);
  else blur_any<T, kBlurPair>(g2, b - n1, sm);
}

// ---------------------------------------------------------------- 8-bit streams
// Both are copies with a conversion, bound by HBM.  Dense images (no gap
// between rows and channels, 16-byte aligned bases) are one run of elements:
// a workgroup converts 4096 of them, a thread in groups of 16 bytes of pixels
// with neighbouring lanes on neighbouring groups, without an index division.  1080p RGB FP32: quantise 18.5 us and dequantise 19.7
// (one element per thread and step, two 64-bit divisions each) -> 7.8 and 7.8 (4 TB/s).
// Other images go by rows (convert_rows).
template <typename T>
__device__ inline unsigned int quantize_one(T x, unsigned int mask) {
  const T v = rint(x * T(255));
  const T cl = v < T(0) ? T(0) : (v > T(255) ? T(255) : v);
  return (unsigned int)cl & mask;
}

// A group of V = 16 / sizeof(T) elements as bytes.
template <typename T>
using level_bytes = typename std::conditional<sizeof(T) == 4, unsigned int, unsigned short>::type;

template <typename T>
__global__ __launch_bounds__(256) void k_quantize_dense(const T* src, unsigned char* dst, int64_t total,
                                                        unsigned int mask) {
  constexpr int V = 16 / (int)sizeof(T), NI = 16 / V;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  const int64_t e0 = (int64_t)blockIdx.x * 4096 + threadIdx.x * V;   // group i: e0 + 256 V i
  if ((int64_t)blockIdx.x * 4096 + 4096 <= total) {
    vec v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) v[i] = *(const vec*)(src + e0 + i * 256 * V);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      unsigned int w = 0;
#pragma unroll
      for (int j = 0; j < V; ++j) w |= quantize_one<T>(v[i][j], mask) << (8 * j);
      *(level_bytes<T>*)(dst + e0 + i * 256 * V) = (level_bytes<T>)w;
    }
  } else {
    for (int64_t e = (int64_t)blockIdx.x * 4096 + threadIdx.x; e < total; e += 256)
      dst[e] = (unsigned char)quantize_one<T>(src[e], mask);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_dequantize_dense(const unsigned char* src, T* dst, int64_t total) {
  constexpr int V = 16 / (int)sizeof(T), NI = 16 / V;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  const int64_t e0 = (int64_t)blockIdx.x * 4096 + threadIdx.x * V;
  if ((int64_t)blockIdx.x * 4096 + 4096 <= total) {
    level_bytes<T> w[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) w[i] = *(const level_bytes<T>*)(src + e0 + i * 256 * V);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      vec v;
#pragma unroll
      for (int j = 0; j < V; ++j) v[j] = (T)(((unsigned int)w[i] >> (8 * j)) & 0xFFu) / T(255);
      *(vec*)(dst + e0 + i * 256 * V) = v;
    }
  } else {
    for (int64_t e = (int64_t)blockIdx.x * 4096 + threadIdx.x; e < total; e += 256) dst[e] = (T)src[e] / T(255);
  }
}

// Pitched images: channels blockIdx.z + gridDim.z i.  A row has 2^lx lanes (at
// most 256) and a thread takes 2^lc columns of it, 256 apart (more than 1024
// columns: blockIdx.x), in 4 / 2^lc rows, so narrow rows share a workgroup: one
// row a workgroup would leave most of its lanes idle.  FP32 quantise of a
// million rows of 8 in a pitched image: 22 us element by element with two 64-bit
// divisions each, 508 a row at a time, 13 so; 100000 rows of 300: 71, 61, 49.
struct row_split {
  int lx, lc;
};

template <typename S, typename D, typename F>
__device__ inline void convert_rows(const S* src, int64_t sp, int64_t scs, D* dst, int64_t dp, int64_t dcs, int H, int W,
                                    int nch, row_split rs, F one) {
  const int tid = threadIdx.x;
  const int rows = 256 >> rs.lx, per = rows * (4 >> rs.lc);   // rows of the lanes, of the workgroup
  const int x0 = (int)blockIdx.x * 1024 + (tid & ((1 << rs.lx) - 1));
  for (int c = blockIdx.z; c < nch; c += gridDim.z) {
    const S* s = src + (int64_t)c * scs;
    D* d = dst + (int64_t)c * dcs;
    for (int64_t y0 = (int64_t)blockIdx.y * per + (tid >> rs.lx); y0 < H; y0 += (int64_t)gridDim.y * per) {
      S v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t y = y0 + (i >> rs.lc) * rows;
        const int x = x0 + (i & ((1 << rs.lc) - 1)) * 256;
        if (x < W && y < H) v[i] = s[y * sp + x];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t y = y0 + (i >> rs.lc) * rows;
        const int x = x0 + (i & ((1 << rs.lc) - 1)) * 256;
        if (x < W && y < H) d[y * dp + x] = one(v[i]);
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_quantize(const T* src, int64_t sp, int64_t scs, unsigned char* dst, int64_t dp,
                                                  int64_t dcs, int H, int W, int nch, row_split rs, unsigned int mask) {
  convert_rows(src, sp, scs, dst, dp, dcs, H, W, nch, rs,
               [&](T x) { return (unsigned char)quantize_one<T>(x, mask); });
}

template <typename T>
__global__ __launch_bounds__(256) void k_dequantize(const unsigned char* src, int64_t sp, int64_t scs, T* dst,
                                                    int64_t dp, int64_t dcs, int H, int W, int nch, row_split rs) {
  convert_rows(src, sp, scs, dst, dp, dcs, H, W, nch, rs, [](unsigned char q) { return (T)q / T(255); });
}

}  // namespace

// Frames of one turn of the launches: a launch holds fewer than 2^32 threads,
// and a frame has 2S probes of 128 and two first draws of 256.  Half of that.
constexpr int draw_slice(int S) { return (1 << 23) / std::max(S, 2); }

hipError_t launch_draw_pairs(unsigned long long seed, long long frame0, int nframes, int k1, int k2, int S,
                             double* K1s, double* K2s, int* attempts, double* min_ratio, hipStream_t st) {
  const size_t lds = draw_lds_bytes(k1, k2);
  for (int f = 0; f < nframes;) {
    const int n = std::min(nframes - f, draw_slice(S));
    double* K1 = K1s + (size_t)f * k1 * k1;
    double* K2 = K2s + (size_t)f * k2 * k2;
    int* at = attempts + f;
    double* mr = min_ratio ? min_ratio + f : nullptr;
    if (std::max(k1, k2) <= kDrawWave)
      hipLaunchKernelGGL(k_draw_first<1>, dim3((n + 1) / 2), dim3(256), 0, st, seed, frame0 + f, 2 * n, k1, k2, K1, K2,
                         at, mr);
    else
      hipLaunchKernelGGL(k_draw_first<4>, dim3(2 * n), dim3(256), 0, st, seed, frame0 + f, 2 * n, k1, k2, K1, K2, at, mr);
    if (k1 + k2 > 2) {   // two 1 x 1 kernels have no Sylvester system
      hipLaunchKernelGGL(k_draw_probe, dim3(n * 2 * S), dim3(128), lds, st, k1, k2, S, K1, K2, at, mr);
      // (65536 frames and more: workgroups that only look cost more than the looking)
      const int per = (n + 65535) / 65536;
      hipLaunchKernelGGL(k_draw_again, dim3((n + per - 1) / per), dim3(SMALL_NT), lds, st, seed, frame0 + f, k1, k2, S,
                         K1, K2, at, mr, n, per);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    f += n;
  }
  return hipSuccess;
}

void set_encoder_attrs() {
  for (const void* f : {(const void*)k_draw_probe, (const void*)k_draw_again})
    hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)draw_lds_bytes(CBP_MAX_K, CBP_MAX_K));
}

namespace {

template <typename T, int K>
void blur_stream(int k, const blur_args<T>& g, hipStream_t st) {
  if (k == K) hipLaunchKernelGGL((k_blur<T, K>), dim3(g.ntx * g.nty * g.nch), dim3(256), 0, st, g);
  else if constexpr (K > 1) blur_stream<T, K - 1>(k, g, st);
}

}  // namespace

template <typename T>
hipError_t launch_blur(const T* L, int64_t lp, int64_t lcs, int m, int n, int nch, const double* K1, int k1,
                       const double* K2, int k2, T* B1, int64_t p1, int64_t cs1, T* B2, int64_t p2, int64_t cs2,
                       hipStream_t st) {
  blur_args<T> g[2];
  for (int s = 0; s < 2; ++s) {
    const int k = s ? k2 : k1;
    g[s] = {L, lp, lcs, m, n, nch, s ? K2 : K1, s ? B2 : B1, s ? p2 : p1, s ? cs2 : cs1, k,
            (n + k - 1 + kTX - 1) / kTX, (m + k - 1 + kTY - 1) / kTY};
  }
  if (std::max(k1, k2) <= kBlurPair) {
    const int grid = (g[0].ntx * g[0].nty + g[1].ntx * g[1].nty) * nch;
    hipLaunchKernelGGL(k_blur_pair<T>, dim3(grid), dim3(256), 0, st, g[0], g[1]);
  } else {
    for (int s = 0; s < 2; ++s) blur_stream<T, CBP_MAX_K>(g[s].k, g[s], st);
  }
  return hipGetLastError();
}

namespace {

// No gap between rows and channels (a one-channel image's stride is unused).
bool dense(int64_t pitch, int64_t cs, int H, int W, int nch) {
  return pitch == W && (nch == 1 || cs == (int64_t)H * W);
}
bool aligned16(const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; }
row_split split_rows(int W) {
  row_split r = {0, W > 512 ? 2 : W > 256 ? 1 : 0};
  while (r.lx < 8 && 1 << r.lx < W) ++r.lx;
  return r;
}
dim3 row_grid(int H, int W, int nch) {
  const row_split r = split_rows(W);
  const int64_t per = 1024 >> r.lx >> r.lc;
  return dim3((W - 1) / 1024 + 1, (unsigned)std::min<int64_t>((H + per - 1) / per, 65535), std::min(nch, 65535));
}

}  // namespace

template <typename T>
hipError_t launch_quantize(const T* src, int64_t sp, int64_t scs, unsigned char* dst, int64_t dp, int64_t dcs, int H,
                           int W, int nch, int drop, hipStream_t st) {
  const int64_t total = (int64_t)H * W * nch;
  const unsigned int mask = (0xFFu << drop) & 0xFFu;
  if (dense(sp, scs, H, W, nch) && dense(dp, dcs, H, W, nch) && aligned16(src, dst) && total < (int64_t)1 << 40)
    hipLaunchKernelGGL(k_quantize_dense<T>, dim3((unsigned)((total + 4095) / 4096)), dim3(256), 0, st, src, dst, total,
                       mask);
  else
    hipLaunchKernelGGL(k_quantize<T>, row_grid(H, W, nch), dim3(256), 0, st, src, sp, scs, dst, dp, dcs, H, W, nch,
                       split_rows(W), mask);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_dequantize(const unsigned char* src, int64_t sp, int64_t scs, T* dst, int64_t dp, int64_t dcs,
                             int H, int W, int nch, hipStream_t st) {
  const int64_t total = (int64_t)H * W * nch;
  if (dense(sp, scs, H, W, nch) && dense(dp, dcs, H, W, nch) && aligned16(src, dst) && total < (int64_t)1 << 40)
    hipLaunchKernelGGL(k_dequantize_dense<T>, dim3((unsigned)((total + 4095) / 4096)), dim3(256), 0, st, src, dst,
                       total);
  else
    hipLaunchKernelGGL(k_dequantize<T>, row_grid(H, W, nch), dim3(256), 0, st, src, sp, scs, dst, dp, dcs, H, W, nch,
                       split_rows(W));
  return hipGetLastError();
}

template hipError_t launch_blur<float>(const float*, int64_t, int64_t, int, int, int, const double*, int,
                                       const double*, int, float*, int64_t, int64_t, float*, int64_t, int64_t,
                                       hipStream_t);
template hipError_t launch_blur<double>(const double*, int64_t, int64_t, int, int, int, const double*, int,
                                        const double*, int, double*, int64_t, int64_t, double*, int64_t, int64_t,
                                        hipStream_t);
template hipError_t launch_quantize<float>(const float*, int64_t, int64_t, unsigned char*, int64_t, int64_t, int, int,
                                           int, int, hipStream_t);
template hipError_t launch_quantize<double>(const double*, int64_t, int64_t, unsigned char*, int64_t, int64_t, int,
                                            int, int, int, hipStream_t);
template hipError_t launch_dequantize<float>(const unsigned char*, int64_t, int64_t, float*, int64_t, int64_t, int,
                                             int, int, hipStream_t);
template hipError_t launch_dequantize<double>(const unsigned char*, int64_t, int64_t, double*, int64_t, int64_t, int,
                                              int, int, hipStream_t);

}  // namespace cbp
