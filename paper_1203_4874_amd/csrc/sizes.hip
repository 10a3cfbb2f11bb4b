// Blind kernel-size estimation (Sec. 4: the first stage finds the kernel
// degree from the singularity of nested submatrices, after Barnett; Sec. 5
// and Table 1: the "kernel degree estimation" stage).
//
// With the latent size unknown only d = H1 - H2 = k1 - k2 is known.  For a
// trial size k (k1' = k, k2' = k - d) and a unit-circle sample of either
// pass, the 1-D system A(k) = [C_{k-d}(e1) | -C_k(e2)] has a null vector
// exactly when k >= k1 (every solution of b1 u = b2 v is (k2 s, k1 s)), so
// its nullity is max(0, k - k1 + 1).  The test per trial size and sample is
//   s = lambda_min(G(k)) / lambda_max(G(k)),  G(k) = A(k)^H A(k),
// and G(k) is a principal submatrix of the Gram of the largest trial size:
// its entries are the same block-Toeplitz correlations (recover.hip), so one
// set of double-double correlations serves every candidate.
//
// k_size_probe: one workgroup per (candidate, pass, sample): G(k) from the
//   correlations (rounded to FP64), Householder tridiagonalisation on
//   ceil(n / 8) waves (eigblock.h), Sturm multisection for the smallest and the
//   largest eigenvalue.
// k_size_decide: per candidate (one wave each) the median over the 2S samples
//   of log10(max(s, 1e-13)); the estimate is the candidate with the largest
//   drop from the previous candidate's score (0 before the first); a largest
//   drop below 2 decades means no candidate made the systems singular.
#include "eigblock.h"
#include "internal.h"

namespace cbp {

namespace {

constexpr double kSizeFloor = 1e-13;
constexpr double kSizeMinDrop = 2.0;

// Entry (r, c) of the Gram of trial sizes (n1 u taps, n2 v taps) from the
// correlations stored for the largest sizes (K2 u taps, K1 v taps):
// rho11[0..K2), rho22[0..K1), rho12[-(K1-1)..K2-1].
__device__ inline cdd trial_gram(const cdd* rho, int K1, int K2, int n1, int r, int c) {
  const bool ra = r < n1, ca = c < n1;
  const int pr = ra ? r : r - n1, pc = ca ? c : c - n1;   // index inside its block
  cdd v;
  if (ra == ca) {
    const int lag = pr - pc;
    v = rho[(ra ? 0 : K2) + (lag < 0 ? -lag : lag)];
    if (lag < 0) v.im = dd_neg(v.im);
  } else {
    // G12[p][q] = -rho12(p - q) (u index p, v index q); G21 = G12^H
    const int cross = K2 + K1 + (K1 - 1);
    v = ra ? rho[cross + pr - pc] : rho[cross + pc - pr];
    if (!ra) v.im = dd_neg(v.im);
    v = cdd_neg(v);
  }
  return v;
}

// s of one system on its C waves (see block_extreme_ratio).
template <int C>
__device__ inline double probe_ratio(const blk_ws& w, const cdd* rho, int K1, int K2, int n1, int n) {
  const int r = (int)threadIdx.x >> 3, q = threadIdx.x & 7;
  // scaled by the power of two of G's largest entry, one of its diagonal's
  const int ge = __builtin_amdgcn_frexp_exp(fmax(rho[0].re.hi, rho[K2].re.hi));
  c64 a[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = q + 8 * i;
    const bool in = r < n && c < n;
    const cdd g = trial_gram(rho, K1, K2, n1, in ? r : 0, in ? c : 0);
    a[i] = csel(in, c64{__builtin_amdgcn_ldexp(g.re.hi, -ge), __builtin_amdgcn_ldexp(g.im.hi, -ge)}, c64{0.0, 0.0});
  }
  return block_extreme_ratio<C>(w, n, a);
}

// Workgroups of 64 waves_max threads, one per item (candidate, pass, sample)
// of the launch's one frame, the largest candidates (the longest solves)
// first.  The waves beyond ceil(n / 8) of an item end at once (a barrier waits
// for the surviving waves), so small candidates cost what they need.  Bound by
// the reflectors' dependent chain; one wave per item took 256 us for the nine
// odd candidates 9 .. 25 with S = 25, this split 97.
__global__ __launch_bounds__(64 * BLK_MAX_WAVES) void k_size_probe(batch_ref br, size_cands cands, double* ratios) {
  extern __shared__ __attribute__((aligned(16))) char sm_probe[];
  const frame_desc& d = br.descs[0];
  const int S = d.S, K1 = d.k1, K2 = d.k2, NL = 2 * (K1 + K2) - 1;
  const int ci = cands.n - 1 - (int)blockIdx.x / (2 * S), pj = (int)blockIdx.x % (2 * S);
  const int k = cands.k1[ci], n1 = k - cands.d, n = n1 + k;
  const int C = n <= 16 ? 2 : n <= 24 ? 3 : n <= 32 ? 4 : n <= 40 ? 5 : 8;
  if ((int)threadIdx.x >= 64 * C) return;
  cdd* rho = (cdd*)sm_probe;
  for (int t = threadIdx.x; t < NL; t += 64 * C) rho[t] = d.corr[(size_t)pj * NL + t];
  char* fixed = sm_probe + (((size_t)NL * sizeof(cdd) + 15) & ~(size_t)15);
  const blk_ws w = blk_carve(fixed, nullptr);
  __syncthreads();
  double r;
  if (C == 2) r = probe_ratio<2>(w, rho, K1, K2, n1, n);
  else if (C == 3) r = probe_ratio<3>(w, rho, K1, K2, n1, n);
  else if (C == 4) r = probe_ratio<4>(w, rho, K1, K2, n1, n);
  else if (C == 5) r = probe_ratio<5>(w, rho, K1, K2, n1, n);
  else r = probe_ratio<8>(w, rho, K1, K2, n1, n);
  if (threadIdx.x == 0) ratios[(size_t)ci * 2 * S + pj] = r;
}

// Scores (one wave per candidate: a lane's value has as many smaller ones --
// or equal ones in lower lanes -- as its rank), drops and the decision.
// ratios [ncand][2][S].
constexpr int DECIDE_WAVES = 16;
__global__ __launch_bounds__(64 * DECIDE_WAVES) void k_size_decide(size_cands cands, int S, const double* ratios,
                                                                    cbp_size_result* out) {
  __shared__ double mid[CBP_MAX_K][2];
  __shared__ double score[CBP_MAX_K];
  const int l = threadIdx.x, nc = cands.n, m = 2 * S;
  for (int c = threadIdx.x >> 6; c < nc; c += DECIDE_WAVES) {
    const int i = threadIdx.x & 63;
    const double y = i < m ? log10(fmax(ratios[(size_t)c * m + i], kSizeFloor)) : 0.0;
    int rank = 0;
    for (int u = 0; u < m; ++u) {
      const double v = readlane_d(y, u);
      rank += (v < y || (v == y && u < i)) ? 1 : 0;
    }
    if (i < m && rank == m / 2 - 1) mid[c][0] = y;   // m = 2S: the middle two
    if (i < m && rank == m / 2) mid[c][1] = y;
  }
  __syncthreads();
  if (l < nc) score[l] = 0.5 * (mid[l][0] + mid[l][1]);
  __syncthreads();
  if (l == 0) {
    int best = 0;
    double bestd = -1.0;
    for (int c = 0; c < nc; ++c) {
      const double dr = (c == 0 ? 0.0 : score[c - 1]) - score[c];
      out->score[c] = score[c];
      out->drop[c] = dr;
      out->cand[c] = cands.k1[c];
      if (dr > bestd) {
        bestd = dr;
        best = c;
      }
    }
    int flags = 0;
    if (!(bestd >= kSizeMinDrop)) {
      best = nc - 1;
      flags |= CBP_SIZE_NONE_SINGULAR;
    } else if (best == 0) {
      flags |= CBP_SIZE_FIRST_SINGULAR;
    }
    out->k1 = cands.k1[best];
    out->k2 = cands.k1[best] - cands.d;
    out->flags = flags;
    out->ncand = nc;
    out->samples = S;
  }
}

}  // namespace

size_t size_probe_lds_bytes(int NL) {
  return (((size_t)NL * sizeof(cdd) + 15) & ~(size_t)15) + blk_fixed_bytes();
}

hipError_t launch_size_probe(const batch_ref& br, const size_cands& c, int S, int nmax, int NL, double* ratios,
                             hipStream_t st) {
  const int waves = nmax <= 16 ? 2 : nmax <= 24 ? 3 : nmax <= 32 ? 4 : nmax <= 40 ? 5 : 8;
  hipLaunchKernelGGL(k_size_probe, dim3(c.n * 2 * S), dim3(64 * waves), size_probe_lds_bytes(NL), st, br, c, ratios);
  return hipGetLastError();
}

hipError_t launch_size_decide(const size_cands& c, int S, const double* ratios, cbp_size_result* out,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_size_decide, dim3(1), dim3(64 * DECIDE_WAVES), 0, st, c, S, ratios, out);
  return hipGetLastError();
}

}  // namespace cbp
