// The learned form's network: a 32 -> 128 -> 128 -> 2 MLP with ReLU, BF16
// weights and activations on the matrix cores (v_mfma_f32_32x32x16_bf16) with
// FP32 accumulation, FP32 biases, FP32 master weights and Adam moments for
// training.  It reads each sample's Gram spectrum and predicts a confidence
// weight w = clip(softplus(o1), 1e-3, 1e3) and a Tikhonov strength
// tau = exp(clip(o2, -30, 5)); the paper has no counterpart of this form.
//
// Layouts (row-major; "bf16" = bfloat16 bits, round to nearest even):
//   parameters, FP32, packed: W1 [128][32], b1 [128], W2 [128][128], b2 [128],
//                             W3 [2][128], b3 [2]                 (MLP_NPARAM)
//   inference blob: header (4 x uint32: magic, version, 32, 128), then bf16
//                   W1, W2, W3 and FP32 b1, b2, b3                 (mlp_blob)
//   features X [n][32] FP32; outputs [n][2] FP32 (o1, o2).
//
// Matrix-core tiles: a 32 x 32 FP32 tile D = A B^T with A [32][K], B [32][K]
// (k contiguous in LDS).  Lane l supplies row l % 32 of A (and of B) at
// k = k0 + 8 (l / 32) .. + 7; accumulator v of lane l is
// D[8 (v / 4) + 4 (l / 32) + v % 4][l % 32].
#include <algorithm>

#include "mlp.h"

#include "internal.h"

namespace cbp {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__device__ inline unsigned short to_bf16(float f) {
  unsigned int u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__device__ inline float from_bf16(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

// D += A B^T over K (a multiple of 16) for one wave; A, B: 32 rows with row
// stride lda / ldb (elements), k contiguous, 16-byte aligned rows.
__device__ inline void tile_abt(const unsigned short* A, int lda, const unsigned short* B, int ldb, int K,
                                v16f& acc) {
  const int l = threadIdx.x & 63;
  const unsigned short* a = A + (size_t)(l & 31) * lda + 8 * (l >> 5);
  const unsigned short* b = B + (size_t)(l & 31) * ldb + 8 * (l >> 5);
  for (int k0 = 0; k0 < K; k0 += 16) {
    const v4u ua = *(const v4u*)(a + k0);
    const v4u ub = *(const v4u*)(b + k0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, ua), __builtin_bit_cast(v8bf, ub), acc,
                                                  0, 0, 0);
  }
}

__device__ inline int tile_row(int v) { return 8 * (v >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (v & 3); }
__device__ inline int tile_col() { return threadIdx.x & 31; }

constexpr int RB = 64;          // rows per workgroup in the row-blocked kernels
constexpr int LD1 = MLP_FEAT + 8;    // LDS row strides (bf16), padded against bank conflicts
constexpr int LDH = MLP_HIDDEN + 8;

// ------------------------------------------------------------------ forward
// One workgroup (4 waves) per block of 64 rows.  Layer 1 and 2 on the matrix
// cores; the 2-output head on the vector units in FP32.
struct fwd_args {
  const float* X;
  int n;
  const unsigned short* W1;  // bf16 [128][32]
  const unsigned short* W2;  // bf16 [128][128]
  const float* W3;           // FP32 [2][128] (the head stays FP32)
  const float* b1;
  const float* b2;
  const float* b3;
  float* out;                // [n][2]
};

// LDS of one 64-row block.
struct fwd_lds {
  unsigned short xs[RB * LD1];
  unsigned short w1s[MLP_HIDDEN * LD1];
  unsigned short hs[RB * LDH];
  unsigned short w2s[MLP_HIDDEN * LDH];
  float h2f[RB][MLP_HIDDEN + 1];
  float out[RB][MLP_OUT];
};

// A bf16 matrix [rows][cols] (cols a multiple of 8, 16-byte aligned) into LDS
// rows of stride ld, eight entries per access, by 256 threads.
__device__ inline void stage_bf16(unsigned short* dst, int ld, const unsigned short* src, int rows, int cols) {
  const int per = cols >> 3;
  for (int e = threadIdx.x; e < rows * per; e += 256) {
    const int r = e / per, c = (e - r * per) * 8;
    *(v4u*)(dst + r * ld + c) = *(const v4u*)(src + (size_t)r * cols + c);
  }
}

// Forward of rows [0, nrows) of X (nrows <= 64) into L.out.
__device__ inline void mlp_block(fwd_lds& L, const float* X, int nrows, const unsigned short* W1,
                                 const unsigned short* W2, const float* W3, const float* b1, const float* b2,
                                 const float* b3) {
  const int tid = threadIdx.x, w = tid >> 6;
  for (int e = tid; e < RB * MLP_FEAT; e += 256) {
    const int r = e / MLP_FEAT, f = e % MLP_FEAT;
    L.xs[r * LD1 + f] = r < nrows ? to_bf16(X[(size_t)r * MLP_FEAT + f]) : (unsigned short)0;
  }
  stage_bf16(L.w1s, LD1, W1, MLP_HIDDEN, MLP_FEAT);
  stage_bf16(L.w2s, LDH, W2, MLP_HIDDEN, MLP_HIDDEN);
  __syncthreads();
  // layer 1: 64 x 128 = 2 x 4 tiles of 32 x 32 over the 4 waves
  for (int t = w; t < 8; t += 4) {
    const int ti = t >> 2, tj = t & 3;
    v16f acc = {};
    tile_abt(L.xs + ti * 32 * LD1, LD1, L.w1s + tj * 32 * LD1, LD1, MLP_FEAT, acc);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = ti * 32 + tile_row(v), h = tj * 32 + tile_col();
      L.hs[r * LDH + h] = to_bf16(fmaxf(acc[v] + b1[h], 0.0f));
    }
  }
  __syncthreads();
  // layer 2
  for (int t = w; t < 8; t += 4) {
    const int ti = t >> 2, tj = t & 3;
    v16f acc = {};
    tile_abt(L.hs + ti * 32 * LDH, LDH, L.w2s + tj * 32 * LDH, LDH, MLP_HIDDEN, acc);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = ti * 32 + tile_row(v), h = tj * 32 + tile_col();
      L.h2f[r][h] = from_bf16(to_bf16(fmaxf(acc[v] + b2[h], 0.0f)));
    }
  }
  __syncthreads();
  // head: 2 outputs per row, 128-term FP32 dot products on the vector units
  if (tid < MLP_OUT * RB) {
    const int r = tid >> 1, o = tid & 1;
    float sacc = b3[o];
    for (int h = 0; h < MLP_HIDDEN; ++h) sacc = fmaf(L.h2f[r][h], W3[o * MLP_HIDDEN + h], sacc);
    L.out[r][o] = sacc;
  }
  __syncthreads();
}

__global__ __launch_bounds__(256) void k_mlp_forward(fwd_args a) {
  __shared__ __attribute__((aligned(16))) fwd_lds L;
  const int r0 = blockIdx.x * RB;
  const int nrows = min(RB, a.n - r0);
  mlp_block(L, a.X + (size_t)r0 * MLP_FEAT, nrows, a.W1, a.W2, a.W3, a.b1, a.b2, a.b3);
  if (threadIdx.x < MLP_OUT * RB) {
    const int r = threadIdx.x >> 1, o = threadIdx.x & 1;
    if (r < nrows) a.out[(size_t)(r0 + r) * MLP_OUT + o] = L.out[r][o];
  }
}

// The learned form inside a deblurring call: per frame, the 2S samples'
// features (written by the eigen-solve kernel) through the network, then
//   wts[j] = w of pass-X sample j, wts[S + i] = w of pass-Y sample i,
//   wts[2S] = tau = median of the 2S values tau_j (mean of the middle two).
// Items: one per frame.
__global__ __launch_bounds__(256) void k_mlp_frames(batch_ref br, const mlp_blob* blob) {
  __shared__ __attribute__((aligned(16))) fwd_lds L;
  __shared__ double tj[64];
  __shared__ double mid[2];
  for_items<Q_FINALIZE>(br, [&](const frame_desc& d, int) __attribute__((always_inline)) {
    const int n = 2 * d.S;
    const int t = threadIdx.x;
    // a blob whose header is not this network's: unit weights and tau = 0
    // (the learned assembly then reduces to the plain one) and a flag
    if (blob->magic != MLP_MAGIC || blob->version != MLP_VERSION || blob->feat != MLP_FEAT ||
        blob->hidden != MLP_HIDDEN) {
      if (t < n) d.wts[t] = 1.0;
      if (t == 0) {
        d.wts[n] = 0.0;
        if (d.diag) atomicOr(&d.diag->flags, CBP_DIAG_BAD_NETWORK);
      }
      return;
    }
    mlp_block(L, d.feat, n, blob->W1, blob->W2, blob->W3, blob->b1, blob->b2, blob->b3);
    if (t < n) {
      const double o1 = L.out[t][0], o2 = L.out[t][1];
      const double sp = o1 > 30.0 ? o1 : log1p(exp(o1));
      d.wts[t] = fmin(fmax(sp, 1e-3), 1e3);
      tj[t] = exp(fmin(fmax(o2, -30.0), 5.0));
    }
    __syncthreads();
    if (t < n) {
      const double v = tj[t];
      int rank = 0;
      for (int u = 0; u < n; ++u) rank += (tj[u] < v) || (tj[u] == v && u < t);
      if (rank == n / 2 - 1) mid[0] = v;
      if (rank == n / 2) mid[1] = v;
    }
    __syncthreads();
    if (t == 0) d.wts[n] = 0.5 * (mid[0] + mid[1]);
  });
}

// ------------------------------------------------------------------ training step
// k_mlp_step: forward, loss, backward and the weight gradients of blocks of 64
// rows, everything between the features and the gradient partials in LDS and
// registers (activations and deltas used to make three trips through memory
// between four launches).  Per row: o = (o1, o2), loss_r = (log softplus(o1) -
// t1)^2 + (o2 - t2)^2, dO = d(mean loss)/dO; dZ2 = (dO W3) * [H2 > 0], dZ1 =
// (dZ2 W2) * [H1 > 0] in bf16 (as the forward's activations); dW2 = dZ2^T H1
// and dW1 = dZ1^T X on the matrix cores from transposed copies (r contiguous)
// that the epilogues write beside the row-major ones (four consecutive rows of
// an accumulator are one 8-byte store).  A workgroup takes the row blocks b, b
// + G, ... and writes its sums once: part[b][MLP_PART], in parameter order,
// then the loss.  Latency-bound at one block per workgroup (8192 rows: 128
// workgroups, about ten barriers).
// k_mlp_update: the partials summed over workgroups in order into the
// gradient (and the loss), then, in a training step, Adam on the FP32 master
// weights and the bf16 copies (W1, W2, W2^T).
// 8192 rows: 17 launches, 323 us -> two, 21.5 + 4.1 us.
constexpr int MLP_PART = (MLP_NPARAM + 1 + 63) & ~63;
constexpr int MLP_STEP_WG = 256;            // workgroups at most
constexpr int LDT = RB + 8;                 // stride of the transposed copies

struct step_args {
  const float* X;
  const float* T;
  int n;
  const unsigned short* W1;   // bf16 [128][32]
  const unsigned short* W2;   // bf16 [128][128]
  const unsigned short* W2t;  // its transpose
  const float* p;             // FP32 parameters (biases, head)
  float* part;                // [gridDim.x][MLP_PART]
};

struct step_lds {
  unsigned short xs[RB * LD1];
  unsigned short xt[MLP_FEAT * LDT];
  unsigned short w1s[MLP_HIDDEN * LD1];
  unsigned short w2s[MLP_HIDDEN * LDH];                                  // W2, then W2^T
  unsigned short hs[MLP_HIDDEN * LDT > RB * LDH ? MLP_HIDDEN * LDT : RB * LDH];   // H1 [r][h], then dZ1^T [h][r]
  unsigned short ht[MLP_HIDDEN * LDT];                                   // H1^T
  unsigned short h2[RB * LDH];                                           // H2 [r][h], then dZ2
  unsigned short d2t[MLP_HIDDEN * LDT];                                  // dZ2^T
  float w3[MLP_OUT * MLP_HIDDEN];
  float dos[RB][2];
  float red[4][MLP_HIDDEN];
  float loss[RB];
};

// Four bf16 values of consecutive rows as one 8-byte store.
__device__ inline void store4(unsigned short* p, const unsigned short* v) {
  *(uint2*)p = uint2{(unsigned int)v[0] | (unsigned int)v[1] << 16, (unsigned int)v[2] | (unsigned int)v[3] << 16};
}

__global__ __launch_bounds__(256) void k_mlp_step(step_args a) {
  __shared__ __attribute__((aligned(16))) step_lds L;
  const int tid = threadIdx.x, w = tid >> 6;
  const int nb = (a.n + RB - 1) / RB;
  // both layouts of the second layer in registers (128 x 16 groups of eight)
  v4u r2[8], r2t[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int e = tid + 256 * i;
    r2[i] = ((const v4u*)a.W2)[e];
    r2t[i] = ((const v4u*)a.W2t)[e];
  }
  auto put_w2 = [&](const v4u* v) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = tid + 256 * i;
      *(v4u*)(L.w2s + (e >> 4) * LDH + (e & 15) * 8) = v[i];
    }
  };
  stage_bf16(L.w1s, LD1, a.W1, MLP_HIDDEN, MLP_FEAT);
  if (tid < MLP_OUT * MLP_HIDDEN) L.w3[tid] = a.p[MLP_OFF_W3 + tid];
  v16f g2[4], g1 = {};
#pragma unroll
  for (int t = 0; t < 4; ++t) g2[t] = v16f{};
  const int h = tid & 127, hf = tid >> 7;          // this thread's hidden unit and half of the rows
  float db1 = 0.0f, db2 = 0.0f, dw30 = 0.0f, dw31 = 0.0f, db3 = 0.0f, loss = 0.0f;
  const float w30 = a.p[MLP_OFF_W3 + h], w31 = a.p[MLP_OFF_W3 + MLP_HIDDEN + h];
  for (int b = blockIdx.x; b < nb; b += gridDim.x) {
    const int r0 = b * RB, nrows = min(RB, a.n - r0);
    put_w2(r2);
    // features: eight per thread, row tid / 4
    {
      const int r = tid >> 2, f0 = (tid & 3) * 8;
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = r < nrows ? a.X[(size_t)(r0 + r) * MLP_FEAT + f0 + i] : 0.0f;
      unsigned short q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = to_bf16(x[i]);
        L.xt[(f0 + i) * LDT + r] = q[i];
      }
      store4(L.xs + r * LD1 + f0, q);
      store4(L.xs + r * LD1 + f0 + 4, q + 4);
    }
    __syncthreads();
    // layers 1 and 2: 2 x 4 tiles of 32 x 32 over the four waves
#pragma unroll
    for (int t = w; t < 8; t += 4) {
      const int ti = t >> 2, hh = (t & 3) * 32 + tile_col();
      v16f acc = {};
      tile_abt(L.xs + ti * 32 * LD1, LD1, L.w1s + (t & 3) * 32 * LD1, LD1, MLP_FEAT, acc);
      const float bias = a.p[MLP_OFF_B1 + hh];
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        const int r = ti * 32 + tile_row(v);
        unsigned short q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          q[i] = to_bf16(fmaxf(acc[v + i] + bias, 0.0f));
          L.hs[(r + i) * LDH + hh] = q[i];
        }
        store4(L.ht + hh * LDT + r, q);
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = w; t < 8; t += 4) {
      const int ti = t >> 2, hh = (t & 3) * 32 + tile_col();
      v16f acc = {};
      tile_abt(L.hs + ti * 32 * LDH, LDH, L.w2s + (t & 3) * 32 * LDH, LDH, MLP_HIDDEN, acc);
      const float bias = a.p[MLP_OFF_B2 + hh];
#pragma unroll
      for (int v = 0; v < 16; ++v) L.h2[(ti * 32 + tile_row(v)) * LDH + hh] = to_bf16(fmaxf(acc[v] + bias, 0.0f));
    }
    __syncthreads();
    put_w2(r2t);
    // head and loss: four lanes per row, 32 hidden units each
    {
      const int r = tid >> 2, q = tid & 3;
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const v4u u = *(const v4u*)(L.h2 + r * LDH + q * 32 + i * 8);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float hv = from_bf16((unsigned short)(u[j >> 1] >> (16 * (j & 1))));
          const int c = q * 32 + i * 8 + j;
          s0 = fmaf(hv, L.w3[c], s0);
          s1 = fmaf(hv, L.w3[MLP_HIDDEN + c], s1);
        }
      }
      s0 += __shfl_xor(s0, 1);
      s1 += __shfl_xor(s1, 1);
      s0 += __shfl_xor(s0, 2);
      s1 += __shfl_xor(s1, 2);
      if (q == 0) {
        float d1 = 0.0f, d2 = 0.0f, lr = 0.0f;
        if (r < nrows) {
          const float o1 = s0 + a.p[MLP_OFF_B3], o2 = s1 + a.p[MLP_OFF_B3 + 1];
          const float sp = o1 > 20.0f ? o1 : log1pf(expf(o1));
          const float sg = 1.0f / (1.0f + expf(-o1));
          const float e1 = logf(sp) - a.T[(size_t)(r0 + r) * 2], e2 = o2 - a.T[(size_t)(r0 + r) * 2 + 1];
          lr = e1 * e1 + e2 * e2;
          d1 = 2.0f * e1 / (float)a.n * sg / sp;
          d2 = 2.0f * e2 / (float)a.n;
        }
        L.dos[r][0] = d1;
        L.dos[r][1] = d2;
        L.loss[r] = lr;
      }
    }
    __syncthreads();
    if (tid < 3) {   // db3 and the loss, in row order
      float s = 0.0f;
      for (int r = 0; r < RB; ++r) s += tid < 2 ? L.dos[r][tid] : L.loss[r];
      if (tid < 2) db3 += s;
      else loss += s;
    }
    // dZ2 over H2 (in place, and transposed), db2 and dW3
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      unsigned short q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = hf * 32 + g * 8 + i;
        const float hv = from_bf16(L.h2[r * LDH + h]);
        const float d1 = L.dos[r][0], d2 = L.dos[r][1];
        dw30 = fmaf(d1, hv, dw30);
        dw31 = fmaf(d2, hv, dw31);
        q[i] = hv > 0.0f ? to_bf16(d1 * w30 + d2 * w31) : (unsigned short)0;
        db2 += from_bf16(q[i]);
        L.h2[r * LDH + h] = q[i];
      }
      store4(L.d2t + h * LDT + hf * 32 + g * 8, q);
      store4(L.d2t + h * LDT + hf * 32 + g * 8 + 4, q + 4);
    }
    __syncthreads();
    // dZ1^T into the place of H1 (whose last reader was layer 2)
#pragma unroll
    for (int t = w; t < 8; t += 4) {
      const int ti = t >> 2, hh = (t & 3) * 32 + tile_col();
      v16f acc = {};
      tile_abt(L.h2 + ti * 32 * LDH, LDH, L.w2s + (t & 3) * 32 * LDH, LDH, MLP_HIDDEN, acc);
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        const int r = ti * 32 + tile_row(v);
        const uint2 on = *(const uint2*)(L.ht + hh * LDT + r);
        unsigned short q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned short hv = (unsigned short)((i < 2 ? on.x : on.y) >> (16 * (i & 1)));
          q[i] = from_bf16(hv) > 0.0f ? to_bf16(acc[v + i]) : (unsigned short)0;
        }
        store4(L.hs + hh * LDT + r, q);
      }
    }
    // dW2: 4 x 4 tiles, wave w the tile row w
#pragma unroll
    for (int t = 0; t < 4; ++t)
      tile_abt(L.d2t + w * 32 * LDT, LDT, L.ht + t * 32 * LDT, LDT, RB, g2[t]);
    __syncthreads();
    // dW1: 4 x 1 tiles; db1
    tile_abt(L.hs + w * 32 * LDT, LDT, L.xt, LDT, RB, g1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const v4u u = *(const v4u*)(L.hs + h * LDT + hf * 32 + i * 8);
#pragma unroll
      for (int j = 0; j < 8; ++j) db1 += from_bf16((unsigned short)(u[j >> 1] >> (16 * (j & 1))));
    }
    __syncthreads();   // the next block refills xs, xt and w2s
  }
  float* p = a.part + (size_t)blockIdx.x * MLP_PART;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = w * 32 + tile_row(v);
    p[MLP_OFF_W1 + i * MLP_FEAT + tile_col()] = g1[v];
#pragma unroll
    for (int t = 0; t < 4; ++t) p[MLP_OFF_W2 + i * MLP_HIDDEN + t * 32 + tile_col()] = g2[t][v];
  }
  // the two halves of the rows
  if (hf == 1) {
    L.red[0][h] = db1;
    L.red[1][h] = db2;
    L.red[2][h] = dw30;
    L.red[3][h] = dw31;
  }
  __syncthreads();
  if (hf == 0) {
    p[MLP_OFF_B1 + h] = db1 + L.red[0][h];
    p[MLP_OFF_B2 + h] = db2 + L.red[1][h];
    p[MLP_OFF_W3 + h] = dw30 + L.red[2][h];
    p[MLP_OFF_W3 + MLP_HIDDEN + h] = dw31 + L.red[3][h];
  }
  if (tid < 2) p[MLP_OFF_B3 + tid] = db3;
  if (tid == 2) p[MLP_NPARAM] = loss;
}

struct update_args {
  const float* part;
  int G, n;
  float* g;        // gradient in the state
  float* grads;    // the caller's copy, or NULL
  float* loss;
  int adam;        // 1: also the Adam step below
  float *p, *m, *v;
  unsigned short *W1, *W2, *W2t;
  float lr, b1, b2, eps, c1, c2;
};

// 64 parameters per workgroup (the last index is the loss), four threads each
// a quarter of the partials, eight loads in flight, summed in order.
__global__ __launch_bounds__(256) void k_mlp_update(update_args a) {
  __shared__ float red[4][64];
  const int l = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + l;
  const int per = (a.G + 3) >> 2, g0 = q * per, g1 = min(a.G, g0 + per);
  float s = 0.0f;
  const float* src = a.part + i;     // i < MLP_PART always
  int g = g0;
  for (; g + 8 <= g1; g += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(g + u) * MLP_PART];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; g < g1; ++g) s += src[(size_t)g * MLP_PART];
  red[q][l] = s;
  __syncthreads();
  if (q != 0 || i > MLP_NPARAM) return;
  s = ((red[0][l] + red[1][l]) + red[2][l]) + red[3][l];
  if (i == MLP_NPARAM) {
    *a.loss = s * (1.0f / (float)a.n);
    return;
  }
  a.g[i] = s;
  if (a.grads) a.grads[i] = s;
  if (!a.adam) return;
  const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * s;
  const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * s * s;
  a.m[i] = mi;
  a.v[i] = vi;
  const float pi = a.p[i] - a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
  a.p[i] = pi;
  if (i < MLP_OFF_B1) a.W1[i - MLP_OFF_W1] = to_bf16(pi);
  if (i >= MLP_OFF_W2 && i < MLP_OFF_B2) {
    const int e = i - MLP_OFF_W2;
    a.W2[e] = to_bf16(pi);
    a.W2t[(e % MLP_HIDDEN) * MLP_HIDDEN + e / MLP_HIDDEN] = to_bf16(pi);
  }
}

__global__ void k_mlp_quantise(const float* p, unsigned short* W1, unsigned short* W2, unsigned short* W2t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < MLP_HIDDEN * MLP_FEAT) W1[i] = to_bf16(p[MLP_OFF_W1 + i]);
  if (i < MLP_HIDDEN * MLP_HIDDEN) {
    const unsigned short q = to_bf16(p[MLP_OFF_W2 + i]);
    W2[i] = q;
    W2t[(i % MLP_HIDDEN) * MLP_HIDDEN + i / MLP_HIDDEN] = q;
  }
}

__global__ void k_mlp_zero2(float* a, float* b, int np) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < np) { a[i] = 0.0f; b[i] = 0.0f; }
}

// The inference blob from the FP32 master weights.
__global__ void k_mlp_export(const float* p, mlp_blob* b) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) { b->magic = MLP_MAGIC; b->version = MLP_VERSION; b->feat = MLP_FEAT; b->hidden = MLP_HIDDEN; }
  if (i < MLP_HIDDEN * MLP_FEAT) b->W1[i] = to_bf16(p[MLP_OFF_W1 + i]);
  if (i < MLP_HIDDEN * MLP_HIDDEN) b->W2[i] = to_bf16(p[MLP_OFF_W2 + i]);
  if (i < MLP_OUT * MLP_HIDDEN) b->W3[i] = p[MLP_OFF_W3 + i];
  if (i < MLP_HIDDEN) { b->b1[i] = p[MLP_OFF_B1 + i]; b->b2[i] = p[MLP_OFF_B2 + i]; }
  if (i < MLP_OUT) b->b3[i] = p[MLP_OFF_B3 + i];
}

}  // namespace

// ------------------------------------------------------------------ host side
namespace {

struct state_view {
  float *p, *m, *v, *g;                 // MLP_NPARAM each
  unsigned short *W1, *W2, *W2t;        // bf16 copies
  float* part;                          // partial sums of the step's workgroups
};

int step_workgroups(int rows) { return std::min((rows + RB - 1) / RB, MLP_STEP_WG); }

size_t part_floats(int rows) { return (size_t)step_workgroups(rows) * MLP_PART; }

state_view carve(void* base, int rows) {
  char* c = (char*)base;
  auto take = [&](size_t bytes) { char* at = c; c += (bytes + 255) & ~(size_t)255; return at; };
  state_view s;
  s.p = (float*)take(MLP_NPARAM * 4);
  s.m = (float*)take(MLP_NPARAM * 4);
  s.v = (float*)take(MLP_NPARAM * 4);
  s.g = (float*)take(MLP_NPARAM * 4);
  s.W1 = (unsigned short*)take(MLP_HIDDEN * MLP_FEAT * 2);
  s.W2 = (unsigned short*)take(MLP_HIDDEN * MLP_HIDDEN * 2);
  s.W2t = (unsigned short*)take(MLP_HIDDEN * MLP_HIDDEN * 2);
  s.part = (float*)take(part_floats(rows) * 4);
  return s;
}

size_t carve_bytes(int rows) {
  state_view s = carve(nullptr, rows);
  return (size_t)((char*)s.part - (char*)nullptr) + ((part_floats(rows) * 4 + 255) & ~(size_t)255);
}

}  // namespace

size_t mlp_state_bytes(int rows) { return carve_bytes(rows); }

hipError_t launch_mlp_frames(const batch_ref& br, int grid, const void* blob,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_frames, dim3(grid), dim3(256), 0, st, br, (const mlp_blob*)blob);
  return hipGetLastError();
}

hipError_t mlp_forward_blob(const void* blob, const float* X, int n, float* out, hipStream_t st) {
  const mlp_blob* b = (const mlp_blob*)blob;
  fwd_args a = {X, n, b->W1, b->W2, b->W3, b->b1, b->b2, b->b3, out};
  hipLaunchKernelGGL(k_mlp_forward, dim3((n + RB - 1) / RB), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t mlp_set_params(void* state, int rows, const float* params, hipStream_t st) {
  const state_view s = carve(state, rows);
  const hipError_t e = hipMemcpyAsync(s.p, params, MLP_NPARAM * 4, hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_zero2, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, st, s.m, s.v, MLP_NPARAM);
  hipLaunchKernelGGL(k_mlp_quantise, dim3((MLP_HIDDEN * MLP_HIDDEN + 255) / 256), dim3(256), 0, st, s.p, s.W1, s.W2,
                     s.W2t);
  return hipGetLastError();
}

hipError_t mlp_get_params(const void* state, int rows, float* params, hipStream_t st) {
  const state_view s = carve(const_cast<void*>(state), rows);
  return hipMemcpyAsync(params, s.p, MLP_NPARAM * 4, hipMemcpyDeviceToDevice, st);
}

// Checkpoint of the training state: master weights and both Adam moments,
// [3][MLP_NPARAM] FP32.  Loading restores them and the bf16 copies.
hipError_t mlp_save_state(const void* state, int rows, float* out, hipStream_t st) {
  const state_view s = carve(const_cast<void*>(state), rows);
  const float* src[3] = {s.p, s.m, s.v};
  for (int i = 0; i < 3; ++i) {
    const hipError_t e = hipMemcpyAsync(out + (size_t)i * MLP_NPARAM, src[i], MLP_NPARAM * 4,
                                        hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t mlp_load_state(void* state, int rows, const float* in, hipStream_t st) {
  const state_view s = carve(state, rows);
  float* dst[3] = {s.p, s.m, s.v};
  for (int i = 0; i < 3; ++i) {
    const hipError_t e = hipMemcpyAsync(dst[i], in + (size_t)i * MLP_NPARAM, MLP_NPARAM * 4,
                                        hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_mlp_quantise, dim3((MLP_HIDDEN * MLP_HIDDEN + 255) / 256), dim3(256), 0, st, s.p, s.W1, s.W2,
                     s.W2t);
  return hipGetLastError();
}

namespace {

// Forward, loss and backward over n <= rows rows: the gradient of the mean
// loss into the state (and into grads when not NULL), the loss into *loss;
// then, with u.adam set, the Adam step.
hipError_t step(void* state, int rows, const float* X, const float* T, int n, float* loss, float* grads,
                update_args u, hipStream_t st) {
  const state_view s = carve(state, rows);
  const int G = step_workgroups(n);
  const step_args a = {X, T, n, s.W1, s.W2, s.W2t, s.p, s.part};
  hipLaunchKernelGGL(k_mlp_step, dim3(G), dim3(256), 0, st, a);
  u.part = s.part;
  u.G = G;
  u.n = n;
  u.g = s.g;
  u.grads = grads;
  u.loss = loss;
  u.p = s.p;
  u.m = s.m;
  u.v = s.v;
  u.W1 = s.W1;
  u.W2 = s.W2;
  u.W2t = s.W2t;
  hipLaunchKernelGGL(k_mlp_update, dim3(MLP_PART / 64), dim3(256), 0, st, u);
  return hipGetLastError();
}

}  // namespace

hipError_t mlp_gradients(void* state, int rows, const float* X, const float* T, int n, float* loss, float* grads,
                         hipStream_t st) {
  return step(state, rows, X, T, n, loss, grads, update_args{}, st);
}

// The gradient and one Adam step (beta1 0.9, beta2 0.999, eps 1e-8); k counts
// from 1.
hipError_t mlp_train_step(void* state, int rows, const float* X, const float* T, int n, float lr, int k, float* loss,
                          hipStream_t st) {
  update_args u = {};
  u.adam = 1;
  u.lr = lr;
  u.b1 = 0.9f;
  u.b2 = 0.999f;
  u.eps = 1e-8f;
  u.c1 = 1.0f / (1.0f - powf(u.b1, (float)k));
  u.c2 = 1.0f / (1.0f - powf(u.b2, (float)k));
  return step(state, rows, X, T, n, loss, nullptr, u, st);
}

hipError_t mlp_export(const void* state, int rows, void* blob, hipStream_t st) {
  const state_view s = carve(const_cast<void*>(state), rows);
  hipLaunchKernelGGL(k_mlp_export, dim3((MLP_HIDDEN * MLP_HIDDEN + 255) / 256), dim3(256), 0, st, s.p,
                     (mlp_blob*)blob);
  return hipGetLastError();
}

}  // namespace cbp
