// Unit-circle evaluation of the blurred frames (Sec. 4 eq. 3; Sec. 5: the
// evaluation at points around the unit circle is a DFT along one axis).
//
// For w_j = exp(-2 pi i j / S):
//   EX[j][x] = sum_y B[y][x] w_j^y = sum_{r<S} w_j^r F[r][x],  F[r][x] = sum_{y = r mod S} B[y][x]
//   EY[i][y] = sum_x B[y][x] w_i^x = sum_{r<S} w_i^r G[y][r],  G[y][r] = sum_{x = r mod S} B[y][x]
// i.e. a fold of the frame modulo S along one axis (one FP64 add per pixel)
// followed by an S-point DFT.  All accumulation is FP64 whatever the frame
// type.  The column fold runs over row groups and residues (partials per
// group, summed in a fixed order by the evaluation kernel), the row fold one
// row per wave.
//
// Layouts (cf = 2*channel + frame):
//   fpart [RG][ncf][S][Wmax] double, EX [ncf][S][Wmax] c64, EY [ncf][S][Hmax] c64.
// The row evaluation of a deblurring call is done by the forward row FFT
// kernel (same arithmetic, same order) from the rows it loads anyway; k_front
// serves kernel-only calls and the one-frame evaluation.
#include "eigsmall.h"
#include "internal.h"

namespace cbp {

namespace {

// The column evaluation.  Items: (column block, cf).
__global__ __launch_bounds__(256) void k_eval_cols(batch_ref br) {
  __shared__ double F[CBP_MAX_S][16];
  __shared__ c64 tw[CBP_MAX_S];
  for_items<Q_EVAL_COLS>(br, [&](const frame_desc& d, int item) __attribute__((always_inline)) {
    eval_cols_item(d, item, F, tw);
  });
}

// Row fold and S-point DFT: two waves per row.  With G = floor(128 / S)
// lane groups, lane l = g S + r (g < G) of the pair sums the row entries
// x = r + S (g + G i), i = 0, 1, ... in order; residue r is then the sum of
// its G partials in group order.  The row passes fold the rows they hold with
// the same lanes and the same order, so both give the same bits.
// Items: (pair of rows, cf).
template <typename T>
__device__ inline void eval_rows_item(const frame_desc& d, int item, double (*part)[128], double (*g)[CBP_MAX_S],
                                      c64* tw) {
  const int ny = (d.Hmax + 1) / 2;
  const int by = item % ny, cf = item / ny;
  const int S = d.S, G = 128 / S;
  const T* b;
  int64_t pitch;
  int H, W;
  pick_frame(d, cf, b, pitch, H, W);
  const int w = threadIdx.x >> 7, l = threadIdx.x & 127;
  const int y = by * 2 + w;
  const int gl = l / S, r = l - gl * S;
  unit_twiddles(tw, S);
  double acc = 0.0;
  if (y < H && gl < G) acc = fold_strided(b + (int64_t)y * pitch, 1, r + S * gl, S * G, W);
  part[w][l] = acc;
  __syncthreads();
  if (l < S) {
    double sr = part[w][l];
    for (int q = 1; q < G; ++q) sr += part[w][q * S + l];
    g[w][l] = sr;
  }
  __syncthreads();
  if (y < H && l < S) d.ey[((size_t)cf * S + l) * d.Hmax + y] = dft_at(g[w], 1, tw, S, l);
}

// A call's first launch without a row FFT: g.fold workgroups fold columns,
// g.eval evaluate rows, g.twid fill the twiddle tables (independent work in
// one launch instead of two or three, each of which costs ~5 us however
// little it does).  Kernels only, 1080p RGB FP32: fold 21.5 and rows 12.8 us ->
// 22.7 (the fold in groups of four columns per lane).
template <typename T>
__global__ __launch_bounds__(256) void k_front(batch_ref br_ws, front_grid g, inline_head ih) {
  __shared__ double part[2][128];
  __shared__ double gs[2][CBP_MAX_S];
  __shared__ c64 tw[CBP_MAX_S];
  const batch_ref br = first_launch_head(br_ws, ih);
  const int b = (int)blockIdx.x;
  if (b < g.fold)
    for_wave_items<Q_FOLD>(br, b, g.fold, [&](const frame_desc& d, int item, int lane)
                                              __attribute__((always_inline)) { fold_item<T>(d, item, lane); });
  else if (b < g.fold + g.eval)
    for_items_part<Q_EVAL_ROWS>(br, b - g.fold, g.eval, [&](const frame_desc& d, int item)
                                                            __attribute__((always_inline)) {
                                                              eval_rows_item<T>(d, item, part, gs, tw);
                                                            });
  else
    for_items_part<Q_TWID>(br, b - g.fold - g.eval, g.twid, [&](const frame_desc& d, int item)
                                                                __attribute__((always_inline)) { twiddle_item(d, item); });
}

}  // namespace

template <typename T>
hipError_t launch_front(const batch_ref& br, const front_grid& g, const inline_head* ih, hipStream_t st) {
  prof_begin(PH_FOLD, st);
  inline_head h;
  if (ih) h = *ih;
  else h.ndesc_bytes = h.nstart_bytes = 0;
  hipLaunchKernelGGL(k_front<T>, dim3(g.fold + g.eval + g.twid), dim3(256), 0, st, br, g, h);
  prof_end(PH_FOLD, st);
  return hipGetLastError();
}

hipError_t launch_eval_cols(const batch_ref& br, int grid, hipStream_t st) {
  prof_begin(PH_EVAL_COLS, st);
  hipLaunchKernelGGL(k_eval_cols, dim3(grid), dim3(256), 0, st, br);
  prof_end(PH_EVAL_COLS, st);
  return hipGetLastError();
}

template hipError_t launch_front<float>(const batch_ref&, const front_grid&, const inline_head*, hipStream_t);
template hipError_t launch_front<double>(const batch_ref&, const front_grid&, const inline_head*, hipStream_t);

}  // namespace cbp
