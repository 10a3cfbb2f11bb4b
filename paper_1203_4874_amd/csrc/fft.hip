// Two-channel regularised Fourier division (Sec. 4: the latent is obtained by
// dividing a blurred frame by the recovered kernel in the Fourier domain;
// Sec. 5: an inverse FFT of the divided spectrum).  Over a Py x Px grid that
// covers both frames (no wrap-around of the full convolutions):
//   Lhat = (conj(K1hat) B1hat + conj(K2hat) B2hat) / (|K1hat|^2 + |K2hat|^2 + lambda),
//   L    = IFFT2(Lhat) cropped to m x n
// (with the single-channel variant, the paper's B1 / K1: the K2 terms drop).
//
// Three passes, each a hand-written Stockham FFT in LDS (fft_core.h):
//   1. row pass: row y of B1 and row y of B2 packed as one complex row
//      B1 + i B2, one complex FFT, split into the two half spectra
//      T_c[y][0..Px/2] (Hermitian symmetry of real rows);
//   2. column pass: for a strip of half-spectrum columns, forward FFT of the
//      T_1 and T_2 columns (zero rows beyond H_c), the filter above with the
//      kernel spectra evaluated in place from the k x k kernels, inverse FFT,
//      keep the first m rows -> U[y][kx];
// T and U rows have a pitch of hxp >= hx entries, a multiple of 128 bytes, so
// the column pass reads and writes whole row segments.
//   3. inverse row pass: two rows of U packed as one complex spectrum (each
//      completed by Hermitian symmetry), one inverse FFT, real / imaginary
//      parts are the two output rows, scaled by 1/(Py Px), cropped to n.
// T is float (mixed form) or double (FP64 form).
#include <algorithm>
#include <atomic>
#include "eigsmall.h"
#include "internal.h"

namespace cbp {

namespace {

// ---------------------------------------------------------------- in-place passes
// The transforms run in place in LDS: every pass reads its butterflies'
// inputs into registers, synchronises, and writes the outputs over them (one
// buffer instead of a ping-pong pair).  Twiddles come from the plan's pass
// tables in LDS (fft_core.h tw_pitch), FP64 sincospi rounded once to T (one
// read per twiddle).
//
// What bounds them is vector instructions (55 to 70% of the issue slots) and
// the two barriers of a pass, not memory: a third to a half of the
// instructions were addresses, and registers held for nothing (see any_value
// and full_twiddles) kept workgroups off the CUs.  Strides as running adds,
// range checks by the buffer unit, half spectra read once, tables gathered
// from one: 8 x 1080p RGB FP32 columns 409 -> 377 us, forward rows 319 -> 255,
// inverse rows 138 -> 104 (the rows with the pass order of kDefaultTuning);
// 719x1277 FP64 columns 47 -> 29.8, single rows 27.6 -> 22.8.  With the plans
// of fft_costs and the strip widths and evaluations of later, 336, 214, 100;
// 26.2 (with the kernels' row transforms) and 21.8.  These are launches of the
// default shapes; an autotuned stream's differ by a few per cent.

// threadIdx.x behind an empty asm statement: values derived from it are
// recomputed where they are used instead of being hoisted out of the item
// loop, where they would stay live (one register each) across the kernel.
__device__ __attribute__((always_inline)) inline int local_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// A raw buffer over `bytes` bytes at p (both wave-uniform).  The hardware checks
// each access against its length: a load past the end returns zero, a store past
// it is dropped.  The rows and strips are read and written through it, so a
// lane's entry costs one 32-bit offset: no clamped 64-bit address, and no zero
// put in for the entries beyond the frame.
__device__ __attribute__((always_inline)) inline __amdgpu_buffer_rsrc_t raw_buffer(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// An offset past the end of every buffer here (all below 2^27 bytes), also with
// a strip's row offsets added.
constexpr int kPastEnd = (int)0x80000000u;

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename V>
__device__ __attribute__((always_inline)) inline V buf_load(__amdgpu_buffer_rsrc_t b, int off) {
  static_assert(sizeof(V) == 4 || sizeof(V) == 8 || sizeof(V) == 16, "one load");
  if constexpr (sizeof(V) == 4) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0));
  else if constexpr (sizeof(V) == 8) return __builtin_bit_cast(V, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
  else return __builtin_bit_cast(V, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}

template <typename V>
__device__ __attribute__((always_inline)) inline void buf_store(__amdgpu_buffer_rsrc_t b, int off, const V& v) {
  static_assert(sizeof(V) == 4 || sizeof(V) == 8 || sizeof(V) == 16, "one store");
  if constexpr (sizeof(V) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), b, off, 0, 0);
  else if constexpr (sizeof(V) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, off, 0, 0);
}

// Gives v a value on every path (any; empty asm, no instruction) where it is set
// and read only under one condition.  Without it the compiler takes the paths
// that do not set v to keep what the last loop turn left in it: registers held
// across the loop, and copies.
template <typename V>
__device__ __attribute__((always_inline)) inline void any_value(V& v) {
  asm volatile("" : "=v"(v));
}
template <typename T>
__device__ __attribute__((always_inline)) inline void any_value(cplx<T>& v) {
  any_value(v.re);
  any_value(v.im);
}

// Butterflies per thread of a radix-R pass over at most MAXE entries.
template <int NT, int R, int MAXE>
constexpr int ip_mb() { return (MAXE / R + NT - 1) / NT; }

// w_N^t, t < N, into tw by the workgroup's nt threads: FP64 sincospi rounded
// once to T, the second half from the first's conjugates.  Most of a
// workgroup's start is this function (some 60 FP64 instructions a value), so
// the other tables are gathered from it.  A call: inlined, sincospi's
// constants would be kept in some forty registers across the item loops.
template <typename T>
__device__ __attribute__((noinline)) void full_twiddles(__attribute__((address_space(3))) cplx<T>* tw, int N, int nt) {
  for (int t = threadIdx.x; 2 * t <= N; t += nt) {
    double sn, cs;
    sincospi(-2.0 * (double)t / (double)N, &sn, &cs);
    tw[t].re = T(cs);
    tw[t].im = T(sn);
    if (t > 0) {
      tw[N - t].re = T(cs);
      tw[N - t].im = T(-sn);
    }
  }
}

// unit_twiddles as a call, for the same reason.
__device__ __attribute__((noinline)) void row_unit_twiddles(__attribute__((address_space(3))) c64* tw, int S) {
  unit_twiddles((c64*)tw, S);
}

// The pass twiddle tables of plan p into tws from its full table tw.  Entry
// k P + r - 1 of the pass with stride Ns is w_(Ns R)^(r k) = w_N^(r k N / (Ns R)).
template <typename T>
__device__ __attribute__((always_inline)) inline void pass_twiddles(cplx<T>* tws, const cplx<T>* tw, const fft_plan& p,
                                                                    int nt) {
  int Ns = plan_radix(p, 0), off = 0;
  for (int s = 1; s < p.npass; ++s) {
    const int R = plan_radix(p, s), P = tw_pitch(R), n = Ns * P, step = p.N / (Ns * R);
    const float rp = __builtin_amdgcn_rcpf((float)P);
    for (int e = threadIdx.x; e < n; e += nt) {
      const int k = fdiv_floor(e, rp), r = e - mul24(k, P) + 1;
      tws[off + e] = tw[r < R ? mul24(mul24(r, k), step) : 0];
    }
    off += n;
    Ns *= R;
  }
}

// Both tables of a row pass's plan when tws holds another plan's (tabN,
// tabCode: the length and pass order it holds, wave-uniform); a, the row's
// buffer, holds the full table meanwhile.  Ends with a barrier when it wrote.
template <typename T>
__device__ __attribute__((always_inline)) inline void row_twiddles(cplx<T>* a, cplx<T>* tws, const fft_plan& p, int& tabN,
                                                                   unsigned long long& tabCode) {
  if (tabN == p.N && tabCode == p.code) return;
  full_twiddles<T>((__attribute__((address_space(3))) cplx<T>*)a, p.N, 256);
  __syncthreads();
  pass_twiddles(tws, a, p, 256);
  __syncthreads();
  tabN = p.N;
  tabCode = p.code;
}

// One radix-R pass (stride Ns) over 2^lnc transforms of length N at
// buf + c ld, in place: butterfly j of transform c reads
// buf[c ld + j + r N/R] and writes buf[c ld + (j - k) R + k + r Ns],
// k = j mod Ns (the Stockham indexing of fft_core.h, read and write phases
// separated by a barrier); tws: the pass's twiddle table.  2^lnc N <= MAXE.
// Butterfly b of the pass is (c, j) = (b mod 2^lnc, b >> lnc): consecutive
// lanes take the same j of consecutive transforms, whose entries the strip's
// column stride puts in distinct banks, and a thread's butterflies are all of
// one transform.  Strides are wave-uniform, so an entry's address is one add.
// TW: Ns > 1 (the first pass has no twiddles).
template <int R, int DIR, int NT, int MAXE, bool TW, typename T>
__device__ __attribute__((always_inline)) inline void ip_pass(cplx<T>* buf, int ld, int N, int Ns,
                                                              const cplx<T>* tws, int lnc) {
  constexpr int MB = ip_mb<NT, R, MAXE>();
  const int NR = N / R;
  // within one unit in the last place of 1 / Ns, as fdiv_floor allows at these sizes
  const float rns = __builtin_amdgcn_rcpf((float)Ns);
  cplx<T> v[MB][R];
  int pos[MB];
#pragma unroll
  for (int q = 0; q < MB; ++q) {
    any_value(pos[q]);
#pragma unroll
    for (int r = 0; r < R; ++r) any_value(v[q][r]);
  }
  const int tid = local_tid();
  cplx<T>* col = buf + mul24(tid & ((1 << lnc) - 1), ld);
  const int j0 = tid >> lnc, js = NT >> lnc;
#pragma unroll
  for (int q = 0; q < MB; ++q) {
    const int j = j0 + q * js;
    if (j < NR) {
      const int k = TW ? j - mul24(fdiv_floor(j, rns), Ns) : 0;
      pos[q] = stockham_read<R, DIR, TW>(col, NR, tws, j, k, v[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < MB; ++q)
    if (j0 + q * js < NR) {
      cplx<T>* o = col + pos[q];
#pragma unroll
      for (int r = 0; r < R; ++r, o += Ns) *o = v[q][r];
    }
  __syncthreads();
}

// The pass of radix R.
template <int DIR, int NT, int MAXE, bool TW, typename T>
__device__ __attribute__((always_inline)) inline void ip_radix(int R, cplx<T>* buf, int ld, int N, int Ns,
                                                               const cplx<T>* tws, int lnc) {
  switch (R) {
    case 2: ip_pass<2, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 3: ip_pass<3, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 4: ip_pass<4, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 5: ip_pass<5, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 6: ip_pass<6, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 7: ip_pass<7, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 9: ip_pass<9, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 10: ip_pass<10, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 12: ip_pass<12, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 14: ip_pass<14, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    case 15: ip_pass<15, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
    default: ip_pass<8, DIR, NT, MAXE, TW>(buf, ld, N, Ns, tws, lnc); break;
  }
}

// All passes of plan p over 2^lnc transforms (2^lnc p.N <= MAXE), in place;
// tws: the plan's pass tables (pass_twiddles).
template <int DIR, int NT, int MAXE, typename T>
__device__ __attribute__((always_inline)) inline void ip_fft(cplx<T>* buf, int ld, const fft_plan& p,
                                                             const cplx<T>* tws, int lnc) {
  if (p.npass == 0) return;   // N = 1
  int Ns = plan_radix(p, 0);
  ip_radix<DIR, NT, MAXE, false>(Ns, buf, ld, p.N, 1, tws, lnc);
  const cplx<T>* t = tws;   // this pass's table
  for (int s = 1; s < p.npass; ++s) {
    const int R = plan_radix(p, s);
    ip_radix<DIR, NT, MAXE, true>(R, buf, ld, p.N, Ns, t, lnc);
    t += Ns * tw_pitch(R);
    Ns *= R;
  }
}

// Largest row length (entries) of the row passes.
constexpr int ROW_MAXE = CBP_MAX_FFT_F32 > CBP_MAX_FFT_F64 ? CBP_MAX_FFT_F32 : CBP_MAX_FFT_F64;
constexpr int ROW_HALF = (ROW_MAXE / 2 + 1 + 255) / 256;   // half-spectrum entries per thread of the row passes

// ---------------------------------------------------------------- pass 1
// Rows y of both frames of channel ch into registers, entries t 256 + tid:
// zero beyond each frame's width and in rows past its height.
template <typename T>
__device__ __attribute__((always_inline)) inline void fetch_rows(const frame_desc& d, int ch, int y, T (&u)[8], T (&w)[8]) {
  const auto r1 = raw_buffer((const T*)d.b1 + ch * d.cs1 + (int64_t)min(y, d.H1 - 1) * d.p1,
                             y < d.H1 ? d.W1 * (int)sizeof(T) : 0);
  const auto r2 = raw_buffer((const T*)d.b2 + ch * d.cs2 + (int64_t)min(y, d.H2 - 1) * d.p2,
                             y < d.H2 ? d.W2 * (int)sizeof(T) : 0);
  const int off = local_tid() * (int)sizeof(T);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    u[t] = buf_load<T>(r1, off + t * 256 * (int)sizeof(T));
    w[t] = buf_load<T>(r2, off + t * 256 * (int)sizeof(T));
  }
}

// Rows y of both frames of channel ch, packed as B1 + i B2 in a (LDS, zero
// beyond each frame; a barrier since its store): the FFT and the two half
// spectra, and the fold of both rows modulo S into gy[frame][S] by the
// last wave (the caller's DFT of it, row_eval, needs no more).  twf: the plan's
// pass tables.  Ends with a barrier.
//
// The fold has k_front's lanes and order: waves 2 fr, 2 fr + 1 fold frame fr's
// row into partials, lane g S + r of the pair summing x = r + S (g + G i); a
// residue then adds its G partials in order.  The partials are behind the
// passes' barriers when they are added, so the fold adds none of its own.
template <typename T>
__device__ __attribute__((always_inline)) inline void row_transform(const frame_desc& d, int ch, int y, cplx<T>* a,
                                                                    const cplx<T>* twf, double (*gy)[CBP_MAX_S],
                                                                    double (*fpart_l)[128]) {
  static_assert(2 * CBP_MAX_S <= 64, "both rows' residues fill one wave");
  const fft_plan& px = d.fx;
  const int N = px.N, hx = d.hx, S = d.S;
  const bool in1 = y < d.H1, in2 = y < d.H2;
  const int G = 128 / S;
  {
    const int fr = threadIdx.x >> 7, l = threadIdx.x & 127;
    double acc = 0.0;
    if ((fr ? in2 : in1) && l < G * S) acc = fold_strided((const T*)a + fr, 2, l, S * G, fr ? d.W2 : d.W1);
    fpart_l[fr][l] = acc;
    if (px.npass == 0) __syncthreads();   // N = 1
  }
  ip_fft<-1, 256, ROW_MAXE>(a, N, px, twf, 0);
  {
    const int lane = (int)threadIdx.x - 192, fr = lane >= S, l = fr ? lane - S : lane;
    if (lane >= 0 && lane < 2 * S) {
      double sr = fpart_l[fr][l];
      for (int q = 1; q < G; ++q) sr += fpart_l[fr][q * S + l];
      gy[fr][l] = sr;
    }
  }
  const int64_t to = (int64_t)ch * d.Hmax * d.hxp + (int64_t)y * d.hxp;
  const int row = hx * (int)sizeof(cplx<T>);
  const auto o1 = raw_buffer((cplx<T>*)d.t1 + to, in1 ? row : 0), o2 = raw_buffer((cplx<T>*)d.t2 + to, in2 ? row : 0);
  for (int k = threadIdx.x; k < hx; k += 256) {
    const cplx<T> zk = a[k];
    const cplx<T> zn = conj(a[k == 0 ? 0 : N - k]);
    const cplx<T> s = zk + zn, df = zk - zn;
    const int off = k * (int)sizeof(cplx<T>);
    buf_store(o1, off, cplx<T>{T(0.5) * s.re, T(0.5) * s.im});       // (Z_k + conj Z_{N-k}) / 2
    buf_store(o2, off, cplx<T>{T(0.5) * df.im, T(-0.5) * df.re});    // (Z_k - conj Z_{N-k}) / (2i)
  }
  __syncthreads();
}

// The S-point DFTs of the folds gy[i] of rows y0 + i S, i < n, both frames
// (threads tid of nt): the row evaluation of k_front, output for output.
__device__ __attribute__((always_inline)) inline void row_eval(const frame_desc& d, int ch, int y0, int n, int tid, int nt,
                                                               const double (*gy)[2][CBP_MAX_S], const c64* twS) {
  const int S = d.S;
  for (int o = tid; o < n * 2 * S; o += nt) {
    const int i = o / (2 * S), rest = o - i * 2 * S, fr = rest >= S, l = fr ? rest - S : rest;
    const int y = y0 + i * S;
    if (y < (fr ? d.H2 : d.H1)) d.ey[((size_t)(2 * ch + fr) * S + l) * d.Hmax + y] = dft_at(gy[i][fr], 1, twS, S, l);
  }
}

// Items: (channel, row group g, residue r): the rows y = g rpg + r + S i,
// i < rpg / S, y < Hmax, in increasing y.  Each row of both frames is packed
// as B1 + i B2 and transformed; while the rows pass, the workgroup folds them
// (the column fold of fold_item: the same rows of the same residue and
// group, summed in increasing y in FP64, hence the same bits) and writes
// the group's partial sums, so the frames are read once.  The unit-circle
// evaluation of both rows (fold modulo S and S-point DFT, as
// eval_rows_item: the same lanes, the same order, hence the same bits) is taken
// from the row in LDS; the DFTs of up to EY_ROWS rows run together, over all
// threads, instead of on 2 S of them while the row waits, with two barriers of
// their own (8 x 1080p RGB 255 -> 248 us, 16 x 720p 110 -> 105; without a switch
// to leave them out, and the register it spilled, 214 and 93).  The grid is
// persistent: a workgroup loads its next row into registers while it
// transforms the current one.
static_assert(CBP_MAX_FFT_F32 <= 8 * 256 && CBP_MAX_FFT_F64 <= 8 * 256, "one row is eight loads per thread");

constexpr int EY_ROWS = 8;

template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 2) void k_row_fwd(batch_ref br) {
  extern __shared__ __attribute__((aligned(16))) char sm_rf[];
  __shared__ double gy[EY_ROWS][2][CBP_MAX_S];
  __shared__ double fpart_l[2][128];
  __shared__ c64 twS[CBP_MAX_S];
  __shared__ int st[BATCH_CHUNK + 1];
  const int nf = br.nframes;
  const int* sq = br.starts + (size_t)Q_ROW_FWD * (nf + 1);
  for (int t = threadIdx.x; t <= nf; t += blockDim.x) st[t] = sq[t];
  __syncthreads();
  int first, end, step;
  xcd_items(__builtin_amdgcn_readfirstlane(st[nf]), (int)blockIdx.x, (int)gridDim.x, first, end, step);
  // frame of item it (st[fi] <= it < st[fi + 1]), wave-uniform
  auto frame_of = [&](int it) __attribute__((always_inline)) {
    int lo = 0, hi = nf;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (st[mid] <= it) lo = mid;
      else hi = mid;
    }
    return __builtin_amdgcn_readfirstlane(lo);
  };
  // descriptors are read-only while kernels run: reading them through the
  // constant address space with a wave-uniform index lets the scalar unit
  // load them into SGPRs
  auto desc = [&](int fi) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) frame_desc cdesc;
    return ((const cdesc*)br.descs)[fi];
#else
    return br.descs[fi];
#endif
  };
  // item it -> (channel, first row y0, rows of the item below Hmax)
  struct rows_of_item { int ch, g, r, y0, nv; };
  auto item_rows = [&](const frame_desc& d, int item) __attribute__((always_inline)) {
    const int S = d.S, RG = d.RG, gi = d.rpg / S;
    rows_of_item q;
    q.r = item % S;
    const int rest = item / S;
    q.g = rest % RG;
    q.ch = rest / RG;
    q.y0 = q.g * d.rpg + q.r;
    q.nv = q.y0 >= d.Hmax ? 0 : min(gi, (d.Hmax - 1 - q.y0) / S + 1);
    return q;
  };
  // the two rows y of channel ch into registers (fetch_rows)
  T uv[8], wv[8];
  auto fetch = [&](const frame_desc& d, int ch, int y) __attribute__((always_inline)) { fetch_rows<T>(d, ch, y, uv, wv); };
  // the first row of the first item at or after it that has rows (it >= end: none)
  auto fetch_from = [&](int it) __attribute__((always_inline)) {
    for (; it < end; it += step) {
      const int fi = frame_of(it);
      const frame_desc d = desc(fi);
      const rows_of_item q = item_rows(d, it - __builtin_amdgcn_readfirstlane(st[fi]));
      if (q.nv > 0) {
        fetch(d, q.ch, q.y0);
        return;
      }
    }
  };
  fetch_from(first);
  int tabN = 0;                  // plan of the pass tables in LDS (length,
  unsigned long long tabCode = 0;  // pass order)
  int tabS = 0;                  // S of the unit twiddles in twS
  for (int it = first; it < end; it += step) {
    const int fi = frame_of(it);
    const frame_desc d = desc(fi);
    const rows_of_item q = item_rows(d, it - __builtin_amdgcn_readfirstlane(st[fi]));
    const fft_plan& px = d.fx;
    const int N = px.N, S = d.S;
    cplx<T>* a = (cplx<T>*)sm_rf;
    cplx<T>* twf = a + N;
    const int ch = q.ch;
    // the column fold of this item's rows, both frames (FP64, increasing y)
    double f1[8], f2[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) f1[t] = f2[t] = 0.0;
    for (int i = 0; i < q.nv; ++i) {
      const int y = q.y0 + S * i;
      row_twiddles(a, twf, px, tabN, tabCode);
      if (S != tabS) {
        // w_t for the row evaluation (made again only when S changes: behind
        // the last item's evaluation, and the barrier after the row's store
        // orders it before its use)
        __syncthreads();
        row_unit_twiddles((__attribute__((address_space(3))) c64*)twS, S);
        tabS = S;
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int x = t * 256 + local_tid();
        f1[t] += (double)uv[t];
        f2[t] += (double)wv[t];
        if (x < N) a[x] = {uv[t], wv[t]};
      }
      __syncthreads();
      // the next row is in flight while this one is transformed
      if (i + 1 < q.nv) fetch(d, ch, y + S);
      else fetch_from(it + step);
      const int e = i % EY_ROWS;
      row_transform<T>(d, ch, y, a, twf, gy[e], fpart_l);
      if (e == EY_ROWS - 1 || i + 1 == q.nv) row_eval(d, ch, y - e * S, e + 1, threadIdx.x, 256, gy, twS);
    }
    // the group's column-fold partials (fold_item's layout), for x < W
    const auto fp1 = raw_buffer(d.fpart + (((size_t)q.g * d.ncf + 2 * ch) * S + q.r) * (size_t)d.Wmax, d.W1 * 8);
    const auto fp2 = raw_buffer(d.fpart + (((size_t)q.g * d.ncf + 2 * ch + 1) * S + q.r) * (size_t)d.Wmax, d.W2 * 8);
    const int off = local_tid() * 8;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      buf_store(fp1, off + t * 2048, f1[t]);
      buf_store(fp2, off + t * 2048, f2[t]);
    }
  }
}

// The split row pass, a call's first launch (a small call, see split_rows in
// api.hip): g.rows workgroups take single rows (channel, y), g.fold fold the
// columns from the frames themselves (k_front's fold, the same bits), g.twid
// fill the twiddle tables.  A row is a workgroup of its own instead of a
// turn of one residue's: 480x640 (168 items of three rows) 22.7 us and 4.7 for
// the launch before it -> 13.6 (12.2 since); 64x64 FP64 38.8 and 4.5 -> 8.4 (8.6).
template <typename T>
__global__ __launch_bounds__(256) void k_rows_front(batch_ref br_ws, front_grid g, inline_head ih) {
  extern __shared__ __attribute__((aligned(16))) char sm_rf[];
  __shared__ double gy[1][2][CBP_MAX_S];
  __shared__ double fpart_l[2][128];
  __shared__ c64 twS[CBP_MAX_S];
  const batch_ref br = first_launch_head(br_ws, ih);
  const int b = (int)blockIdx.x;
  if (b >= g.rows) {
    if (b < g.rows + g.fold)
      for_wave_items<Q_FOLD>(br, b - g.rows, g.fold, [&](const frame_desc& d, int item, int lane)
                                                         __attribute__((always_inline)) { fold_item<T>(d, item, lane); });
    else
      for_items_part<Q_TWID>(br, b - g.rows - g.fold, g.twid,
                             [&](const frame_desc& d, int item) __attribute__((always_inline)) { twiddle_item(d, item); });
    return;
  }
  int tabN = 0, tabS = 0;
  unsigned long long tabCode = 0;
  for_items_part<Q_ROWS>(br, b, g.rows, [&](const frame_desc& d, int item) __attribute__((always_inline)) {
    const int N = d.fx.N, ch = item / d.Hmax, y = item - ch * d.Hmax;
    cplx<T>* a = (cplx<T>*)sm_rf;
    cplx<T>* twf = a + N;
    T uv[8], wv[8];
    fetch_rows<T>(d, ch, y, uv, wv);
    row_twiddles(a, twf, d.fx, tabN, tabCode);
    if (d.S != tabS) {
      __syncthreads();   // the last item's evaluation reads twS
      row_unit_twiddles((__attribute__((address_space(3))) c64*)twS, d.S);
      tabS = d.S;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int x = t * 256 + local_tid();
      if (x < N) a[x] = {uv[t], wv[t]};
    }
    __syncthreads();
    row_transform<T>(d, ch, y, a, twf, gy[0], fpart_l);
    row_eval(d, ch, y, 1, threadIdx.x, 256, gy, twS);
  });
}

// ---------------------------------------------------------------- pass 2
// The column pass keeps one strip of cw columns (cw up to 8: row
// segments of up to 64 bytes, 128 in FP64) in LDS, column-major with an odd leading dimension, and
// transforms it in place.  One buffer per strip instead of two frames'
// ping-pong pairs is what makes wide strips fit; frame 2's spectrum waits in
// registers while frame 1 is transformed.  The workgroup has NT = 256 or 512
// threads.

// Column stride of a strip in LDS: the smallest ld >= N whose residue modulo
// the entries of one 128-byte bank row (16 FP32 / 8 FP64 complex) is that
// count over cw (1 when cw is larger).  The row segments the strip is loaded
// from and stored to (cw columns of consecutive rows on consecutive lanes)
// then fall in distinct banks.
template <typename T>
__host__ __device__ inline int col_ld(int N, int cw) {
  constexpr int B = 128 / (int)sizeof(cplx<T>);
  const int t = cw < B ? B / cw : 1;
  return N + (((t - N) % B) + B) % B;
}

// Largest cw * N of a strip: 9 FP32 (4.5 FP64) complex entries per thread,
// so each thread's share of a pass and of the stashed spectrum stays in
// registers.
template <typename T, int NT>
constexpr int col_max_elems() { return NT * 72 / (int)sizeof(cplx<T>); }


// The strip's entries as each thread holds them for the stash and the
// filter: column c = tid / (NT / cw) (wave-uniform: NT / cw >= 64) and rows in
// groups of g = 4, 5, 7, 3 or 1 (g divides N): rows y + j N/g, j < g,
// y = tid mod (NT / cw) + i NT / cw < N/g, whose twiddles w_N^(y + j N/g)
// differ by the g-th roots of unity.  Group i holds slots g i .. g i + g - 1.
template <typename T, int NT, int G>
constexpr int col_groups() { return (col_max_elems<T, NT>() / G + NT - 1) / NT; }

// Entries of one kernel's row DFTs at one column in LDS: CBP_MAX_K and zeros for
// the last coefficients of a group's polynomials (a multiple of g <= 7 past k).
constexpr int KR_LD = CBP_MAX_K + 4;
static_assert((CBP_MAX_K + 6) / 7 * 7 <= KR_LD && (CBP_MAX_K + 4) / 5 * 5 <= KR_LD && (CBP_MAX_K + 2) / 3 * 3 <= KR_LD &&
                  (CBP_MAX_K + 3) / 4 * 4 <= KR_LD, "group padding");

// The kernels' row DFTs at columns kx0 .. kx0 + cw into kr [cw][2][KR_LD], zero
// past hx and past each kernel's rows: k_kernel_dft's sums.  at: LDS for the
// kernels and the columns' twiddles.  (A call: inlined, it costs the column pass
// of every launch some five registers.)
template <typename T, int NT>
__device__ __attribute__((noinline)) void own_row_dfts(__attribute__((address_space(3))) char* at,
                                                       __attribute__((address_space(3))) cplx<T>* kr, const double* K1,
                                                       const double* K2, const c64* twd, int k1, int k2, int Px, int hx,
                                                       int kx0, int cw) {
  typedef __attribute__((address_space(3))) double lds_d;
  const int n1 = k1 * k1, nk = n1 + k2 * k2;
  lds_d* Kl = (lds_d*)at;                    // K1, K2
  lds_d* wl = Kl + ((nk + 1) & ~1);          // [cw][CBP_MAX_K] w_Px^(kx x), re and im
  for (int e = threadIdx.x; e < nk; e += NT) Kl[e] = e < n1 ? K1[e] : K2[e - n1];
  for (int e = threadIdx.x; e < cw * CBP_MAX_K; e += NT) {
    const int c = e / CBP_MAX_K, x = e - c * CBP_MAX_K;
    const c64 w = twd[min(kx0 + c, hx - 1) * x % Px];
    wl[2 * e] = w.re;
    wl[2 * e + 1] = w.im;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < cw * 2 * KR_LD; e += NT) {
    const int row = e / KR_LD, yy = e - row * KR_LD, c = row >> 1;   // row = 2 column + kernel
    const int k = row & 1 ? k2 : k1;
    double sr = 0.0, si = 0.0;
    if (yy < k && kx0 + c < hx) {
      lds_d* kv = Kl + (row & 1 ? n1 : 0) + yy * k;
      lds_d* w = wl + 2 * c * CBP_MAX_K;
      for (int x = 0; x < k; ++x) {
        sr += kv[x] * w[2 * x];
        si += kv[x] * w[2 * x + 1];
      }
    }
    kr[e].re = T(sr);
    kr[e].im = T(si);
  }
}

// Items: (strip of cw columns, channel).  A workgroup that owns several
// items loads the next strip (and frame 1's strip of the current item) into
// registers while it transforms.
// G: rows per group of the filter's kernel-spectrum evaluation.  A launch
// takes the items of the frames whose group (col_group_size of their N) is
// G and passes over the others, which a launch with their G takes: each
// frame is filtered with its own group whatever the batch, and a
// compile-time group keeps the stashed spectrum's slots compile-time
// indices, in registers.
template <typename T, int NT, int G>
__global__ __launch_bounds__(NT, sizeof(T) == 4 ? 4 : 2) void k_col_filter(batch_ref br, int own) {
  extern __shared__ __attribute__((aligned(16))) char sm_cf[];
  __shared__ int st[BATCH_CHUNK + 1];
  constexpr int SM = G * col_groups<T, NT, G>();
  constexpr int PF = (col_max_elems<T, NT>() + NT - 1) / NT;   // strip entries per thread
  constexpr int LNT = NT == 512 ? 9 : 8;
  __shared__ int s_next[2];   // the workgroup's next items (thread 0 takes them), alternate slots
  const int nf = br.nframes;
  const int* sq = br.starts + (size_t)Q_COL * (nf + 1);
  for (int t = threadIdx.x; t <= nf; t += NT) st[t] = sq[t];
  __syncthreads();
  // items handed out dynamically from this group's counters (dyn_items);
  // with no more items than workgroups, one item per workgroup as
  // xcd_items assigns them (a workgroup that took two, one ahead, would
  // leave another idle)
  const int ntot = __builtin_amdgcn_readfirstlane(st[nf]);
  const bool dyn = ntot > (int)gridDim.x;
  const dyn_items q = make_dyn_items(br.ctr + CTR_COL + 8 * col_group_index(G), ntot, (int)blockIdx.x,
                                     (int)gridDim.x);
  const int end = q.hi;
  auto frame_of = [&](int it) __attribute__((always_inline)) {
    int lo = 0, hi = nf;   // st[lo] <= it < st[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (st[mid] <= it) lo = mid;
      else hi = mid;
    }
    return __builtin_amdgcn_readfirstlane(lo);
  };
  auto desc = [&](int fi) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) frame_desc cdesc;
    return ((const cdesc*)br.descs)[fi];
#else
    return br.descs[fi];
#endif
  };
  // frame fr's strip of item it into registers: column c = tid mod cw (cw
  // consecutive threads read one row segment), rows tid / cw + i NT / cw;
  // zero in rows past the frame and columns past hx
  cplx<T> pre[PF];
  auto fetch = [&](int it, int fr) __attribute__((always_inline)) {
    const int fi = frame_of(it);
    const frame_desc d = desc(fi);
    const int item = it - __builtin_amdgcn_readfirstlane(st[fi]);
    const int cw = d.cw, hx = d.hx, tp = d.hxp, lcw = __builtin_ctz(cw);
    const int nstrip = (hx + cw - 1) / cw;
    const int kx0 = (item % nstrip) * cw, ch = item / nstrip;
    const auto src = raw_buffer((const cplx<T>*)(fr ? d.t2 : d.t1) + ch * (int64_t)d.Hmax * tp + kx0,
                                ((fr ? d.H2 : d.H1) * tp - kx0) * (int)sizeof(cplx<T>));
    const int tid = local_tid();
    const int c = tid & (cw - 1);
    const int off = kx0 + c < hx ? (mul24(tid >> lcw, tp) + c) * (int)sizeof(cplx<T>) : kPastEnd;
    const int step = (NT >> lcw) * tp * (int)sizeof(cplx<T>);
#pragma unroll
    for (int i = 0; i < PF; ++i) pre[i] = buf_load<cplx<T>>(src, off + i * step);
  };
  auto first_frame = [&](int it) __attribute__((always_inline)) {
    return (desc(frame_of(it)).variant & VAR_DIVIDE_B1) ? 0 : 1;   // frame 2 first when both are divided
  };
  // Thread 0: from the item raw taken (its counter value, whose atomic may
  // still be in flight), the first item of a frame with group G (end: none;
  // the items of other groups are passed over, their launch has its own
  // counters).
  auto settle = [&](int raw) __attribute__((always_inline)) {
    int i = raw;
    while (i < end && col_group_size(desc(frame_of(i)).fy.N) != G) i = dyn ? q.take() : end;
    return i;
  };
  // one item ahead: the counter value taken while an item is processed is
  // read only when the next one starts, so the atomic's latency is hidden
  int ahead = end;
  if (threadIdx.x == 0) {
    if (dyn) {
      s_next[0] = settle(q.take());
      ahead = q.lo + atomicAdd(q.ctr, 1);
    } else {
      int first, last, step;
      xcd_items(ntot, (int)blockIdx.x, (int)gridDim.x, first, last, step);
      s_next[0] = settle(first < last ? first : end);
    }
  }
  __syncthreads();
  const int it0 = __builtin_amdgcn_readfirstlane(s_next[0]);
  if (it0 < end) fetch(it0, first_frame(it0));
  int tabN = 0;                     // plan of the tables in LDS (length,
  unsigned long long tabCode = 0;   // pass order)
  for (int it = it0, nit, par = 1; it < end; it = nit, par ^= 1) {
    // the item after this one, read by every thread after the next barrier
    // (slot par: its last reads were two items ago)
    if (threadIdx.x == 0) {
      s_next[par] = settle(ahead < end ? ahead : end);
      ahead = dyn ? q.lo + atomicAdd(q.ctr, 1) : end;
    }
    const int fi = frame_of(it);
    const frame_desc d = desc(fi);
    const int item = it - __builtin_amdgcn_readfirstlane(st[fi]);
    const fft_plan& py = d.fy;
    const int N = py.N, cw = d.cw, hx = d.hx, tp = d.hxp, m = d.m;
    const int ld = col_ld<T>(N, cw);
    const int k1 = d.k1, k2 = d.k2;
    const T lam = (T)d.lambda;
    const bool two = !(d.variant & VAR_DIVIDE_B1);   // two-channel division, or B1 / K1 alone
    cplx<T>* buf = (cplx<T>*)sm_cf;                   // [cw][ld]
    cplx<T>* kr = buf + (size_t)cw * ld;              // [cw][2][KR_LD] row DFTs of the kernels at kx
    cplx<T>* tw = kr + (size_t)cw * 2 * KR_LD;        // [N] w_N^t (the filter's kernel spectra)
    // the filter's row groups (see col_groups) and its w_N^(G y), y < N / G
    cplx<T>* twg = tw + N;
    cplx<T>* twp = G > 1 ? twg + N / G : twg;         // the plan's pass tables
    const int nstrip = (hx + cw - 1) / cw;
    const int kx0 = (item % nstrip) * cw, ch = item / nstrip;
    const int lcw = __builtin_ctz(cw);                // cw is a power of two
    // the registers' strip into buf[c ld + y]
    auto spill = [&]() __attribute__((always_inline)) {
      const int tid = local_tid();
      const int y = tid >> lcw, ys = NT >> lcw;
      cplx<T>* at = buf + mul24(tid & (cw - 1), ld) + y;
#pragma unroll
      for (int i = 0; i < PF; ++i)
        if (y + i * ys < N) at[i * ys] = pre[i];
    };
    // the tables, when those in LDS are another plan's (the last item's reads
    // of them are behind its closing barrier)
    if (tabN != N || tabCode != py.code) {
      full_twiddles<T>((__attribute__((address_space(3))) cplx<T>*)tw, N, NT);
      __syncthreads();
      if (G > 1)
        for (int y = threadIdx.x; y < N / G; y += NT) twg[y] = tw[G * y];
      pass_twiddles(twp, tw, py, NT);
      tabN = N;
      tabCode = py.code;
    }
    // the kernels' row DFTs at this strip's columns, zero past hx: from
    // k_kernel_dft, or (own: the place in LDS of the kernels and the columns'
    // twiddles) formed here, the same sums
    if (own) {
      own_row_dfts<T, NT>((__attribute__((address_space(3))) char*)(sm_cf + own), (__attribute__((address_space(3))) cplx<T>*)kr,
                          d.K1, d.K2, d.twxd, k1, k2, d.Px, hx, kx0, cw);
    } else {
      const cplx<T>* krg = (const cplx<T>*)d.kr;
      for (int e = threadIdx.x; e < cw * 2 * KR_LD; e += NT) {
        const int row = e / KR_LD, yy = e - row * KR_LD;   // row = 2 column + kernel
        kr[e] = kx0 + (row >> 1) < hx && yy < CBP_MAX_K ? krg[((size_t)kx0 * 2 + row) * CBP_MAX_K + yy]
                                                        : cplx<T>{T(0), T(0)};
      }
    }
    // the entries this thread holds (see col_groups): f(group size, slot of
    // the group's first row, column, y, N / group size)
    auto for_held = [&](auto&& f) __attribute__((always_inline)) {
      const int tid = local_tid();
      const int ltpc = LNT - lcw;
      const int c = tid >> ltpc, r = tid & ((1 << ltpc) - 1);
      const int q = N / G;
#pragma unroll
      for (int i = 0; i < col_groups<T, NT, G>(); ++i) {
        const int y = r + (i << ltpc);
        if (y < q) f(std::integral_constant<int, G>(), G * i, c, y, q);
      }
    };
    cplx<T> st2[SM];
#pragma unroll
    for (int j = 0; j < SM; ++j) any_value(st2[j]);
    if (two) {
      spill();
      __syncthreads();
      fetch(it, 0);   // frame 1's strip in flight while frame 2's is transformed
      ip_fft<-1, NT, col_max_elems<T, NT>()>(buf, ld, py, twp, lcw);
      for_held([&](auto GC, int a, int c, int y, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < GC(); ++j) st2[a + j] = buf[mul24(c, ld) + y + j * q];
      });
      __syncthreads();   // buf is refilled with frame 1
    }
    spill();
    __syncthreads();
    ip_fft<-1, NT, col_max_elems<T, NT>()>(buf, ld, py, twp, lcw);
    // filter: the combined spectrum in place of frame 1's
    const int kmax = k1 > k2 ? k1 : k2;
    auto filt = [&](cplx<T>* at, const cplx<T>& kh1, const cplx<T>& kh2, const cplx<T>& b2)
        __attribute__((always_inline)) {
      const cplx<T> B1 = *at;
      const cplx<T> num = two ? cmulc(kh1, B1) + cmulc(kh2, b2) : cmulc(kh1, B1);
      const T kk = two ? norm2(kh1) + norm2(kh2) : norm2(kh1);
      const T den = kk + lam;
      const T inv = den > T(0) ? T(1) / den : T(0);
      // where both kernel spectra vanish (a zeroed kernel pair) the
      // quotient is zero, whatever the frames hold
      *at = kk > T(0) ? cplx<T>{num.re * inv, num.im * inv} : cplx<T>{T(0), T(0)};
    };
    for_held([&](auto GC, int a, int c, int y, int q) __attribute__((always_inline)) {
      // kernel spectra at (ky, kx) = sum_yy kr[yy] z^yy, z = w_N^ky.  For the
      // group's rows ky = y + j N/g (z = w_N^y times the g-th roots of unity
      // w_g^j): K = sum_p z^p E_p(z^g), E_p(u) = sum_t kr[g t + p] u^t
      // by Horner's rule in u = w_N^(g y), then the g-point DFT of the
      // z^p E_p.  kr is zero beyond each kernel's size; the column is
      // wave-uniform.
      constexpr int g = GC();
      const cplx<T>* kr1 = kr + c * 2 * KR_LD;
      const cplx<T>* kr2 = kr1 + KR_LD;
      const int nt = (kmax + g - 1) / g;          // coefficients per E_p
      const cplx<T> u = g == 1 ? tw[y] : twg[y];
      cplx<T> P1[g], P2[g];
#pragma unroll
      for (int p = 0; p < g; ++p) {
        P1[p] = kr1[g * (nt - 1) + p];
        P2[p] = kr2[g * (nt - 1) + p];
      }
      for (int t = nt - 2; t >= 0; --t) {
#pragma unroll
        for (int p = 0; p < g; ++p) {
          P1[p] = P1[p] * u + kr1[g * t + p];
          P2[p] = P2[p] * u + kr2[g * t + p];
        }
      }
#pragma unroll
      for (int p = 1; p < g; ++p) {
        const cplx<T> zp = tw[p * y];
        P1[p] = zp * P1[p];
        P2[p] = zp * P2[p];
      }
      cplx<T>* col = buf + mul24(c, ld) + y;
      if constexpr (g > 1) {
        dft_small<g, -1>(P1);
        dft_small<g, -1>(P2);
      }
#pragma unroll
      for (int j = 0; j < g; ++j, col += q) filt(col, P1[j], P2[j], st2[a + j]);
    });
    __syncthreads();
    // the next item's first strip in flight during the inverse transform (not
    // earlier: its registers and the stashed spectrum's are never both held)
    nit = __builtin_amdgcn_readfirstlane(s_next[par]);
    if (nit < end) fetch(nit, first_frame(nit));
    ip_fft<+1, NT, col_max_elems<T, NT>()>(buf, ld, py, twp, lcw);
    // the first m rows, row segments of cw columns
    {
      const auto uo = raw_buffer((cplx<T>*)d.u + ch * (int64_t)m * tp + kx0, (m * tp - kx0) * (int)sizeof(cplx<T>));
      const int tid = local_tid();
      const int c = tid & (cw - 1), y = tid >> lcw, ys = NT >> lcw;
      const int off = kx0 + c < hx ? (mul24(y, tp) + c) * (int)sizeof(cplx<T>) : kPastEnd;
      const int step = ys * tp * (int)sizeof(cplx<T>);
      const cplx<T>* at = buf + mul24(c, ld) + y;
#pragma unroll
      for (int i = 0; i < PF; ++i)
        if (y + i * ys < m) buf_store(uo, off + i * step, at[i * ys]);
    }
    __syncthreads();   // the next item refills buf, kr and tw
  }
}

// ---------------------------------------------------------------- kernel row DFTs
// kr[kx][fr][yy] = sum_x K_fr[yy][x] exp(-2 pi i kx x / Px) for every
// half-spectrum column kx < hx (zero for yy >= k_fr), in FP64 from the FP64
// twiddle table, rounded once to T: the column pass evaluates each kernel's
// spectrum at (ky, kx) from these along y.  Once per frame, shared by its
// channels; a call whose strips all run at once forms them in its column pass
// instead (see own_kr_bytes in api.hip).  Items: 256 consecutive entries of [0, hx * 2 * CBP_MAX_K).
static_assert(2 * CBP_MAX_K == 64, "one column's entries fill one wave");

template <typename T>
__global__ __launch_bounds__(256) void k_kernel_dft(batch_ref br) {
  for_items<Q_KRDFT>(br, [&](const frame_desc& d, int item) __attribute__((always_inline)) {
    const int e = item * 256 + (int)threadIdx.x;
    const int hx = d.hx, Px = d.Px;
    if (e >= hx * 2 * CBP_MAX_K) return;
    // a wave's 64 entries share one column kx (2 CBP_MAX_K = 64): its
    // twiddles are wave-uniform (scalar loads)
    const int kx = __builtin_amdgcn_readfirstlane(e / (2 * CBP_MAX_K)), rem = e - kx * 2 * CBP_MAX_K;
    const int fr = rem / CBP_MAX_K, yy = rem - fr * CBP_MAX_K;
    const int k = fr ? d.k2 : d.k1;
    const double* K = fr ? d.K2 : d.K1;
    const c64* twd = d.twxd;
    double sr = 0.0, si = 0.0;
    if (yy < k) {
      // eight (twiddle, coefficient) pairs loaded per batch, summed in x order
      int t = 0;
      for (int x0 = 0; x0 < k; x0 += 8) {
        c64 w[8];
        double kv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          w[u] = twd[t];
          kv[u] = K[yy * k + min(x0 + u, k - 1)];
          t += kx;
          if (t >= Px) t -= Px;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (x0 + u < k) {
            sr += kv[u] * w[u].re;
            si += kv[u] * w[u].im;
          }
      }
    }
    ((cplx<T>*)d.kr)[e] = {T(sr), T(si)};
  });
}

// ---------------------------------------------------------------- pass 3
// Items: (pair of output rows, channel).  A workgroup that owns several items
// loads the next item's spectra into registers while it transforms the
// current one.
template <typename T>
__global__ __launch_bounds__(256) void k_row_inv(batch_ref br) {
  extern __shared__ __attribute__((aligned(16))) char sm_ri[];
  __shared__ int st[BATCH_CHUNK + 1];
  const int nf = br.nframes;
  const int* sq = br.starts + (size_t)Q_ROW_INV * (nf + 1);
  for (int t = threadIdx.x; t <= nf; t += blockDim.x) st[t] = sq[t];
  __syncthreads();
  int first, end, step;
  xcd_items(__builtin_amdgcn_readfirstlane(st[nf]), (int)blockIdx.x, (int)gridDim.x, first, end, step);
  auto frame_of = [&](int it) __attribute__((always_inline)) {
    int lo = 0, hi = nf;   // st[lo] <= it < st[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (st[mid] <= it) lo = mid;
      else hi = mid;
    }
    return __builtin_amdgcn_readfirstlane(lo);
  };
  auto desc = [&](int fi) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) frame_desc cdesc;
    return ((const cdesc*)br.descs)[fi];
#else
    return br.descs[fi];
#endif
  };
  // the half spectra of item it's two rows into registers, entries
  // t 256 + tid < hx (the second row is zero past the last)
  cplx<T> Av[ROW_HALF], Bv[ROW_HALF];
  auto fetch = [&](int it) __attribute__((always_inline)) {
    const int fi = frame_of(it);
    const frame_desc d = desc(fi);
    const int item = it - __builtin_amdgcn_readfirstlane(st[fi]);
    const int m = d.m, row = d.hx * (int)sizeof(cplx<T>);
    const int npair = (m + 1) / 2;
    const int ya = 2 * (item % npair), ch = item / npair;
    const cplx<T>* ua = (const cplx<T>*)d.u + (int64_t)ch * m * d.hxp + (int64_t)ya * d.hxp;
    const bool hb = ya + 1 < m;
    const auto ra = raw_buffer(ua, row), rb = raw_buffer(hb ? ua + d.hxp : ua, hb ? row : 0);
    const int off = local_tid() * (int)sizeof(cplx<T>);
#pragma unroll
    for (int t = 0; t < ROW_HALF; ++t) {
      Av[t] = buf_load<cplx<T>>(ra, off + t * 256 * (int)sizeof(cplx<T>));
      Bv[t] = buf_load<cplx<T>>(rb, off + t * 256 * (int)sizeof(cplx<T>));
    }
  };
  if (first < end) fetch(first);
  int tabN = 0;                  // plan of the pass tables in LDS (length,
  unsigned long long tabCode = 0;  // pass order)
  for (int it = first; it < end; it += step) {
    const int fi = frame_of(it);
    const frame_desc d = desc(fi);
    const int item = it - __builtin_amdgcn_readfirstlane(st[fi]);
    const fft_plan& px = d.fx;
    const int N = px.N, hx = d.hx, m = d.m, n = d.n;
    const T scale = (T)(1.0 / ((double)d.Py * (double)d.Px));
    cplx<T>* a = (cplx<T>*)sm_ri;
    cplx<T>* twf = a + N;
    row_twiddles(a, twf, px, tabN, tabCode);
    const int npair = (m + 1) / 2;
    const int ya = 2 * (item % npair), yb = ya + 1, ch = item / npair;
    const bool hb = yb < m;
    // A + i B at k and, from the conjugates, at N - k
#pragma unroll
    for (int t = 0; t < ROW_HALF; ++t) {
      const int k = t * 256 + local_tid();
      if (k < hx) {
        cplx<T> A = Av[t], B = Bv[t];
        if ((k == 0) || (2 * k == N)) { A.im = T(0); B.im = T(0); }
        a[k] = {A.re - B.im, A.im + B.re};
        if (k > 0) a[N - k] = {A.re + B.im, B.re - A.im};
      }
    }
    __syncthreads();
    // the next item's spectra are in flight while this one is transformed
    if (it + step < end) fetch(it + step);
    ip_fft<+1, 256, ROW_MAXE>(a, N, px, twf, 0);
    const cplx<T>* z = a;
    T* oa = (T*)d.out + ch * d.ocs + (int64_t)ya * d.opitch;
    const auto ba = raw_buffer(oa, n * (int)sizeof(T)), bb = raw_buffer(hb ? oa + d.opitch : oa, hb ? n * (int)sizeof(T) : 0);
    for (int x = threadIdx.x; x < n; x += 256) {
      const int off = x * (int)sizeof(T);
      buf_store(ba, off, z[x].re * scale);
      buf_store(bb, off, z[x].im * scale);
    }
    __syncthreads();
  }
}

}  // namespace

// a row and the plan's pass twiddle tables (twn entries)
size_t row_lds_bytes(int N, int twn, int esize) { return ((size_t)N + (size_t)twn) * 2 * esize; }
// the strip (column stride col_ld <= N + 15), the kernels' row DFTs, the
// full twiddle table and twn more entries (col_table_entries: the filter's
// w_N^(g y) and the plan's pass twiddle tables)
size_t col_lds_bytes(int N, int cw, int twn, int esize) {
  return ((size_t)cw * (N + 15) + (size_t)cw * 2 * KR_LD + (size_t)N + (size_t)twn) * 2 * esize;
}

// Threads of the column-pass workgroup for a strip of cw * N entries: 256 when
// its registers hold the strip with at least one wave per column, else 512.
int col_threads(int N, int cw, int esize) {
  const int l256 = esize == 4 ? col_max_elems<float, 256>() : col_max_elems<double, 256>();
  return cw <= 4 && (int64_t)cw * N <= l256 ? 256 : 512;
}

int col_max_strip_elems(int esize) { return esize == 4 ? col_max_elems<float, 512>() : col_max_elems<double, 512>(); }

// Resident forward or inverse row-pass workgroups per CU (its registers and lds
// bytes of LDS), for the persistent grid: a workgroup beyond that would start
// only when another ends and leave a tail, fewer leave the CU's waits unfilled
// (inverse rows, four a CU / as many as fit: 16 x 720p 40.2 / 36.8 us, six a CU;
// 16 x 256x256 12.3 / 11.6).
// Kept per (direction, element size, LDS in 4 KiB steps).
int row_per_cu(bool inverse, size_t lds, int esize) {
  static std::atomic<int> cache[2][2][41];
  const int b = std::min((int)((lds + 4095) / 4096), 40);
  std::atomic<int>& c = cache[inverse][esize == 8][b];
  int n = c.load(std::memory_order_relaxed);
  if (n > 0) return n;
  const void* f = inverse ? (esize == 8 ? (const void*)k_row_inv<double> : (const void*)k_row_inv<float>)
                          : (esize == 8 ? (const void*)k_row_fwd<double> : (const void*)k_row_fwd<float>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 256, (size_t)b * 4096) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    return 1;
  }
  c.store(n, std::memory_order_relaxed);
  return n;
}

// Resident column-pass workgroups per CU for strips of cw columns of length
// N (its variant's registers and LDS), for the persistent grid.  Kept per
// (element size, variant, LDS in 4 KiB steps).
// The column-pass instance of element type T, workgroup size nt and filter
// group g.
template <typename T, int NT>
const void* col_kernel_of(int g) {
  return g == 4 ? (const void*)k_col_filter<T, NT, 4> : g == 5 ? (const void*)k_col_filter<T, NT, 5>
         : g == 7 ? (const void*)k_col_filter<T, NT, 7> : g == 3 ? (const void*)k_col_filter<T, NT, 3>
                                                                 : (const void*)k_col_filter<T, NT, 1>;
}

template <typename T>
const void* col_kernel(int nt, int g) {
  return nt == 256 ? col_kernel_of<T, 256>(g) : col_kernel_of<T, 512>(g);
}

int col_per_cu(int N, int cw, int twn, int g, int esize) {
  static std::atomic<int> cache[2][2][5][41];
  const int nt = col_threads(N, cw, esize);
  const int b = std::min((int)((col_lds_bytes(N, cw, twn, esize) + 4095) / 4096), 40);
  std::atomic<int>& c = cache[esize == 8][nt == 512][col_group_index(g)][b];
  int n = c.load(std::memory_order_relaxed);
  if (n > 0) return n;
  const void* f = esize == 8 ? col_kernel<double>(nt, g) : col_kernel<float>(nt, g);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, nt, (size_t)b * 4096) != hipSuccess ||
      n < 1) {
    (void)hipGetLastError();
    return 1;
  }
  c.store(n, std::memory_order_relaxed);
  return n;
}

void set_fft_attrs() {
  const void* fns[] = {(const void*)k_row_fwd<float>,  (const void*)k_row_inv<float>,  (const void*)k_rows_front<float>,
                       (const void*)k_row_fwd<double>, (const void*)k_row_inv<double>, (const void*)k_rows_front<double>};
  for (const void* f : fns) hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  for (int nt : {256, 512})
    for (int g : COL_GROUPS) {
      hipFuncSetAttribute(col_kernel<float>(nt, g), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      hipFuncSetAttribute(col_kernel<double>(nt, g), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    }
}

template <typename T>
hipError_t launch_row_fwd(const batch_ref& br, int grid, int maxPx, int maxTw, hipStream_t st) {
  prof_begin(PH_ROW_FWD, st);
  hipLaunchKernelGGL(k_row_fwd<T>, dim3(grid), dim3(256), row_lds_bytes(maxPx, maxTw, (int)sizeof(T)), st, br);
  prof_end(PH_ROW_FWD, st);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_col(const batch_ref& br, int grid, int maxPy, int maxcw, int maxTw, int gmask, int ownBytes,
                      hipStream_t st) {
  prof_begin(PH_COL_FILTER, st);
  const size_t strip = (col_lds_bytes(maxPy, maxcw, maxTw, (int)sizeof(T)) + 15) & ~(size_t)15, lds = strip + ownBytes;
  const int nt = col_threads(maxPy, maxcw, (int)sizeof(T));
  int own = ownBytes ? (int)strip : 0;
  void* args[] = {(void*)&br, (void*)&own};
  hipError_t e = hipSuccess;
  for (int g : COL_GROUPS)
    if ((gmask >> g & 1) && e == hipSuccess) e = hipLaunchKernel(col_kernel<T>(nt, g), dim3(grid), dim3(nt), args, lds, st);
  prof_end(PH_COL_FILTER, st);
  return e != hipSuccess ? e : hipGetLastError();
}

template <typename T>
hipError_t launch_kernel_dft(const batch_ref& br, int grid, hipStream_t st) {
  prof_begin(PH_KR_DFT, st);
  hipLaunchKernelGGL(k_kernel_dft<T>, dim3(grid), dim3(256), 0, st, br);
  prof_end(PH_KR_DFT, st);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_row_inv(const batch_ref& br, int grid, int maxPx, int maxTw, hipStream_t st) {
  prof_begin(PH_ROW_INV, st);
  hipLaunchKernelGGL(k_row_inv<T>, dim3(grid), dim3(256), row_lds_bytes(maxPx, maxTw, (int)sizeof(T)), st, br);
  prof_end(PH_ROW_INV, st);
  return hipGetLastError();
}


template <typename T>
hipError_t launch_rows_front(const batch_ref& br, const front_grid& g, int maxPx, int maxTw, const inline_head* ih,
                             hipStream_t st) {
  prof_begin(PH_ROW_FWD, st);
  inline_head h;
  if (ih) h = *ih;
  else h.ndesc_bytes = h.nstart_bytes = 0;
  hipLaunchKernelGGL(k_rows_front<T>, dim3(g.rows + g.fold + g.twid), dim3(256),
                     row_lds_bytes(maxPx, maxTw, (int)sizeof(T)), st, br, g, h);
  prof_end(PH_ROW_FWD, st);
  return hipGetLastError();
}

template hipError_t launch_rows_front<float>(const batch_ref&, const front_grid&, int, int, const inline_head*,
                                             hipStream_t);
template hipError_t launch_rows_front<double>(const batch_ref&, const front_grid&, int, int, const inline_head*,
                                              hipStream_t);
template hipError_t launch_row_fwd<float>(const batch_ref&, int, int, int, hipStream_t);
template hipError_t launch_row_fwd<double>(const batch_ref&, int, int, int, hipStream_t);
template hipError_t launch_col<float>(const batch_ref&, int, int, int, int, int, int, hipStream_t);
template hipError_t launch_col<double>(const batch_ref&, int, int, int, int, int, int, hipStream_t);
template hipError_t launch_kernel_dft<float>(const batch_ref&, int, hipStream_t);
template hipError_t launch_kernel_dft<double>(const batch_ref&, int, hipStream_t);
template hipError_t launch_row_inv<float>(const batch_ref&, int, int, int, hipStream_t);
template hipError_t launch_row_inv<double>(const batch_ref&, int, int, int, hipStream_t);

}  // namespace cbp
