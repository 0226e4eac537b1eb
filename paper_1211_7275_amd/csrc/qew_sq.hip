// qew_sq.hip -- structure factor S_q(t) of Eq. (6) of arXiv:1211.7275.
//
//   S_n = | L^-1 sum_x u_x exp(-i 2 pi n x / L) |^2,  q = 2 pi n / L,
//
// for every sample of a batch of equal power-of-two lengths L, in FP64, at a
// measurement step.  For real u the modes n and L - n are equal, so n = 1 ..
// L/2 is produced.  The real transform of length L is one complex transform
// of length N = L/2 on z_k = u_2k + i u_2k+1 (after subtracting the sample's
// first site, which only moves mode 0), followed by the usual split of the
// even and odd halves.
//   - Up to kSmallN points (64 KB) the whole transform of a sample stays in the
//     LDS of one workgroup (k_sq_small): one kernel from the chain to |U_n|^2.
//   - Longer ones are Stockham auto-sort passes of radix 32, 64 or 128
//     (k_fft_wide), the first reading the chain, the last forming |U_n|^2 and
//     its sum over the samples: the batch crosses the memory once per pass, and
//     L = 2^22 takes three.
// Twiddles come from sincospi in FP64.  The per-mode sums are then averaged
// over the samples and over caller-given ranges of n (cut into chunks of
// modes), in a fixed order (no atomics), so repeated runs give identical bits.
#include "qew_internal.hpp"

namespace qew {

namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// multiply by -i
__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }

// In-register DFT of R points: X_q = sum_r v_r exp(-2 pi i r q / R).
template <int R>
__device__ __forceinline__ void dft(double2* v);

template <>
__device__ __forceinline__ void dft<2>(double2* v) {
  const double2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <>
__device__ __forceinline__ void dft<4>(double2* v) {
  const double2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
  const double2 s13 = cadd(v[1], v[3]), d13 = mul_mi(csub(v[1], v[3]));
  v[0] = cadd(s02, s13);
  v[1] = cadd(d02, d13);
  v[2] = csub(s02, s13);
  v[3] = csub(d02, d13);
}

template <>
__device__ __forceinline__ void dft<8>(double2* v) {
  // radix-4 transforms of the even and odd points, then one radix-2 layer
  double2 e[4] = {v[0], v[2], v[4], v[6]};
  double2 o[4] = {v[1], v[3], v[5], v[7]};
  dft<4>(e);
  dft<4>(o);
  constexpr double h = 0.70710678118654752440;  // 1/sqrt(2)
  const double2 w1 = make_double2(h, -h), w3 = make_double2(-h, -h);
  const double2 t0 = o[0], t1 = cmul(o[1], w1), t2 = mul_mi(o[2]), t3 = cmul(o[3], w3);
  v[0] = cadd(e[0], t0);
  v[4] = csub(e[0], t0);
  v[1] = cadd(e[1], t1);
  v[5] = csub(e[1], t1);
  v[2] = cadd(e[2], t2);
  v[6] = csub(e[2], t2);
  v[3] = cadd(e[3], t3);
  v[7] = csub(e[3], t3);
}

// exp(-2 pi i m / 16)
__device__ __forceinline__ double2 w16(int m) {
  constexpr double c = 0.92387953251128675613, s = 0.38268343236508977173, h = 0.70710678118654752440;
  constexpr double re[16] = {1, c, h, s, 0, -s, -h, -c, -1, -c, -h, -s, 0, s, h, c};
  constexpr double im[16] = {0, -s, -h, -c, -1, -c, -h, -s, 0, s, h, c, 1, c, h, s};
  return make_double2(re[m & 15], im[m & 15]);
}

template <>
__device__ __forceinline__ void dft<16>(double2* v) {
  // radix-4 transforms over the points r = r0 + 4 i, then over r0
  double2 t[16];
#pragma unroll
  for (int r0 = 0; r0 < 4; ++r0) {
    double2 x[4] = {v[r0], v[r0 + 4], v[r0 + 8], v[r0 + 12]};
    dft<4>(x);
#pragma unroll
    for (int q = 0; q < 4; ++q) t[4 * q + r0] = cmul(x[q], w16(r0 * q));
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    dft<4>(t + 4 * q);
#pragma unroll
    for (int m = 0; m < 4; ++m) v[q + 4 * m] = t[4 * q + m];
  }
}

// All transform lengths are powers of two, so every index split below is a
// shift or a mask.  blockIdx.y walks the samples (grid-stride for large S).

// Points of the complex transform: from the previous pass's buffer, or (the
// first pass) packed on the fly from the chain, z_m = (u_2m - K) + i (u_2m+1 - K)
// with K = u_0 of the sample.
enum { kSrcBuffer = 0, kSrcPlain = 1, kSrcSplit = 2 };
struct FftSource {
  const double2* buf;      // kSrcBuffer: [S][N]
  const int64_t* off;      // chains: sample offsets
  const double* u;         // kSrcPlain
  const int32_t* cell;     // kSrcSplit
  const float* frac;
};

template <int SRC>
__device__ __forceinline__ double sample_shift(const FftSource& src, int s) {
  if constexpr (SRC == kSrcPlain) return src.u[src.off[s]];
  else if constexpr (SRC == kSrcSplit) return (double)src.cell[src.off[s]] + (double)src.frac[src.off[s]];
  else return 0.0;
}

template <int SRC>
__device__ __forceinline__ double2 load_point(const FftSource& src, int s, int lgN, int m, double K) {
  if constexpr (SRC == kSrcBuffer) {
    return src.buf[((int64_t)s << lgN) + m];
  } else if constexpr (SRC == kSrcPlain) {
    const double2 x = *reinterpret_cast<const double2*>(src.u + src.off[s] + 2 * (int64_t)m);
    return make_double2(x.x - K, x.y - K);
  } else {
    const int64_t b = src.off[s] + 2 * (int64_t)m;
    const int2 c = *reinterpret_cast<const int2*>(src.cell + b);
    const float2 r = *reinterpret_cast<const float2*>(src.frac + b);
    return make_double2(((double)c.x + (double)r.x) - K, ((double)c.y + (double)r.y) - K);
  }
}

__device__ __forceinline__ double2 unit(double turns) {  // exp(2 pi i turns)
  double sn, cs;
  sincospi(2.0 * turns, &sn, &cs);
  return make_double2(cs, sn);
}

// |U_n / L|^2 of the real transform from Z_n and Z_{N-n} of the half-length
// complex one; W = exp(-2 pi i n / L).
__device__ __forceinline__ double mode_power(double2 zn, double2 zc, double2 W, double inv_l2) {
  const double2 zm = make_double2(zc.x, -zc.y);  // conj(Z_{N-n})
  const double2 A = make_double2(0.5 * (zn.x + zm.x), 0.5 * (zn.y + zm.y));
  const double2 D = csub(zn, zm);
  const double2 B = make_double2(0.5 * D.y, -0.5 * D.x);  // D / (2i)
  const double2 U = cadd(A, cmul(W, B));
  return (U.x * U.x + U.y * U.y) * inv_l2;
}

// ---------------------------------------------------------------------------
// Whole transform of a sample in one workgroup, N = 2^lgN <= kSmallN points:
// S_n, n = 0 .. N, into row s of `rows`.  Passes of radix 8 (the first 2 or 4
// where lgN is no multiple of 3) through one LDS buffer: every thread reads the
// points of its butterflies, then all write.  Points are padded by one in
// eight against bank conflicts of the strided writes.  Bound by the latency of
// its few barriers (one butterfly of radix 8 per thread and pass); four launches of 5 us
// and their gaps took its place at L = 8192 x 64.
// ---------------------------------------------------------------------------
constexpr int kLgSmallN = 12;
constexpr int kSmallN = 1 << kLgSmallN;
constexpr int kSmallBlock = 512;
constexpr int kSmallPoints = kSmallN / kSmallBlock;  // points per thread
__device__ __forceinline__ int pad8(int i) { return i + (i >> 3); }

template <int R, bool FIRST, int SRC>
__device__ __forceinline__ void small_pass(const FftSource& src, int s, double K, double2* z, int lgN, int lgNs) {
  constexpr int lgR = R == 8 ? 3 : (R == 4 ? 2 : 1);
  constexpr int B = kSmallPoints / R;  // butterflies per thread at most
  const int NR = 1 << (lgN - lgR);
  double2 v[B][R];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int j = threadIdx.x + i * kSmallBlock;
    if (j < NR) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (FIRST) v[i][r] = load_point<SRC>(src, s, lgN, j + r * NR, K);
        else v[i][r] = z[pad8(j + r * NR)];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int j = threadIdx.x + i * kSmallBlock;
    if (j < NR) {
      const int k = j & ((1 << lgNs) - 1);
      if constexpr (!FIRST) {
        const double2 w1 = unit(-(double)k / (double)(1 << (lgNs + lgR)));
        double2 w = w1;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          v[i][r] = cmul(v[i][r], w);
          w = cmul(w, w1);
        }
      }
      dft<R>(v[i]);
      const int base = ((j >> lgNs) << (lgNs + lgR)) + k;
#pragma unroll
      for (int q = 0; q < R; ++q) z[pad8(base + (q << lgNs))] = v[i][q];
    }
  }
  __syncthreads();
}

template <int SRC>
__global__ void __launch_bounds__(kSmallBlock)
    k_sq_small(FftSource src, double* __restrict__ rows, int lgN, int S, double inv_l2) {
  __shared__ double2 z[kSmallN + kSmallN / 8];
  const int N = 1 << lgN;
  for (int s = blockIdx.x; s < S; s += gridDim.x) {
    const double K = sample_shift<SRC>(src, s);
    int lgNs = lgN % 3;
    if (lgNs == 1) small_pass<2, true, SRC>(src, s, K, z, lgN, 0);
    else if (lgNs == 2) small_pass<4, true, SRC>(src, s, K, z, lgN, 0);
    else {
      small_pass<8, true, SRC>(src, s, K, z, lgN, 0);
      lgNs = 3;
    }
    for (; lgNs < lgN; lgNs += 3) small_pass<8, false, SRC>(src, s, K, z, lgN, lgNs);
    double* row = rows + (int64_t)s * (N + 1);
    for (int n = threadIdx.x; n <= N; n += kSmallBlock)
      row[n] = mode_power(z[pad8(n == N ? 0 : n)], z[pad8(n == 0 ? 0 : N - n)], unit(-0.5 * (double)n / (double)N),
                          inv_l2);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// One Stockham pass of radix R = 2^LG = 16 x R2 over every transform of the
// batch: sub-transforms of Ns = 2^lgNs points are done, this pass makes them
// Ns R.  A workgroup holds C = 4096 / R columns j, R2 threads each: thread
// (r2, c) loads the points r = r2 + R2 i of column c (C consecutive points per
// row), transforms over i, and after the inner twiddle exchanges through LDS
// for the R2-point transforms: output q = q1 + 16 q2 of column j goes to
// base(j) + q Ns.
//   FIRST (Ns = 1): reads the chain; the outputs of a workgroup are one
//     contiguous run, ordered through LDS before they are written.
//   LAST (Ns = N / R): the columns are C / 2 consecutive ones and their mirror
//     images Ns - j, so that Z_n and Z_{N-n} meet in the workgroup: it forms
//     |U_n / L|^2 and sums it over the samples of its group (blockIdx.y) into
//     row blockIdx.y of `rows`.  (Column 0 is its own mirror image; its partner's
//     place holds column Ns / 2, which is its own too.)
// Bound by memory: 16 B read and 16 B written per point and pass (the last
// writes 8 B per mode).  L = 2^22 x 4: three passes of 128 points, 52, 47 and
// 46 us (the second at 5.7 TB/s); radix-8 and radix-64 passes, a split and a mean kernel took 67, 3 x 47,
// 46 and 14 us.
// ---------------------------------------------------------------------------
template <int LG, int SRC, bool LAST>
__global__ void __launch_bounds__(kBlock, 2)
    k_fft_wide(FftSource src, double2* __restrict__ out, int lgN, int lgNs, int S, double* __restrict__ rows,
               double inv_l2) {
  constexpr bool FIRST = SRC != kSrcBuffer;
  static_assert(!(FIRST && LAST), "a transform of one pass is k_sq_small's");
  constexpr int R = 1 << LG, R2 = R / 16, C = 4096 / R;
  constexpr int M = 16 / R2;  // stage-2 transforms per thread
  __shared__ double2 x[4096 + (FIRST ? 4096 / 16 : 0)];
  __shared__ double2 wq[LAST ? R : 1];
  const int c = threadIdx.x & (C - 1), r2 = threadIdx.x / C;
  const int64_t NR = (int64_t)1 << (lgN - LG);  // columns
  int64_t j;
  if constexpr (LAST) {
    const int64_t j0 = (int64_t)blockIdx.x * (C / 2);
    j = c < C / 2 ? j0 + c : NR - (j0 + (c - C / 2));
    if (j == NR) j = NR / 2;  // the place of column 0's mirror image
  } else {
    j = (int64_t)blockIdx.x * C + c;
  }
  const int64_t k = LAST ? j : (j & (((int64_t)1 << lgNs) - 1));
  double2 a, b;  // pass twiddle of r = r2 + R2 i: a b^i
  if constexpr (!FIRST) {
    const double per = 1.0 / (double)((int64_t)R << lgNs);
    a = unit(-(double)(r2 * k) * per);
    b = unit(-(double)(R2 * k) * per);
  }
  double2 in1 = unit(-(double)r2 / (double)R);  // inner twiddle of q1: in1^q1
  if constexpr (LAST) {
    if (threadIdx.x < R) wq[threadIdx.x] = unit(-0.5 * (double)threadIdx.x / (double)R);
  }
  double2 wj = make_double2(1.0, 0.0);
  if constexpr (LAST) wj = unit(-0.5 * (double)j / (double)((int64_t)1 << lgN));
  double acc[LAST ? 16 : 1], accN = 0.0;
#pragma unroll
  for (int i = 0; i < (LAST ? 16 : 1); ++i) acc[i] = 0.0;
  // Samples: one per blockIdx.y, or (LAST) the group's consecutive ones.
  const int per_group = LAST ? (S + (int)gridDim.y - 1) / (int)gridDim.y : 1;
  const int s0 = LAST ? (int)blockIdx.y * per_group : (int)blockIdx.y;
  const int s1 = LAST ? (s0 + per_group < S ? s0 + per_group : S) : S;
  for (int s = s0; s < s1; s += LAST ? 1 : (int)gridDim.y) {
    // Powers of the twiddles are formed anew for every sample: kept across the
    // loop they would take a hundred registers.
    asm volatile("" : "+v"(in1.x), "+v"(in1.y));
    if constexpr (!FIRST) {
      asm volatile("" : "+v"(a.x), "+v"(a.y));
      asm volatile("" : "+v"(b.x), "+v"(b.y));
    }
    const double K = sample_shift<SRC>(src, s);
    double2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = load_point<SRC>(src, s, lgN, (int)(j + (r2 + R2 * i) * NR), K);
    if constexpr (!FIRST) {
      double2 w = a;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        v[i] = cmul(v[i], w);
        w = cmul(w, b);
      }
    }
    dft<16>(v);
    {
      double2 w = in1;
#pragma unroll
      for (int q1 = 1; q1 < 16; ++q1) {
        v[q1] = cmul(v[q1], w);
        w = cmul(w, in1);
      }
    }
#pragma unroll
    for (int q1 = 0; q1 < 16; ++q1) x[(q1 * R2 + r2) * C + c] = v[q1];
    __syncthreads();
    // Stage 2: this thread's q1 = r2 + R2 m; v[m R2 + q2] = output q1 + 16 q2.
#pragma unroll
    for (int m = 0; m < M; ++m) {
#pragma unroll
      for (int p = 0; p < R2; ++p) v[m * R2 + p] = x[((r2 + R2 * m) * R2 + p) * C + c];
      dft<R2>(v + m * R2);
    }
    __syncthreads();
    if constexpr (FIRST) {
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q2 = 0; q2 < R2; ++q2) {
          const int at = c * R + (r2 + R2 * m) + 16 * q2;
          x[at + (at >> 4)] = v[m * R2 + q2];
        }
      __syncthreads();
      double2* o = out + ((int64_t)s << lgN) + (int64_t)blockIdx.x * 4096;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int at = threadIdx.x + i * kBlock;
        o[at] = x[at + (at >> 4)];
      }
      __syncthreads();
    } else if constexpr (!LAST) {
      double2* o = out + ((int64_t)s << lgN) + ((j >> lgNs) << (lgNs + LG)) + k;
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q2 = 0; q2 < R2; ++q2) o[(int64_t)(r2 + R2 * m + 16 * q2) << lgNs] = v[m * R2 + q2];
    } else {
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q2 = 0; q2 < R2; ++q2) x[(r2 + R2 * m + 16 * q2) * C + c] = v[m * R2 + q2];
      __syncthreads();
      const bool self0 = j == 0, self = self0 || j == NR / 2;
      const int pc = self ? c : (c < C / 2 ? c + C / 2 : c - C / 2);
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q2 = 0; q2 < R2; ++q2) {
          const int q = r2 + R2 * m + 16 * q2;
          const int pq = self0 ? ((R - q) & (R - 1)) : R - 1 - q;
          const double2 zc = x[pq * C + pc];
          acc[m * R2 + q2] += mode_power(v[m * R2 + q2], zc, cmul(wj, wq[q]), inv_l2);
          if (m == 0 && q2 == 0 && self0 && q == 0) accN += mode_power(zc, zc, make_double2(-1.0, 0.0), inv_l2);
        }
      __syncthreads();
    }
  }
  if constexpr (LAST) {
    const int64_t N = (int64_t)1 << lgN;
    double* row = rows + (int64_t)blockIdx.y * (N + 1);
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int q2 = 0; q2 < R2; ++q2) row[j + (r2 + R2 * m + 16 * q2) * NR] = acc[m * R2 + q2];
    if (j == 0 && r2 == 0) row[N] = accN;
  }
}

// Mean over the samples of every mode, from G partial sums (in order).
__global__ void __launch_bounds__(64)
    k_sq_mean(const double* __restrict__ rows, double* __restrict__ mean, int N, int G, int S) {
  const int n = blockIdx.x * 64 + threadIdx.x;
  if (n > N) return;
  double acc = 0.0;
#pragma unroll 16
  for (int g = 0; g < G; ++g) acc += rows[(int64_t)g * (N + 1) + n];
  mean[n] = acc / (double)S;
}

// Chunk c: sum over its modes of the mean over the samples, from G partial sums
// (fixed order: thread stride, then a tree).  Bound by the latency of its loads,
// so some 16 of them are in flight (L = 2^16 x 4 in 32 bins: one after
// the other 61 us a measurement, 49 now).
template <int G>
__global__ void __launch_bounds__(kBlock)
    k_sq_chunk(const double* __restrict__ rows, const int32_t* __restrict__ chunk_lo, int N, int S,
               double* __restrict__ part) {
  constexpr int A = 16 / G;  // modes at a time
  __shared__ double red[kBlock];
  const int c = blockIdx.x;
  const int lo = chunk_lo[c], hi = chunk_lo[c + 1];
  double acc = 0.0;
  for (int n = lo + threadIdx.x; n < hi; n += A * kBlock) {
    double x[A][G];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int m = n + a * kBlock;
        x[a][g] = rows[(int64_t)g * (N + 1) + (m < hi ? m : n)];
      }
#pragma unroll
    for (int a = 0; a < A; ++a) {
      double sum = 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) sum += x[a][g];
      if (n + a * kBlock < hi) acc += sum / (double)S;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[c] = red[0];
}

// Bin b: its chunks' sums (a wave per bin: lane stride, then a tree), divided
// by its number of modes.
__global__ void __launch_bounds__(kBlock)
    k_sq_bin(const double* __restrict__ part, const int32_t* __restrict__ chunk_lo,
             const int32_t* __restrict__ chunk_first, int n_bins, double* __restrict__ out) {
  const int b = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (b >= n_bins) return;
  const int c0 = chunk_first[b], c1 = chunk_first[b + 1];
  double acc = 0.0;
  for (int c = c0 + (threadIdx.x & 63); c < c1; c += 64) acc += part[c];
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1) acc += __shfl_xor(acc, h, 64);
  if ((threadIdx.x & 63) == 0) out[b] = acc / (double)(chunk_lo[c1] - chunk_lo[c0]);
}

// Bins of few modes (one chunk each, every mode a bin or nearly so): one
// thread per bin straight from the partial sums over samples.
__global__ void __launch_bounds__(64)
    k_sq_narrow(const double* __restrict__ rows, const int32_t* __restrict__ chunk_lo, int n_bins, int N, int G,
                int S, double* __restrict__ out) {
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (b >= n_bins) return;
  const int lo = chunk_lo[b], hi = chunk_lo[b + 1];
  double sum = 0.0;
  for (int n = lo; n < hi; ++n) {
    double acc = 0.0;
#pragma unroll 16
    for (int g = 0; g < G; ++g) acc += rows[(int64_t)g * (N + 1) + n];
    sum += acc / (double)S;
  }
  out[b] = sum / (double)(hi - lo);
}

// A workgroup's passes of a transform of 2^lgN points, lgN > kLgSmallN: bits per pass, 5 to 7.
struct Passes {
  int n, lg[8];
};
Passes plan_passes(int lgN) {
  Passes p{};
  p.n = (lgN + 6) / 7;
  for (int i = 0; i < p.n; ++i) p.lg[i] = lgN / p.n + (i < lgN % p.n ? 1 : 0);
  return p;
}

template <int LG, int SRC, bool LAST>
void launch_wide(const FftSource& src, double2* out, int lgN, int lgNs, int S, int groups, double* rows, double inv_l2,
                 hipStream_t st) {
  const unsigned gx = (unsigned)((((int64_t)1 << lgN) >> 12) < 1 ? 1 : (((int64_t)1 << lgN) >> 12));
  const unsigned gy = LAST ? (unsigned)groups : (unsigned)(S < 65535 ? S : 65535);
  hipLaunchKernelGGL((k_fft_wide<LG, SRC, LAST>), dim3(gx, gy), dim3(kBlock), 0, st, src, out, lgN, lgNs, S, rows,
                     inv_l2);
}

template <int SRC, bool LAST>
void launch_wide_lg(int lg, const FftSource& src, double2* out, int lgN, int lgNs, int S, int groups, double* rows,
                    double inv_l2, hipStream_t st) {
  if (lg == 7) launch_wide<7, SRC, LAST>(src, out, lgN, lgNs, S, groups, rows, inv_l2, st);
  else if (lg == 6) launch_wide<6, SRC, LAST>(src, out, lgN, lgNs, S, groups, rows, inv_l2, st);
  else launch_wide<5, SRC, LAST>(src, out, lgN, lgNs, S, groups, rows, inv_l2, st);
}

// Workgroups the last pass should have: below, the samples are split into
// groups whose sums are added afterwards.
constexpr int64_t kLastPassBlocks = 1024;
// Bins of at most so many modes are summed by one thread each.
constexpr int kNarrowModes = 8;

}  // namespace

hipError_t launch_sq(const int64_t* off, int S, int64_t L, const double* u_plain, SplitBuf split,
                     double2* bufA, double2* bufB, const int32_t* chunk_lo, int n_chunks,
                     const int32_t* chunk_first, int n_bins, int max_bin, double* part, double* out,
                     hipStream_t st) {
  const int N = (int)(L / 2);
  int lgN = 0;
  while ((1 << lgN) < N) ++lgN;
  hipError_t e = hipSuccess;
  const FftSource chain{nullptr, off, u_plain, split.cell, split.frac};
  const double inv_l2 = 1.0 / ((double)L * (double)L);
  double* rows = nullptr;  // [G][N + 1] sums over groups of samples
  int G = S;
  if (lgN <= kLgSmallN) {
    rows = reinterpret_cast<double*>(bufA);
    const dim3 g((unsigned)(S < 65535 ? S : 65535));
    if (u_plain) hipLaunchKernelGGL(k_sq_small<kSrcPlain>, g, dim3(kSmallBlock), 0, st, chain, rows, lgN, S, inv_l2);
    else hipLaunchKernelGGL(k_sq_small<kSrcSplit>, g, dim3(kSmallBlock), 0, st, chain, rows, lgN, S, inv_l2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else {
    const Passes ps = plan_passes(lgN);
    double2* in = bufA;
    double2* other = bufB;
    if (u_plain) launch_wide_lg<kSrcPlain, false>(ps.lg[0], chain, in, lgN, 0, S, 0, nullptr, 0.0, st);
    else launch_wide_lg<kSrcSplit, false>(ps.lg[0], chain, in, lgN, 0, S, 0, nullptr, 0.0, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int lgNs = ps.lg[0];
    for (int i = 1; i + 1 < ps.n; ++i) {
      launch_wide_lg<kSrcBuffer, false>(ps.lg[i], FftSource{in, nullptr, nullptr, nullptr, nullptr}, other, lgN, lgNs, S,
                                        0, nullptr, 0.0, st);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      lgNs += ps.lg[i];
      double2* t = in;
      in = other;
      other = t;
    }
    const int64_t blocks = N >> 12;
    const int64_t want = (kLastPassBlocks + blocks - 1) / blocks;
    G = (int)(want < S ? want : S);
    if (G > 65535) G = 65535;
    G = (S + (S + G - 1) / G - 1) / ((S + G - 1) / G);  // no empty group
    rows = reinterpret_cast<double*>(other);
    launch_wide_lg<kSrcBuffer, true>(ps.lg[ps.n - 1], FftSource{in, nullptr, nullptr, nullptr, nullptr}, nullptr, lgN,
                                     lgNs, S, G, rows, inv_l2, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (n_chunks == n_bins && max_bin <= kNarrowModes) {
    hipLaunchKernelGGL(k_sq_narrow, dim3((n_bins + 63) / 64), dim3(64), 0, st, rows, chunk_lo, n_bins, N, G, S, out);
    return hipGetLastError();
  }
  int samples = S;
  if (G > 4) {  // many rows: one thread per mode adds them first
    double* mean = rows + (int64_t)G * (N + 1);  // fits behind the rows: (G + 1) (N + 1) <= 2 S N
    hipLaunchKernelGGL(k_sq_mean, dim3((unsigned)(N / 64 + 1)), dim3(64), 0, st, rows, mean, N, G, S);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    rows = mean;
    G = samples = 1;
  }
  const dim3 gc(n_chunks), bc(kBlock);
  if (G == 1) hipLaunchKernelGGL(k_sq_chunk<1>, gc, bc, 0, st, rows, chunk_lo, N, samples, part);
  else if (G == 2) hipLaunchKernelGGL(k_sq_chunk<2>, gc, bc, 0, st, rows, chunk_lo, N, samples, part);
  else if (G == 3) hipLaunchKernelGGL(k_sq_chunk<3>, gc, bc, 0, st, rows, chunk_lo, N, samples, part);
  else hipLaunchKernelGGL(k_sq_chunk<4>, gc, bc, 0, st, rows, chunk_lo, N, samples, part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_sq_bin, dim3((n_bins + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock), 0, st, part, chunk_lo,
                     chunk_first, n_bins, out);
  return hipGetLastError();
}

}  // namespace qew
