// Front end on the device: real time series -> normalised complex spectrum.
//
// The correlation (Section 1, eq. 2) runs on the Fourier spectrum of the
// observation. This file produces it from a real series of n = 2M samples
// without leaving the device:
//   1. z[j] = x[2j] + i x[2j+1] (the series read as M complex values) is
//      transformed: one transform when M is a compiled length, else the
//      four-step split M = N1 N2 with j = N2 n1 + n2, k = k1 + N1 k2
//      (transforms of length N1 over n1, the twiddles W_M^(n2 k1), transforms
//      of length N2 over n2);
//   2. the real-input split A[k] = E[k] + W_n^k O[k], with
//      E = (Z[k] + conj Z[M-k]) / 2 and O = (Z[k] - conj Z[M-k]) / 2i,
//      gives bins 0 .. M-1 of the real transform (eq. 3 sign; the Nyquist bin
//      is not formed), and |A[k]|^2;
//   3. the median of |A[k]|^2 over bins 1 .. M-1 (an odd count, M being a
//      power of two) by a three-pass radix select on the bit patterns
//      (non-negative floats order as unsigned integers);
//   4. A[k] *= sqrt(ln 2 / median) (unit mean noise power; unscaled when the
//      median is 0) and A[0] = 0.
// Every step is a kernel on the caller's stream; nothing returns to the host.
//
// Five launches (three for short series; four for those of one transform: clear,
// transform, real split, select and normalise), each of which waits for the one
// before, so their number and the chain inside each are what a short series
// costs, and passes over memory what a long one costs:
//   columns   transforms over n1 of a few neighbouring columns, read and
//             written in place of a transpose, with the twiddles;
//   rows      transforms over n2 of a few rows k1 together with their mirror
//             rows N1 - k1, so that Z[k] and Z[M-k] meet in LDS: the real
//             split, the spectrum in natural order, its powers, and the
//             histogram of their first digit;
//   histogram (second digit), histogram (third digit): each block of these
//             and of the last kernel finds the previous digit for itself from
//             the finished histogram, which is cheaper than a kernel between;
//   normalise (up to 2^16 bins the last three are one kernel).
// As 13 launches with three transposes and a one-block kernel per digit: 142 us
// for 2^22 samples and 60 us for 2^16, against 52 and 17. At 2^22 samples the
// two transform kernels take 14 and 19 us for 33 and 41 MB each: what bounds
// them is the 32-byte pieces in which the columns lie, one round of blocks with
// nothing to cover its loads and stores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "fft_batch.hpp"
#include "fft_block.hpp"
#include "fft_radix.hpp"
#include "frontend.hpp"

namespace fdas {

namespace {

constexpr int kSelBins = 2048;  // widest radix-select digit (11 bits)
// Copies of the first two histograms, so that fewer blocks add to one line:
// an exponential distribution fills some 80 bins of the first, and a block adds
// a few hundred counts to the 64 lines of the second (one copy: 17 us for 2^21
// powers, four: 7.5 us).
constexpr int kSelCopies = 4;
constexpr int kShift[3] = {21, 10, 0}, kBins[3] = {2048, 2048, 1024};

struct __attribute__((aligned(16))) SelState {
  unsigned prefix[2];  // high bits of the order statistic after 1, 2 digits
  unsigned rank[2];    // remaining rank inside that prefix
  unsigned hist0[kSelCopies][kSelBins];
  unsigned hist1[kSelCopies][kSelBins];
  unsigned hist2[kSelBins];
};

typedef unsigned u4v __attribute__((ext_vector_type(4)));

// Clears `words` (a multiple of 4) counters; every thread of the grid takes part.
__device__ __forceinline__ void sel_clear(unsigned *h, int words) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < words / 4; i += gridDim.x * blockDim.x)
    reinterpret_cast<u4v *>(h)[i] = u4v{0u, 0u, 0u, 0u};
}
// The histograms of the later digits, which a kernel clears that runs before
// they are counted.
__device__ __forceinline__ void sel_clear_later(SelState *st) {
  sel_clear(&st->hist1[0][0], (kSelCopies + 1) * kSelBins);
}

// Tile of this block: blocks are dealt out to the eight XCDs in turn; each run
// of RUN neighbouring tiles, which share 128-byte lines, goes to one XCD and
// its L2, and the runs go round. (2^21 points as 2048 x 1024, tiles of 32
// bytes: columns 14.2 us; 15.8 us with an eighth of the row on each XCD, whose
// lines then lie in few of its L2's channels; 20 us with the tiles in turn.)
template <int RUN>
__device__ __forceinline__ int xcd_tile() {
  const int nb = gridDim.x, b = blockIdx.x;
  return nb % (8 * RUN) == 0 ? (b / (8 * RUN) * 8 + b % 8) * RUN + b / 8 % RUN : b;
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));  // two complex values
typedef float f4a __attribute__((ext_vector_type(4)));

// a (w + d), where d is what w lost in rounding
__device__ __forceinline__ c32 cmul_fine(c32 a, c32 w, c32 d) {
  const float re = __builtin_fmaf(a.x, d.x, -a.y * d.y), im = __builtin_fmaf(a.x, d.y, a.y * d.x);
  return {__builtin_fmaf(a.x, w.x, __builtin_fmaf(-a.y, w.y, re)),
          __builtin_fmaf(a.x, w.y, __builtin_fmaf(a.y, w.x, im))};
}

// Offset of stage i's factors in a stage table (see frontend.hpp).
template <class Gm>
constexpr int stage_table_off(int i) {
  int o = 0;
  for (int j = 0; j < i; ++j) o += (Gm::R[j] - 1) * Gm::S(j);
  return o;
}
template <class Gm, bool FINE>
__global__ void stage_table_kernel(c32 *__restrict__ out) {
  static_for_up<0, Gm::P - 1>([&](auto ic) {
    constexpr int I = decltype(ic)::value;
    constexpr int S = Gm::S(I), N = Gm::R[I] * S;
    for (int i = threadIdx.x; i < (Gm::R[I] - 1) * S; i += blockDim.x) {
      double sn, cs;
      sincospi(-2.0 * (double)((i / S + 1) * (i % S)) / (double)N, &sn, &cs);
      const c32 w = {(float)cs, (float)sn};
      const int at = stage_table_off<Gm>(I) + i;
      if constexpr (FINE) {
        out[2 * at] = w;
        out[2 * at + 1] = {(float)(cs - (double)w.x), (float)(sn - (double)w.y)};
      } else {
        out[at] = w;
      }
    }
  });
}

// Forward transform of one sequence held by T threads in the layout of stage
// 0, with factors from a stage table; leaves it in LDS in the layout of the
// last stage (addr_of_freq).
template <class Gm, bool FINE>
__device__ __forceinline__ void fft_to_lds(c32 (&x)[Gm::E], c32 *buf, int t,
                                           gptr<const c32> tw) {
  constexpr int P = Gm::P;
  static_for_up<0, P>([&](auto ic) {
    constexpr int I = decltype(ic)::value;
    constexpr int R = Gm::R[I];
    if constexpr (I > 0) exchange<Gm, I - 1, I, 0>(x, buf, buf, t);
#pragma unroll
    for (int j = 0; j < Gm::B(I); ++j) {
      dft<-1, R>(&x[j * R]);
      if constexpr (I < P - 1) {
        const int mi = stage_suffix<Gm, I>(t, j);
#pragma unroll
        for (int k = 1; k < R; ++k) {
          const int at = stage_table_off<Gm>(I) + (k - 1) * Gm::S(I) + mi;
          if constexpr (FINE) {
            const f4a w = *reinterpret_cast<gptr<const f4a>>(tw + 2 * at);
            x[j * R + k] = cmul_fine(x[j * R + k], {w[0], w[1]}, {w[2], w[3]});
          } else {
            x[j * R + k] = cmul(x[j * R + k], ldg(tw + at));
          }
        }
      }
    }
  });
  // (every thread writes the addresses that it alone has read)
  exchange_put<Gm, P - 1>(x, buf, t);
  __syncthreads();
}

// Column transforms: in [N1][N2] -> out [k1][n2], times W_M^(n2 k1). A block
// takes C neighbouring columns (32 bytes of each row for C = 4).
template <class G0, int C, bool FINE>
__global__ void __launch_bounds__(G0::T *C)
    columns_kernel(const c32 *__restrict__ in_, c32 *__restrict__ out_, int N2, float inv_m2,
                   const c32 *__restrict__ tw_, SelState *__restrict__ st) {
  using Gm = OneBuf<G0>;
  constexpr int L = Gm::L, T = Gm::T, E = Gm::E, H = C / 2;
  __shared__ c32 lds[C][Gm::LP];
  const int tid = threadIdx.x;
  const int c0 = xcd_tile<(C < 16 ? 16 / C : 1)>() * C;
  const auto in = to_global(in_);
  const auto out = to_global(out_);
  {
    f4u v[E / 2];
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      const int i = q * (T * C) + tid, n = i / H, h = i % H;
      v[q] = *reinterpret_cast<gptr<const f4u>>(in + (int64_t)n * N2 + c0 + 2 * h);
    }
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      const int i = q * (T * C) + tid, n = i / H, h = i % H;
      lds[2 * h][pad<Gm>(n)] = {v[q][0], v[q][1]};
      lds[2 * h + 1][pad<Gm>(n)] = {v[q][2], v[q][3]};
    }
  }
  __syncthreads();
  const int g = tid / T, t = tid % T;
  c32 x[E];
  exchange_get<Gm, 0>(x, lds[g], t);
  fft_to_lds<Gm, FINE>(x, lds[g], t, to_global(tw_));
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    const int i = q * (T * C) + tid, k = i / H, h = i % H;
    const int a = pad<Gm>(addr_of_freq<Gm>(k));
    c32 u[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // n2 k1 < M <= 2^24 is exact in FP32, and so is the scaled argument
      float sn, cs;
      sincospif(-(float)(k * (c0 + 2 * h + e)) * inv_m2, &sn, &cs);
      u[e] = cmul(lds[2 * h + e][a], c32{cs, sn});
    }
    *reinterpret_cast<gptr<f4u>>(out + (int64_t)k * N2 + c0 + 2 * h) = f4u{u[0].x, u[0].y, u[1].x, u[1].y};
  }
  sel_clear(&st->hist0[0][0], kSelCopies * kSelBins);  // (last: no load waits for these stores)
}

// The real split of one pair: z = Z[k], zm = Z[M-k], w = W_n^k; A[k] and, since
// W_n^(M-k) = -conj W_n^k, A[M-k] = conj(E - W_n^k O).
__device__ __forceinline__ void real_split(c32 z, c32 zm, c32 w, c32 *a, c32 *am) {
  const c32 e = {0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y)};
  const c32 o = {0.5f * (z.y + zm.y), -0.5f * (z.x - zm.x)};  // (z - conj zm) / 2i
  const c32 t = cmul(o, w);
  *a = {e.x + t.x, e.y + t.y};
  *am = {e.x - t.x, t.y - e.y};
}
__device__ __forceinline__ c32 unit_turn(int64_t k, float inv_m) {
  float sn, cs;
  sincospif(-(float)k * inv_m, &sn, &cs);  // W_n^k = exp(-2 pi i k / 2M), k < 2^24 exact
  return {cs, sn};
}
__device__ __forceinline__ float power(c32 v) { return __builtin_fmaf(v.x, v.x, v.y * v.y); }

__device__ __forceinline__ void count0(unsigned *h, float p) {
  atomicAdd(&h[__float_as_uint(p) >> kShift[0]], 1u);
}
// Adds a block's first-digit counts to one of the global copies.
__device__ __forceinline__ void flush0(const unsigned *h, SelState *st) {
  unsigned *to = st->hist0[blockIdx.x % kSelCopies];
  for (int i = threadIdx.x; i < kSelBins / 4; i += blockDim.x) {
    const u4v v = reinterpret_cast<const u4v *>(h)[i];
    if ((v[0] | v[1] | v[2] | v[3]) == 0u) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (v[e]) atomicAdd(&to[4 * i + e], v[e]);
  }
}
__device__ __forceinline__ void zero_bins(unsigned *h) {
  for (int i = threadIdx.x; i < kSelBins / 4; i += blockDim.x)
    reinterpret_cast<u4v *>(h)[i] = u4v{0u, 0u, 0u, 0u};
}

// Row transforms in [k1][N2] -> Z[k1 + N1 k2], the real split, powers and
// first digits. A block takes rows p0 .. p0+P-1 and their mirrors N1-p; row 0
// and row N1/2, which are their own mirrors, stand together.
template <class G0, int P, bool FINE>
__global__ void __launch_bounds__(G0::T * 2 * P)
    rows_kernel(const c32 *__restrict__ in_, c32 *__restrict__ A_, float *__restrict__ pw_, int N1,
                float inv_m, const c32 *__restrict__ tw_, SelState *__restrict__ st) {
  using Gm = OneBuf<G0>;
  constexpr int L = Gm::L, T = Gm::T, E = Gm::E, R0 = Gm::R[0], S0 = Gm::S(0), NT = T * 2 * P;
  __shared__ c32 lds[2 * P][Gm::LP];
  __shared__ __attribute__((aligned(16))) unsigned hist[kSelBins];
  const int tid = threadIdx.x;
  const int g = tid / T, t = tid % T;
  const int tile = xcd_tile<(P < 16 ? 16 / P : 1)>();
  const int p0 = tile * P;
  const auto A = to_global(A_);
  const auto pw = to_global(pw_) + (int64_t)tile * (2 * P * L);
  auto high = [&](int p) { return p == 0 ? N1 / 2 : N1 - p; };
  const auto in = to_global(in_) + (int64_t)(g < P ? p0 + g : high(p0 + g - P)) * L;
  c32 x[E];
#pragma unroll
  for (int j = 0; j < Gm::B(0); ++j)
#pragma unroll
    for (int n = 0; n < R0; ++n) x[j * R0 + n] = ldg(in + n * S0 + t + j * T);
  zero_bins(hist);
  fft_to_lds<Gm, FINE>(x, lds[g], t, to_global(tw_));
  auto at = [&](int r, int k2) { return lds[r][pad<Gm>(addr_of_freq<Gm>(k2))]; };
  for (int k2 = tid; k2 < L; k2 += NT) {
    const int m2 = L - 1 - k2;  // the mirror of (p, k2) is (N1 - p, m2)
    c32 lo[P], hi[P];
    float pl[P], ph[P];
#pragma unroll
    for (int s = 0; s < P; ++s) {
      const int p = p0 + s;
      if (p == 0) {
        // rows 0 and N1/2: the mirror of (0, k2) is (0, -k2), that of
        // (N1/2, k2) is (N1/2, m2)
        c32 none;
        real_split(at(0, k2), at(0, (L - k2) & (L - 1)), unit_turn((int64_t)N1 * k2, inv_m), &lo[s],
                   &none);
        real_split(at(P, k2), at(P, m2), unit_turn((int64_t)N1 * k2 + N1 / 2, inv_m), &hi[s], &none);
      } else {
        real_split(at(s, k2), at(P + s, m2), unit_turn((int64_t)N1 * k2 + p, inv_m), &lo[s], &hi[s]);
      }
      pl[s] = power(lo[s]);
      ph[s] = power(hi[s]);
      if (p + k2 > 0) count0(hist, pl[s]);  // (bin 0 is not ranked)
      count0(hist, ph[s]);
    }
    const int64_t kl = (int64_t)N1 * k2 + p0;
    const int64_t kh = (int64_t)N1 * m2 + N1 - p0 - (P - 1);  // of s = P - 1, downwards
#pragma unroll
    for (int s = 0; s < P; s += 2)
      *reinterpret_cast<gptr<f4u>>(A + kl + s) = f4u{lo[s].x, lo[s].y, lo[s + 1].x, lo[s + 1].y};
    if (p0 == 0) {
      *reinterpret_cast<gptr<f2v>>(A + (int64_t)N1 * k2 + N1 / 2) = f2v{hi[0].x, hi[0].y};
#pragma unroll
      for (int s = 1; s < P; ++s)
        *reinterpret_cast<gptr<f2v>>(A + kh + (P - 1 - s)) = f2v{hi[s].x, hi[s].y};
    } else {
#pragma unroll
      for (int s = P - 1; s > 0; s -= 2)
        *reinterpret_cast<gptr<f4u>>(A + kh + (P - 1 - s)) =
            f4u{hi[s].x, hi[s].y, hi[s - 1].x, hi[s - 1].y};
    }
    // The powers only pass through the select, so they lie as they are made
    // (bin 0 first: tile 0, k2 0).
    const auto pk = pw + k2 * (2 * P);
#pragma unroll
    for (int s = 0; s < P; s += 2) {
      *reinterpret_cast<gptr<f2v>>(pk + s) = f2v{pl[s], pl[s + 1]};
      *reinterpret_cast<gptr<f2v>>(pk + P + s) = f2v{ph[s], ph[s + 1]};
    }
  }
  sel_clear_later(st);
  __syncthreads();
  flush0(hist, st);
}

// One-transform lengths: the real split, powers and first digits from Z.
__global__ void __launch_bounds__(256)
    split_kernel(const c32 *__restrict__ Z_, c32 *__restrict__ A_, float *__restrict__ P_,
                 int64_t M, float inv_m, SelState *__restrict__ st) {
  __shared__ __attribute__((aligned(16))) unsigned hist[kSelBins];
  const auto Z = to_global(Z_);
  const auto A = to_global(A_);
  const auto P = to_global(P_);
  zero_bins(hist);
  __syncthreads();
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < M) {
    c32 a, none;
    real_split(ldg(Z + k), ldg(Z + ((M - k) & (M - 1))), unit_turn(k, inv_m), &a, &none);
    *reinterpret_cast<gptr<f2v>>(A + k) = f2v{a.x, a.y};
    const float p = power(a);
    P[k] = p;
    if (k > 0) count0(hist, p);
  }
  __syncthreads();
  flush0(hist, st);
}

__global__ void __launch_bounds__(256) sel_clear_kernel(SelState *st) {
  sel_clear(&st->hist0[0][0], kSelCopies * kSelBins);
  sel_clear_later(st);
}

// The digit of `rank` in a finished histogram and the rank left inside it,
// by a block of NT threads (bins a multiple of NT); all threads receive it.
template <int NT, int BINS, int COPIES>
__device__ __forceinline__ void find_digit(const unsigned *hist, unsigned rank, unsigned *digit,
                                           unsigned *left) {
  constexpr int PER = BINS / NT;
  __shared__ unsigned wave_sum[NT / 64];
  __shared__ unsigned found[2];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  unsigned c[PER], sum = 0u;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    c[j] = 0u;
#pragma unroll
    for (int q = 0; q < COPIES; ++q) c[j] += hist[q * kSelBins + t * PER + j];
    sum += c[j];
  }
  unsigned upto = sum;  // inclusive scan over the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned v = __shfl_up(upto, off);
    if (lane >= off) upto += v;
  }
  if (lane == 63) wave_sum[w] = upto;
  __syncthreads();
  for (int q = 0; q < w; ++q) upto += wave_sum[q];
  unsigned below = upto - sum;
  if (rank >= below && rank < upto) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (rank >= below && rank < below + c[j]) {
        found[0] = (unsigned)(t * PER + j);
        found[1] = rank - below;
      }
      below += c[j];
    }
  }
  __syncthreads();
  *digit = found[0];
  *left = found[1];
}

// Histogram of digit PASS (1 or 2) of the powers, but the first (bin 0's),
// whose higher digits are those of the order statistic.
template <int PASS>
__global__ void __launch_bounds__(256)
    sel_hist_kernel(const float *__restrict__ P_, int64_t M, SelState *__restrict__ st,
                    unsigned rank0) {
  constexpr int NB = kBins[PASS], SH = kShift[PASS];
  __shared__ unsigned h[NB];
  const auto P = to_global(reinterpret_cast<const unsigned *>(P_));
  for (int i = threadIdx.x; i < NB; i += blockDim.x) h[i] = 0u;
  unsigned digit, left, prefix;
  if constexpr (PASS == 1) {
    find_digit<256, kBins[0], kSelCopies>(&st->hist0[0][0], rank0, &digit, &left);
    prefix = digit << kShift[0];
  } else {
    find_digit<256, kBins[1], kSelCopies>(&st->hist1[0][0], st->rank[0], &digit, &left);
    prefix = st->prefix[0] | digit << kShift[1];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->prefix[PASS - 1] = prefix;
    st->rank[PASS - 1] = left;
  }
  constexpr unsigned mask = ~0u << kShift[PASS - 1];
  auto count = [&](unsigned u) {
    if ((u & mask) == prefix) atomicAdd(&h[(u >> SH) & (NB - 1)], 1u);
  };
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;  // in groups of four
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M / 4; i += stride) {
    const u4v u = *reinterpret_cast<gptr<const u4v>>(P + 4 * i);
    if (i > 0) count(u[0]);  // (bin 0 is not ranked)
    count(u[1]);
    count(u[2]);
    count(u[3]);
  }
  __syncthreads();
  unsigned *to = PASS == 1 ? st->hist1[blockIdx.x % kSelCopies] : st->hist2;
  for (int i = threadIdx.x; i < NB; i += blockDim.x) {
    const unsigned v = h[i];
    if (v) atomicAdd(&to[i], v);
  }
}

__device__ __forceinline__ float scale_of(float median) {
  const double med = (double)median;
  return med > 0.0 ? (float)sqrt(0.69314718055994530942 / med) : 1.0f;
}
// A[k] *= scale for the pairs of bins first, first + stride, ..., A[0] = 0;
// stats = (scale, median) if given.
__device__ __forceinline__ void normalise(gptr<c32> A, int64_t M, float med, float *stats) {
  const float s = scale_of(med);
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (first == 0 && stats) {
    stats[0] = s;
    stats[1] = med;
  }
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = first; i < M / 2; i += stride) {
    const gptr<f4u> p = reinterpret_cast<gptr<f4u>>(A + 2 * i);
    f4u v = *p * s;
    if (i == 0) v[0] = v[1] = 0.f;
    *p = v;
  }
}

__global__ void __launch_bounds__(256)
    normalise_kernel(c32 *__restrict__ A, int64_t M, const SelState *__restrict__ st,
                     float *__restrict__ stats) {
  unsigned digit, left;
  find_digit<256, kBins[2], 1>(st->hist2, st->rank[1], &digit, &left);
  normalise(to_global(A), M, __uint_as_float(st->prefix[1] | digit), stats);
}

// Short spectra: the last two digits and the scale in one kernel. Every block
// holds all powers in registers (Q groups of four per thread) and selects for
// itself, then scales its part (9 us at 32768 bins, where the three kernels
// take 12).
constexpr int kShortThreads = 1024;
template <int Q>
__global__ void __launch_bounds__(kShortThreads)
    select_normalise_kernel(const float *__restrict__ P_, c32 *__restrict__ A, int64_t M,
                            const SelState *__restrict__ st, unsigned rank,
                            float *__restrict__ stats) {
  constexpr int NT = kShortThreads;
  __shared__ unsigned h[2][kSelBins];
  const auto P = to_global(reinterpret_cast<const unsigned *>(P_));
  const int tid = threadIdx.x;
  u4v u[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = q * NT + tid;
    if (i < M / 4) u[q] = *reinterpret_cast<gptr<const u4v>>(P + 4 * i);
  }
  for (int i = tid; i < 2 * kSelBins; i += NT) (&h[0][0])[i] = 0u;
  unsigned prefix = 0u, digit;
  find_digit<NT, kBins[0], kSelCopies>(&st->hist0[0][0], rank, &digit, &rank);
  prefix |= digit << kShift[0];
  auto count = [&](unsigned *to, unsigned mask, int shift, int bins) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = q * NT + tid;
      if (i >= M / 4) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((i > 0 || e > 0) && (u[q][e] & mask) == prefix)
          atomicAdd(&to[(u[q][e] >> shift) & (bins - 1)], 1u);
    }
  };
  count(h[0], ~0u << kShift[0], kShift[1], kBins[1]);
  __syncthreads();
  find_digit<NT, kBins[1], 1>(h[0], rank, &digit, &rank);
  prefix |= digit << kShift[1];
  count(h[1], ~0u << kShift[1], kShift[2], kBins[2]);
  __syncthreads();
  find_digit<NT, kBins[2], 1>(h[1], rank, &digit, &rank);
  normalise(to_global(A), M, __uint_as_float(prefix | digit), stats);
}

// columns a block of the column kernel takes, and pairs of rows one of the
// row kernel: 32 bytes of a row, at least a wave of threads, and what LDS holds
template <class G0>
constexpr int columns_of() {
  return G0::T * 4 >= 64 ? 4 : 64 / G0::T;
}
template <class G0>
constexpr int pairs_of() {
  return G0::L == 4096 ? 2 : (G0::T * 8 >= 64 ? 4 : 32 / G0::T);
}

template <bool FINE, class G0>
hipError_t launch_columns(const FrontendGeom &g, const c32 *z, c32 *work, SelState *st,
                          hipStream_t s) {
  constexpr int C = columns_of<G0>();
  hipLaunchKernelGGL((columns_kernel<G0, C, FINE>), dim3(g.N2 / C), dim3(G0::T * C), 0, s, z, work, g.N2,
                     2.0f / (float)g.M, g.tw1, st);
  return hipGetLastError();
}
template <bool FINE, class G0>
hipError_t launch_rows(const FrontendGeom &g, const c32 *work, c32 *spectrum, float *pw,
                       SelState *st, hipStream_t s) {
  constexpr int P = pairs_of<G0>();
  hipLaunchKernelGGL((rows_kernel<G0, P, FINE>), dim3(g.N1 / 2 / P), dim3(G0::T * 2 * P), 0, s, work,
                     spectrum, pw, g.N1, 1.0f / (float)g.M, g.tw2, st);
  return hipGetLastError();
}

// f with the geometry of an n-point transform: 16 elements per thread, and for
// spectra of at most kFewPoints bins, whose blocks do not fill the chip, 4 or 8,
// so that each wave's chain of instructions is that much shorter (columns 6.5
// -> 3.7 us and rows 8.2 -> 4.8 us at 32768 bins). That makes more stages, whose
// factors come with their rounding errors (FINE), or the error would grow: over
// 400 series of 2^16 samples 1.379e-7 of the spectrum's norm with 16 elements,
// 1.421e-7 with few, and 1.376e-7 this way (16.9 -> 17.0 us there, 24.4 -> 25.0 at
// 2^19, where the gain of few elements is the least).
constexpr int64_t kFewPoints = 1 << 18;
template <class F>
hipError_t with_length(int n, int64_t M, F &&f) {
  if (M <= kFewPoints) switch (n) {
    case 64: return f(Geo<64, 16, 4, 4, 4>{}, std::true_type{});
    case 128: return f(Geo<128, 32, 2, 4, 4, 4>{}, std::true_type{});
    case 256: return f(Geo<256, 64, 4, 4, 4, 4>{}, std::true_type{});
    case 512: return f(Geo<512, 64, 8, 8, 8>{}, std::true_type{});
  }
  else switch (n) {
    case 512: return f(Geo<512, 32, 16, 2, 16>{}, std::false_type{});
    case 1024: return f(Geo<1024, 64, 16, 4, 16>{}, std::false_type{});
    case 2048: return f(Geo<2048, 128, 16, 8, 16>{}, std::false_type{});
    case 4096: return f(Geo<4096, 256, 16, 16, 16>{}, std::false_type{});
  }
  return hipErrorInvalidValue;
}

}  // namespace

size_t frontend_sel_bytes() { return sizeof(SelState); }

hipError_t launch_stage_table(c32 *out, int n, int64_t M, hipStream_t s) {
  return with_length(n, M, [&](auto geo, auto fine) {
    hipLaunchKernelGGL((stage_table_kernel<decltype(geo), decltype(fine)::value>), dim3(1),
                       dim3(1024), 0, s, out);
    return hipGetLastError();
  });
}

hipError_t launch_frontend(const FrontendGeom &g, const float *series, c32 *spectrum, c32 *work,
                           float *pw, void *sel_, float *stats, hipStream_t s) {
  SelState *sel = static_cast<SelState *>(sel_);
  const int64_t M = g.M;
  const c32 *z = reinterpret_cast<const c32 *>(series);
  hipError_t e = hipSuccess;
  if (g.N2 == 1) {
    hipLaunchKernelGGL(sel_clear_kernel, dim3(16), dim3(256), 0, s, sel);
    e = hipGetLastError();
    if (e == hipSuccess) e = g.f1->launch(z, work, 1, -1, g.tw1, s);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(split_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s, work,
                         spectrum, pw, M, 1.0f / (float)M, sel);
      e = hipGetLastError();
    }
  } else {
    e = with_length(g.N1, M, [&](auto geo, auto fine) {
      return launch_columns<decltype(fine)::value, decltype(geo)>(g, z, work, sel, s);
    });
    if (e == hipSuccess)
      e = with_length(g.N2, M, [&](auto geo, auto fine) {
        return launch_rows<decltype(fine)::value, decltype(geo)>(g, work, spectrum, pw, sel, s);
      });
  }
  if (e != hipSuccess) return e;
  // median of bins 1 .. M-1: M is a power of two, so the count is odd and the
  // median is the single middle order statistic
  const unsigned rank = (unsigned)((M - 1) / 2);
  if (M <= 16 * 4 * kShortThreads) {
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)std::max<int64_t>(1, M / 2 / kShortThreads)),
                         dim3(kShortThreads), 0, s, pw, spectrum, M, sel, rank, stats);
      return hipGetLastError();
    };
    const int64_t q = M / 4 / kShortThreads;
    return q <= 2   ? launch(select_normalise_kernel<2>)
           : q <= 4 ? launch(select_normalise_kernel<4>)
           : q <= 8 ? launch(select_normalise_kernel<8>)
                    : launch(select_normalise_kernel<16>);
  }
  const unsigned hblocks = (unsigned)std::min<int64_t>(512, (M / 4 + 255) / 256);
  hipLaunchKernelGGL(sel_hist_kernel<1>, dim3(hblocks), dim3(256), 0, s, pw, M, sel, rank);
  hipLaunchKernelGGL(sel_hist_kernel<2>, dim3(hblocks), dim3(256), 0, s, pw, M, sel, rank);
  const unsigned nblocks = (unsigned)std::min<int64_t>(1024, (M / 2 + 255) / 256);
  hipLaunchKernelGGL(normalise_kernel, dim3(nblocks), dim3(256), 0, s, spectrum, M, sel, stats);
  return hipGetLastError();
}

}  // namespace fdas
