// The Fourier-domain template bank (plan time, FP64): the sums
//   S_z(k) = sum_{q=-m/2}^{m/2} H_z(q) exp(-2 pi i q k / L)
// behind every storage form of the bank T_z[k] = conj(S_z(k)) / L.
//
// Taps q and -q share one cosine and one sine, and so do frequencies k and
// L - k:
//   S(+-k) = P(k) -+ i Q(k),  P = H(0) + sum_{q>0} (H(q) + H(-q)) cos(2 pi q k / L),
//                             Q =        sum_{q>0} (H(q) - H(-q)) sin(2 pi q k / L).
// At integer offsets H_z is even in q (Q = 0) and H_{-z} = conj(H_z), so a
// row of the first half of the z grid also gives its mirror, whose bank row is
// the exact conjugate (the correlation kernels' pair forms rely on it). The
// rows at half-bin offsets have neither symmetry in [-m/2, m/2] and are
// summed one by one, with Q.
//
// The angle is reduced exactly (q k mod L) and its cosine read from a
// quarter-wave table in LDS, which the block makes once with sincospi; a wave
// holds ROWS rows of 64 frequencies in registers, so one table read serves them
// all. One sincospi per term and frequency instead took 227 us for 101 rows of
// 2048 frequencies (257 taps), against 12 us.
//
// ROWS is 4 where that makes more blocks than there are compute units, and 2
// below, where the chip is not full and the chains of table reads and of taps
// from memory bound it: half the rows, and twice the taps staged and table reads
// in flight at a time. (On 256 compute units, 101 rows of 2048: 19.9 us with 4,
// 11.6 with 2. The whole call for 201 rows of 4096, 513 taps, 231 blocks of 4: 67
// against 62 us; of 8192, 455 blocks: 79 against 82.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fdas {

struct c64b {
  double x, y;
};

constexpr int kBankWaves = 4;   // waves per block, on different rows

// put(row, k, re, im) stores S = (re, im) of bank row `row` at frequency k.
// h holds the templates [rows][m + 1]; nzg counts the rows of the z grid.
template <bool HALF, int ROWS, class Put>
__global__ void __launch_bounds__(64 * kBankWaves)
    bank_sum_kernel(const c64b *__restrict__ h, int nzg, int interbin, int m, int L, Put put) {
  constexpr int kBankTaps = 128 / ROWS;  // staged in LDS at a time
  extern __shared__ double cos_tab[];  // cos(2 pi j / L), j in [0, L / 4]
  __shared__ c64b even[kBankWaves * ROWS][kBankTaps];
  __shared__ c64b odd[HALF ? kBankWaves * ROWS : 1][kBankTaps];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int quarter = L >> 2, half_m = m >> 1;
  for (int j = tid; j <= quarter; j += 64 * kBankWaves) cos_tab[j] = cospi(2.0 * (double)j / (double)L);
  const int k = blockIdx.x * 64 + lane;  // up to L / 2
  const int rows = HALF ? nzg : (nzg + 1) >> 1;
  const int r0 = blockIdx.y * (kBankWaves * ROWS);
  auto row_of = [&](int r) { return interbin ? 2 * r + (HALF ? 1 : 0) : r; };
  auto cosine = [&](int j) {  // cos(2 pi j / L), j in [0, L)
    j = j > L / 2 ? L - j : j;
    const bool neg = j > quarter;
    const double c = cos_tab[neg ? L / 2 - j : j];
    return neg ? -c : c;
  };
  double pr[ROWS], pi[ROWS], qr[ROWS], qi[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int r = r0 + w * ROWS + i;
    pr[i] = pi[i] = qr[i] = qi[i] = 0.0;
    if (r < rows) {
      const c64b v = h[(long)row_of(r) * (m + 1) + half_m];
      pr[i] = v.x;
      pi[i] = v.y;
    }
  }
  for (int q0 = 1; q0 <= half_m; q0 += kBankTaps) {
    const int n = min(kBankTaps, half_m + 1 - q0);
    __syncthreads();  // the table is made; the taps before have been read
    for (int i = tid; i < kBankWaves * ROWS * kBankTaps; i += 64 * kBankWaves) {
      const int r = r0 + i / kBankTaps, q = q0 + i % kBankTaps;
      c64b a = {0.0, 0.0}, b = {0.0, 0.0};
      if (r < rows && q <= half_m) {
        const c64b *row = h + (long)row_of(r) * (m + 1) + half_m;
        a = row[q];
        b = row[-q];
      }
      even[i / kBankTaps][i % kBankTaps] = {a.x + b.x, a.y + b.y};
      if constexpr (HALF) odd[i / kBankTaps][i % kBankTaps] = {a.x - b.x, a.y - b.y};
    }
    __syncthreads();
#pragma unroll (16 / ROWS)
    for (int t = 0; t < n; ++t) {
      const int j = (int)(((unsigned)(q0 + t) * (unsigned)k) & (unsigned)(L - 1));
      const double c = cosine(j);
      double sn = 0.0;
      if constexpr (HALF) sn = cosine((j + 3 * quarter) & (L - 1));
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const c64b s = even[w * ROWS + i][t];
        pr[i] = __builtin_fma(s.x, c, pr[i]);
        pi[i] = __builtin_fma(s.y, c, pi[i]);
        if constexpr (HALF) {
          const c64b d = odd[w * ROWS + i][t];
          qr[i] = __builtin_fma(d.x, sn, qr[i]);
          qi[i] = __builtin_fma(d.y, sn, qi[i]);
        }
      }
    }
  }
  if (k > L / 2) return;
  const int mk = (L - k) & (L - 1);
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int r = r0 + w * ROWS + i;
    if (r >= rows) continue;
    // P - i Q at k, P + i Q at L - k
    put(row_of(r), k, pr[i] + qi[i], pi[i] - qr[i]);
    if (mk != k) put(row_of(r), mk, pr[i] - qi[i], pi[i] + qr[i]);
    if (!HALF && nzg - 1 - r != r) {  // the mirror row: the conjugate
      put(row_of(nzg - 1 - r), k, pr[i], -pi[i]);
      if (mk != k) put(row_of(nzg - 1 - r), mk, pr[i], -pi[i]);
    }
  }
}

// Compute units of the current device (256 if that cannot be asked).
static int bank_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 256;
  return cus;
}

template <bool HALF, class Put>
static void launch_bank_part(const void *h, int nzg, int interbin, int m, int L, Put put,
                             hipStream_t s) {
  const int rows = HALF ? nzg : (nzg + 1) / 2;
  const unsigned gx = (unsigned)(L / 2 / 64 + 1);
  const size_t lds = (size_t)(L / 4 + 1) * sizeof(double);
  auto blocks = [&](int per_wave) {
    return dim3(gx, (unsigned)((rows + kBankWaves * per_wave - 1) / (kBankWaves * per_wave)));
  };
  const dim3 wide = blocks(4);
  if ((int64_t)wide.x * wide.y > bank_cus())
    hipLaunchKernelGGL((bank_sum_kernel<HALF, 4, Put>), wide, dim3(64 * kBankWaves), lds, s,
                       static_cast<const c64b *>(h), nzg, interbin, m, L, put);
  else
    hipLaunchKernelGGL((bank_sum_kernel<HALF, 2, Put>), blocks(2), dim3(64 * kBankWaves), lds, s,
                       static_cast<const c64b *>(h), nzg, interbin, m, L, put);
}

// Every row of a bank: `rows` counts bank rows (twice the z grid with interbin).
template <class Put>
static hipError_t launch_bank_sum(const void *h, int rows, int interbin, int m, int L, Put put,
                                  hipStream_t s) {
  const int nzg = interbin ? rows / 2 : rows;
  launch_bank_part<false>(h, nzg, interbin, m, L, put, s);
  if (interbin) launch_bank_part<true>(h, nzg, interbin, m, L, put, s);
  return hipGetLastError();
}

}  // namespace fdas
