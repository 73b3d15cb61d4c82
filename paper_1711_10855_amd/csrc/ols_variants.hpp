// Registry of compiled hot-kernel variants (host side).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cand_place.hpp"
#include "fft_radix.hpp"
#include "launch_units.hpp"
#include "layout.hpp"

namespace fdas {

// Detection epilogue: with `count` set, plane points whose power is at least
// `thr` are counted on `count` and written to `list` while the slot is below
// `cap` (list may be null when cap is 0), instead of the plane being stored.
struct Cand {
  int row;
  float power;
  int64_t r;
};
static_assert(sizeof(Cand) == 16, "candidate record is 16 bytes");
struct CandOut {
  Cand *list;
  unsigned long long *count;
  int64_t cap;
  float thr;
};

// Detection kernels collect a block's candidates in LDS and list them when the
// unit ends: a hit then costs an LDS atomic, not a round trip to memory. A
// segment with a strong signal has hits in most rows, so its block is the one
// that the launch waits for (2^21 bins x 101 rows in FP32 with eight signals,
// against 223 us without a hit: 276 us with a global atomic per power, 254 with
// one per template and wave, 228 collected).
struct CandLds {
  int n;    // entries asked for (see cand_place); from `lim` on they did not fit
  int lim;
  unsigned long long base;
  struct {
    int row;
    float power;
    int rel;  // bin - the block's first kept bin
  } e[kCandLds];
};
__device__ __forceinline__ void cand_store(gptr<Cand> to, int row, float p, int64_t r) {
  typedef int i4v __attribute__((ext_vector_type(4)));
  const i4v v = {row, __builtin_bit_cast(int, p), (int)(uint64_t)r, (int)((uint64_t)r >> 32)};
  *(gptr<i4v>)to = v;  // one 16-byte store
}

// By one thread, before a barrier that precedes the first offer.
__device__ __forceinline__ void cand_begin(CandLds *b) {
  b->n = 0;
  b->lim = kCandLds;
}

// Called by every lane of the wave together (not under divergent control
// flow): lists, at plane row `row`, the lane's powers p[e] that reach the
// threshold at a kept output, at(e) in [0, nkeep). Output 0 is bin rel0 of the
// block's, whose first is bin r0 of the plane.
template <int N, class At>
__device__ __forceinline__ void cand_offer(const CandOut &cd, CandLds *b, int row,
                                           const float (&p)[N], At at, int nkeep, int rel0,
                                           int64_t r0) {
  unsigned long long hit[N];
  int total = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    hit[e] = __builtin_amdgcn_ballot_w64(p[e] >= cd.thr && (unsigned)at(e) < (unsigned)nkeep);
    total += __builtin_popcountll(hit[e]);
  }
  if (total == 0) return;
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  int pos = 0;
  if (lane == 0)
    pos = cand_place(
        total,
        [&] { return __hip_atomic_load(&b->n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); },
        [&](int k) { return atomicAdd(&b->n, k); });
  pos = __builtin_amdgcn_readfirstlane(pos);
  const bool fits = cand_fits(pos, total);
  unsigned long long base = 0ull;
  if (!fits) {  // straight to the list
    if (lane == 0) {
      atomicMin(&b->lim, pos);
      base = atomicAdd(cd.count, (unsigned long long)total);
    }
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)base);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(base >> 32));
    base = ((unsigned long long)hi << 32) | lo;
    pos = 0;
  }
#pragma unroll
  for (int e = 0; e < N; ++e) {
    if (hit[e] == 0ull) continue;
    if (hit[e] >> lane & 1ull) {
      const int k = pos + (int)__builtin_amdgcn_mbcnt_hi(
                              (unsigned)(hit[e] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hit[e], 0u));
      const int rel = rel0 + at(e);
      if (fits)
        b->e[k] = {row, p[e], rel};
      else if (base + (unsigned)k < (unsigned long long)cd.cap)
        cand_store((gptr<Cand>)cd.list + base + k, row, p[e], r0 + rel);
    }
    pos += __builtin_popcountll(hit[e]);
  }
}

// By the whole block after its last offer (block-wide barriers inside); r0 as
// in the offers.
__device__ __forceinline__ void cand_end(const CandOut &cd, CandLds *b, int64_t r0) {
  __syncthreads();
  const int m = cand_listed(b->n, b->lim);
  if (m == 0) return;
  if (threadIdx.x == 0) b->base = atomicAdd(cd.count, (unsigned long long)m);
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += blockDim.x)
    if (b->base + (unsigned)i < (unsigned long long)cd.cap)
      cand_store((gptr<Cand>)cd.list + b->base + i, b->e[i].row, b->e[i].power, r0 + b->e[i].rel);
}

struct OlsArgs {
  const void *spec;  // complex64 [nbins]
  int64_t nbins;
  const void *bank;  // slot-ordered bank [nz][L]
  const void *tw;    // twiddles W_L^j, complex64 [L]
  float *power;      // [nz][ld]
  int64_t ld;
  int nseg;          // ceil(nbins / U)
  int U;             // L - m
  int half;          // m / 2
  int nz;            // rows to produce
  int n1, zpb1, zpb2;  // templates per work unit: zpb1 on the first n1 segment
                       // groups, zpb2 on the others
  int bank_log2;     // mixed precision: the bank is stored times 2^bank_log2
  const void *consts;  // mixed precision: per-lane constants table
  CandOut cand;        // detection epilogue (count == nullptr: store the plane)
  int pair;            // rows z and -z together (see unit_rows)
};

// What a work unit counts: rows, or in the pair form pairs of a row and its
// mirror (z and -z, whose bank rows are complex conjugates; of an odd number
// of rows the middle one stands alone).
__host__ __device__ inline int unit_rows(int rows, bool pair) {
  return pair ? (rows + 1) >> 1 : rows;
}

// The work units of a single-spectrum launch, one per block: first those of
// the segment groups [0, n1), of per1 rows (or pairs) each, then those of the
// others, of per2; row-group major inside each part.
struct UnitGrid {
  int nsb, rows, n1, per1, per2;
  unsigned b1;  // units of the first part
  __host__ long blocks() const {
    return (long)b1 + (long)(nsb - n1) * ((rows + per2 - 1) / per2);
  }
  __device__ __forceinline__ void unit(unsigned b, int *sb, int *z0, int *z1) const {
    const bool second = b >= b1;
    const unsigned i = second ? b - b1 : b, n = second ? nsb - n1 : n1;
    const int per = second ? per2 : per1;
    *sb = (second ? n1 : 0) + (int)(i % n);
    *z0 = (int)(i / n) * per;
    *z1 = *z0 + per < rows ? *z0 + per : rows;
  }
};
// (G: segments per group)
inline UnitGrid unit_grid(const OlsArgs &a, int G, bool pair) {
  UnitGrid u{(a.nseg + G - 1) / G, unit_rows(a.nz, pair), a.n1, unit_rows(a.zpb1, pair),
             unit_rows(a.zpb2, pair), 0u};
  u.b1 = (unsigned)a.n1 * (unsigned)((u.rows + u.per1 - 1) / u.per1);
  return u;
}

// One series of a batch as the persistent kernel sees it.
struct SeriesDesc {
  const void *spec;     // complex64 [nbins]
  float *power;         // [nz][ld]
  int64_t nbins;
  int64_t ld;
  int64_t item_begin;   // first work item of this series
  int nseg;             // segments
  int nz;               // rows of this series' plane
  int row_off;          // first bank row used by this series
  int zpb;              // templates per work item of this series
};

struct BatchArgs {
  const SeriesDesc *desc;
  int nseries;
  int64_t total;        // work items
  unsigned long long *counter;
  const void *bank;
  const void *tw;
  int U, half, zpb;
  int grid;             // persistent blocks
  int bank_log2;        // mixed precision: bank scale
  const void *consts;   // mixed precision: per-lane constants
  int pair;             // as in OlsArgs
};

struct OlsVariant {
  const char *name;
  int L, T, G, nbuf;
  int precision;     // FDAS_FP32 (0), FDAS_MIXED_FP16 (1), FDAS_MIXED_BF16 (2)
  int split;         // 1: hi + lo split products (FDAS_FLAG_SPLIT)
  int pair;          // 1: has a pair form, used where the bank's rows mirror
  int detect_pair;   // 1: so has its detection form
  int zpb_target;    // templates per unit where the size of the GPU is not known:
                     // units of that many, or (0) near-equal ones of at most 40
  UnitModel model;   // of the time of a single-spectrum launch
  BatchModel batch_model;  // and of a batch
  LayoutDesc lay;
  int lds_bytes;
  hipError_t (*launch)(const OlsArgs &, hipStream_t);
  hipError_t (*launch_batch)(const BatchArgs &, hipStream_t);
  int (*batch_blocks_per_cu)(int pair);  // of the batch kernel that runs
  // occupancy of the single-spectrum kernel; detect: of its detection form
  int (*grid_blocks_per_cu)(int pair, int detect);
};

const OlsVariant *fp32_variants(int *count);
const OlsVariant *mixed_variants(int *count);
// (rows: bank rows; interbin: every second one at half-bin offsets)
hipError_t launch_bank_mixed(void *bank, const void *h, int rows, int interbin, int m, int L,
                             int precision, int split, hipStream_t s);
size_t mixed_consts_bytes(int L, int split);
hipError_t launch_mixed_consts(void *out, int L, int precision, int split, hipStream_t s);
hipError_t launch_bank_mixed_natural(c32 *dst, const void *bank, int nz, int L, int precision,
                                     int split, hipStream_t s);

// The 2048-point matrix-core kernel (FP16 and BF16, no split form).
const OlsVariant *mixed2048_variants(int *count);
size_t mixed2048_consts_bytes();
hipError_t launch_mixed2048_consts(void *out, int precision, hipStream_t s);
hipError_t launch_bank_mixed2048(void *bank, const void *h, int rows, int interbin, int m,
                                 int precision, hipStream_t s);
hipError_t launch_bank_mixed2048_natural(c32 *dst, const void *bank, int nz, int precision,
                                         hipStream_t s);

hipError_t launch_reset_counter(unsigned long long *counter, hipStream_t s);
hipError_t launch_templates(void *out, int rows, int m, double zmax, double dz, int interbin,
                            hipStream_t s);
hipError_t launch_twiddles(c32 *tw, int L, hipStream_t s);
hipError_t launch_bank(c32 *bank, const void *h, int rows, int interbin, int m,
                       const LayoutDesc &lay, hipStream_t s);
hipError_t launch_bank_natural(c32 *dst, const c32 *bank, int nz,
                               const LayoutDesc &lay, hipStream_t s);

}  // namespace fdas
