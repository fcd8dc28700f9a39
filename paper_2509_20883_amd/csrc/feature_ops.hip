// Feature transforms fused over many columns (gfx950): bucketize and mod
// (RecIS, "Bucketize and Mod" among the benchmarked operators: a model holds
// dozens to hundreds of them, and one launch for all columns replaces one
// launch per column).
//
// Column c holds elements [col_off[c], col_off[c+1]) of one flat array.  A
// block takes 1024 consecutive elements and copies the column offsets (and
// the boundary offsets or moduli) to LDS in one coalesced trip, counting on
// the way the columns that end at or before its first element: that count is
// its first column, so no search is in the chain.  When the range lies inside
// one column (the usual case: columns are much longer than a block) it stages
// that column's boundaries in LDS and searches there for its four elements at
// once; otherwise each element searches its column, then the boundaries in
// global memory (L1 / L2).
//   bucketize: out = number of boundaries b <= x (upper bound)
//   mod:       out = x mod m in [0, m) (-1 for a modulus <= 0)
#include "device_common.h"

namespace rs {

constexpr int kFeatItems = 4;
constexpr int kFeatTile = kBlock * kFeatItems;  // 1024 elements per block
constexpr int kLdsBounds = 4096;               // boundaries staged in LDS

// Largest c in [lo, hi] with off[c] <= i (off nondecreasing, off[lo] <= i).
template <typename P>
__device__ inline int column_of(P off, int lo, int hi, int64_t i) {
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Upper bound: the index of the first of b[0, nb) (nondecreasing) with
// x < b, or nb -- the number of boundaries b <= x, and nb for a NaN x (which
// compares below no boundary).
template <typename P>
__device__ inline int64_t upper_bound_f(P b, int64_t nb, float x) {
  int64_t lo = 0, hi = nb;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (x < b[mid]) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Up to kLdsCols column offsets (and one per-column array: boundary offsets
// or moduli) are copied to LDS in one coalesced trip; with more columns the
// searches run in global memory (L1 / L2).  Returns the column of element b0:
// the number of columns c < ncols - 1 with col_off[c + 1] <= b0.
constexpr int kLdsCols = 1024;

template <typename T>
__device__ inline int stage_columns(const int64_t* __restrict__ col_off, const T* __restrict__ aux, int naux, int ncols,
                                    int64_t b0, int64_t* lco, T* laux, int* wsum) {
  constexpr int PT = kLdsCols / kBlock;
  int64_t o[PT];
  T a[PT];
#pragma unroll
  for (int j = 0; j < PT; ++j) {  // both arrays in flight together
    const int c = threadIdx.x + j * kBlock;
    o[j] = c <= ncols ? col_off[c] : INT64_MAX;
    a[j] = c < naux ? aux[c] : T(0);
  }
  int before = 0;
#pragma unroll
  for (int j = 0; j < PT; ++j) {
    const int c = threadIdx.x + j * kBlock;
    if (c <= ncols) lco[c] = o[j];
    if (c < naux) laux[c] = a[j];
    before += __popcll(__ballot(c >= 1 && c < ncols && o[j] <= b0));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x / kWave] = before;
  __syncthreads();
  int c0 = 0;
#pragma unroll
  for (int q = 0; q < kBlock / kWave; ++q) c0 += wsum[q];
  return c0;
}

// The columns [c0, c1] of a block's elements [b0, b1).  Where the offsets do
// not fit LDS both are searched in global memory.
struct ColSpan {
  int c0, c1;
};

template <typename T>
__device__ inline ColSpan column_span(const int64_t* __restrict__ col_off, const T* __restrict__ aux, int naux,
                                      int ncols, int64_t b0, int64_t b1, bool lds, int64_t* lco, T* laux, int* wsum) {
  ColSpan sp;
  if (lds) {
    sp.c0 = stage_columns(col_off, aux, naux, ncols, b0, lco, laux, wsum);
    sp.c1 = b1 <= lco[sp.c0 + 1] ? sp.c0 : column_of(static_cast<const int64_t*>(lco), sp.c0, ncols - 1, b1 - 1);
  } else {
    sp.c0 = column_of(col_off, 0, ncols - 1, b0);
    sp.c1 = column_of(col_off, sp.c0, ncols - 1, b1 - 1);
  }
  return sp;
}

// Bound by the latency of its chain (a block per 1024 elements, all resident
// up to ~2M elements): the column offsets, the boundaries, the searches.  The
// first column is counted while staging instead of searched, and the four
// elements of a thread search together, one LDS trip per step for all four:
// 8.9 -> 8.2 us for 100 columns of 10,000 values with 63 boundaries each (the
// launch of 977 blocks and three dependent memory trips remain).
__global__ __launch_bounds__(kBlock) void k_bucketize(const float* __restrict__ values, int64_t n,
                                                      const int64_t* __restrict__ col_off, int ncols,
                                                      const float* __restrict__ bnd,
                                                      const int64_t* __restrict__ bnd_off, int64_t* __restrict__ out) {
  __shared__ float lb[kLdsBounds];
  __shared__ int64_t lco[kLdsCols];
  __shared__ int64_t lbo[kLdsCols];
  __shared__ int wsum[kBlock / kWave];
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * kFeatTile;
  const int64_t b1 = min(b0 + kFeatTile, n);
  float x[kFeatItems];
#pragma unroll
  for (int k = 0; k < kFeatItems; ++k) {  // in flight while the offsets are staged
    const int64_t i = b0 + k * kBlock + threadIdx.x;
    x[k] = i < b1 ? values[i] : 0.0f;
  }
  const bool lds = ncols < kLdsCols;  // ncols + 1 offsets fit
  const ColSpan sp = column_span(col_off, bnd_off, ncols + 1, ncols, b0, b1, lds, lco, lbo, wsum);
  const int c0 = sp.c0, c1 = sp.c1;
  if (c0 == c1) {  // block-uniform
    const int64_t o = lds ? lbo[c0] : bnd_off[c0];
    const int64_t nb = (lds ? lbo[c0 + 1] : bnd_off[c0 + 1]) - o;
    if (nb <= kLdsBounds) {
      for (int64_t j = threadIdx.x; j < nb; j += kBlock) lb[j] = bnd[o + j];
      __syncthreads();
      // the answer of element k is in [base[k], base[k] + len]; every step
      // takes half = ceil(len / 2) off, for all elements alike
      int base[kFeatItems] = {};
      int len = static_cast<int>(max(nb, int64_t(0)));
      while (len > 0) {  // block-uniform
        const int half = (len + 1) >> 1;
#pragma unroll
        for (int k = 0; k < kFeatItems; ++k) {
          const bool above = !(x[k] < lb[base[k] + half - 1]);
          base[k] += above ? half : 0;
        }
        len -= half;
      }
#pragma unroll
      for (int k = 0; k < kFeatItems; ++k) {
        const int64_t i = b0 + k * kBlock + threadIdx.x;
        if (i < b1) out[i] = base[k];
      }
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < kFeatItems; ++k) {
    const int64_t i = b0 + k * kBlock + threadIdx.x;
    if (i >= b1) continue;
    const int c = lds ? column_of(static_cast<const int64_t*>(lco), c0, c1, i) : column_of(col_off, c0, c1, i);
    const int64_t o = lds ? lbo[c] : bnd_off[c];
    const int64_t e = lds ? lbo[c + 1] : bnd_off[c + 1];
    out[i] = upper_bound_f(bnd + o, e - o, x[k]);
  }
}

// floor(x mod m), m in [1, 2^63), with inv = floor((2^64 - 1) / m): the
// quotient estimate umulhi(|x|, inv) is the quotient or one less (inv is
// above 2^64 / m - 1 and |x| < 2^64), so one conditional subtraction ends it
// (Barrett 1986).
__device__ inline int64_t floor_mod(int64_t x, uint64_t m, uint64_t inv) {
  const uint64_t u = x < 0 ? 0ull - static_cast<uint64_t>(x) : static_cast<uint64_t>(x);
  uint64_t r = u - __umul64hi(u, inv) * m;
  r = r >= m ? r - m : r;
  return static_cast<int64_t>(x < 0 && r != 0 ? m - r : r);
}

// Streams 16 bytes per element, but a 64-bit division per element (~130
// instructions) bound it by arithmetic: a block takes the reciprocal of each
// of its columns once (one thread per column, at most kBlock columns) and the
// elements multiply: 29.3 -> 19.7 us for 6M ids in 300 columns (96 MB, 4.9
// TB/s).  A block over more columns (columns of fewer than 4 elements) divides
// per element.
__global__ __launch_bounds__(kBlock) void k_mod(const int64_t* __restrict__ values, int64_t n,
                                                const int64_t* __restrict__ col_off, int ncols,
                                                const int64_t* __restrict__ moduli, int64_t* __restrict__ out) {
  __shared__ int64_t lco[kLdsCols];
  __shared__ int64_t lm[kLdsCols];
  __shared__ int64_t sm[kBlock];    // moduli of the block's columns
  __shared__ uint64_t sinv[kBlock];  // their reciprocals
  __shared__ int wsum[kBlock / kWave];
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * kFeatTile;
  const int64_t b1 = min(b0 + kFeatTile, n);
  int64_t x[kFeatItems];
#pragma unroll
  for (int k = 0; k < kFeatItems; ++k) {
    const int64_t i = b0 + k * kBlock + threadIdx.x;
    x[k] = i < b1 ? values[i] : 0;
  }
  const bool lds = ncols < kLdsCols;
  const ColSpan sp = column_span(col_off, moduli, ncols, ncols, b0, b1, lds, lco, lm, wsum);
  const int c0 = sp.c0, c1 = sp.c1;
  const bool few = c1 - c0 < kBlock;  // block-uniform
  if (few) {
    const int c = c0 + threadIdx.x;
    if (c <= c1) {
      const int64_t m = lds ? lm[c] : moduli[c];
      sm[threadIdx.x] = m;
      sinv[threadIdx.x] = m > 0 ? ~0ull / static_cast<uint64_t>(m) : 0ull;
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < kFeatItems; ++k) {
    const int64_t i = b0 + k * kBlock + threadIdx.x;
    if (i >= b1) continue;
    int c = c0;
    if (c0 != c1) c = lds ? column_of(static_cast<const int64_t*>(lco), c0, c1, i) : column_of(col_off, c0, c1, i);
    const int64_t m = few ? sm[c - c0] : lds ? lm[c] : moduli[c];
    const uint64_t inv = few ? sinv[c - c0] : m > 0 ? ~0ull / static_cast<uint64_t>(m) : 0ull;
    out[i] = m > 0 ? floor_mod(x[k], static_cast<uint64_t>(m), inv) : -1;  // a modulus <= 0 is no bucket
  }
}

hipError_t launch_bucketize(const float* values, int64_t n, const int64_t* col_off, int ncols, const float* bnd,
                            const int64_t* bnd_off, int64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_bucketize<<<grid_for(n, kFeatTile, 1ll << 31), kBlock, 0, s>>>(values, n, col_off, ncols, bnd, bnd_off, out);
  return hipGetLastError();
}

hipError_t launch_mod(const int64_t* values, int64_t n, const int64_t* col_off, int ncols, const int64_t* moduli,
                      int64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_mod<<<grid_for(n, kFeatTile, 1ll << 31), kBlock, 0, s>>>(values, n, col_off, ncols, moduli, out);
  return hipGetLastError();
}

}  // namespace rs
