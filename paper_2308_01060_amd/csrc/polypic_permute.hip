// Particle-order permutations, for gfx950.
//
// The sort (section 3.1's per-step cell ordering) leaves every particle array in
// slot order; a caller that wants its own particle order back, or hands in data in
// that order, permutes whole rows of 4-byte elements:
//
//   gather   dst[r][i] = src[r][idx[i]]        (coalesced writes, indexed reads)
//   scatter  dst[r][idx[i]] = src[r][i]        (coalesced reads, indexed writes)
//   invert   inv[perm[i]] = i
#include "polypic_internal.hpp"

namespace polypic {

namespace {

constexpr int kPermBlock = 256;
constexpr int kPermUnroll = 8;      // whole: rows in flight per thread
// groups: rows of a workgroup, in flight together
constexpr int kGatherRows = 4, kScatterRows = 6;
constexpr int64_t kPermWhole = 64;  // most rows that a thread goes through by itself

// One thread per slot, the slots in XCD-contiguous order: the indexed side of neighbouring
// slots shares lines, which then meet in one L2.  The coalesced side is streamed past the
// caches, which the indexed side uses.
// Up to kPermWhole rows (kGroups false) a thread goes through all rows, so that its slot's
// index is read once; kPermUnroll rows are in flight together, and the rest, after the last
// whole kPermUnroll, one at a time and through the caches: where the index is in no order the
// lines that one row's stores leave part-written have to stay in the caches until the rest of
// them comes, and several rows at once are too many.  With more rows (kGroups) the launch
// sweeps the slots of one group of rows before the next (blockIdx.y), so that few rows are
// open at a time; the index is read once per group.
// (Measured, a set's sort order from cells in row order, then a random order; us, by threads
// that go through all rows in launch order, in groups of 4 rows, and as here.  4.19 M slots: 1
// row gathered 10, 14 and 10, scattered 11, 17 and 11; 4 rows scattered 24, 27 and 23, in
// random order 202, 400 and 202; 9 rows gathered 47, 56 and 47; 81 rows gathered 572, 518 and
// 510, scattered 630, 518 and 513, in random order 13160, 6909 and 6979.  1.77 M slots in
// random order, scattered: 12 rows 330, 494 and 326; 40 rows 1225, 1408 and 1186, where groups
// of 6 take 1463; 81 rows 3918, 2679 and 2693.  Groups of 4 and of 6 rows, 81 rows of 1.77 M
// slots whose order differs by a few hundred slots: gathered 259 and 283, scattered 332 and 314.)
struct PermSlot {
  int64_t i, p;  // slot, and the particle it indexes
};
__device__ __forceinline__ bool perm_slot(const int32_t* __restrict__ idx, int64_t P, PermSlot& s) {
  s.i = block_chunks(kSchedXcd, gridDim.x).begin * kPermBlock + threadIdx.x;
  if (s.i >= P) return false;
  // an index outside [0, P) is clamped: a bad one gives wrong results, never a fault
  s.p = min(max((int64_t)idx[s.i], (int64_t)0), P - 1);
  return true;
}

// dst[r][i] = src[r][idx[i]]: indexed reads, coalesced writes.
template <bool kGroups>
__global__ __launch_bounds__(kPermBlock) void gather_rows_kernel(const uint32_t* __restrict__ src,
                                                                 uint32_t* __restrict__ dst,
                                                                 const int32_t* __restrict__ idx,
                                                                 int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot(idx, P, at)) return;
  if constexpr (kGroups) {
    for (int64_t r = (int64_t)blockIdx.y * kGatherRows; r < rows; r += (int64_t)gridDim.y * kGatherRows) {
      uint32_t v[kGatherRows];
#pragma unroll
      for (int k = 0; k < kGatherRows; ++k)
        if (r + k < rows) v[k] = src[(r + k) * P + at.p];
#pragma unroll
      for (int k = 0; k < kGatherRows; ++k)
        if (r + k < rows) __builtin_nontemporal_store(v[k], dst + (r + k) * P + at.i);
    }
  } else {
    int64_t r = 0;
    for (; r + kPermUnroll <= rows; r += kPermUnroll) {
      uint32_t v[kPermUnroll];
#pragma unroll
      for (int k = 0; k < kPermUnroll; ++k) v[k] = src[(r + k) * P + at.p];
#pragma unroll
      for (int k = 0; k < kPermUnroll; ++k)
        __builtin_nontemporal_store(v[k], dst + (r + k) * P + at.i);
    }
    for (; r < rows; ++r) __builtin_nontemporal_store(src[r * P + at.p], dst + r * P + at.i);
  }
}

// dst[r][idx[i]] = src[r][i]: coalesced reads, indexed writes.
template <bool kGroups>
__global__ __launch_bounds__(kPermBlock) void scatter_rows_kernel(const uint32_t* __restrict__ src,
                                                                  uint32_t* __restrict__ dst,
                                                                  const int32_t* __restrict__ idx,
                                                                  int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot(idx, P, at)) return;
  if constexpr (kGroups) {
    for (int64_t r = (int64_t)blockIdx.y * kScatterRows; r < rows; r += (int64_t)gridDim.y * kScatterRows) {
      uint32_t v[kScatterRows];
#pragma unroll
      for (int k = 0; k < kScatterRows; ++k)
        if (r + k < rows) v[k] = __builtin_nontemporal_load(src + (r + k) * P + at.i);
#pragma unroll
      for (int k = 0; k < kScatterRows; ++k)
        if (r + k < rows) dst[(r + k) * P + at.p] = v[k];
    }
  } else {
    int64_t r = 0;
    for (; r + kPermUnroll <= rows; r += kPermUnroll) {
      uint32_t v[kPermUnroll];
#pragma unroll
      for (int k = 0; k < kPermUnroll; ++k)
        v[k] = __builtin_nontemporal_load(src + (r + k) * P + at.i);
#pragma unroll
      for (int k = 0; k < kPermUnroll; ++k) dst[(r + k) * P + at.p] = v[k];
    }
    for (; r < rows; ++r) dst[r * P + at.p] = src[r * P + at.i];
  }
}

dim3 perm_grid(int64_t rows, int64_t P, int per) {
  const int64_t groups = rows <= kPermWhole ? 1 : (rows + per - 1) / per;
  return dim3((unsigned)((P + kPermBlock - 1) / kPermBlock),
              (unsigned)(groups < 65535 ? groups : 65535));
}

__global__ __launch_bounds__(kPermBlock) void invert_permutation_kernel(
    const int32_t* __restrict__ perm, int32_t* __restrict__ inv, int64_t P) {
  const int64_t i = (int64_t)blockIdx.x * kPermBlock + threadIdx.x;
  if (i >= P) return;
  const int64_t p = min(max((int64_t)perm[i], (int64_t)0), P - 1);
  inv[p] = (int32_t)i;
}

}  // namespace

hipError_t launch_gather_rows(const void* src, void* dst, const int32_t* idx, int64_t rows,
                              int64_t P, hipStream_t stream) {
  if (P == 0 || rows == 0) return hipSuccess;
  (rows <= kPermWhole ? gather_rows_kernel<false> : gather_rows_kernel<true>)
      <<<perm_grid(rows, P, kGatherRows), kPermBlock, 0, stream>>>(
          static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), idx, rows, P);
  return hipGetLastError();
}

hipError_t launch_scatter_rows(const void* src, void* dst, const int32_t* idx, int64_t rows,
                               int64_t P, hipStream_t stream) {
  if (P == 0 || rows == 0) return hipSuccess;
  (rows <= kPermWhole ? scatter_rows_kernel<false> : scatter_rows_kernel<true>)
      <<<perm_grid(rows, P, kScatterRows), kPermBlock, 0, stream>>>(
          static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), idx, rows, P);
  return hipGetLastError();
}

hipError_t launch_invert_permutation(const int32_t* perm, int32_t* inv, int64_t P,
                                     hipStream_t stream) {
  if (P == 0) return hipSuccess;
  invert_permutation_kernel<<<(unsigned)((P + kPermBlock - 1) / kPermBlock), kPermBlock, 0,
                              stream>>>(perm, inv, P);
  return hipGetLastError();
}

}  // namespace polypic
