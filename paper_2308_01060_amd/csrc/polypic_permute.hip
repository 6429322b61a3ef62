// Particle-order permutations, for gfx950.
//
// The sort (section 3.1's per-step cell ordering) leaves every particle array in
// slot order; a caller that wants its own particle order back, or hands in data in
// that order, permutes whole rows of 4-byte elements:
//
//   gather   dst[r][i] = src[r][idx[i]]        (coalesced writes, indexed reads)
//   scatter  dst[r][idx[i]] = src[r][i]        (coalesced reads, indexed writes)
//   invert   inv[perm[i]] = i
#include <type_traits>

#include "polypic_internal.hpp"

namespace polypic {

namespace {

constexpr int kPermUnroll = 8;  // rows in flight per thread that goes through all of them
// Threads per workgroup; PR: rows of a group, 0 where a thread goes through all rows.
template <int PR>
constexpr int kPermBlock = PR ? 512 : 256;

// One thread per slot, the slots in XCD-contiguous order: the indexed side of neighbouring
// slots shares lines, which then meet in one L2.  The coalesced side is streamed past the
// caches, which the indexed side uses.
// A few rows (PR = 0): a thread goes through all of them, so that its slot's index is read once;
// kPermUnroll rows are in flight together, and the rest, after the last whole kPermUnroll, one
// at a time and through the caches.  More rows: the launch sweeps the slots of one group of PR
// rows before the next (blockIdx.y), and the index is read once per group.  What a scatter
// writes decides: the lines that a slot's neighbours in order have not filled yet must stay in
// the caches until they do, over all rows that are open together, and few rows open keep more
// of them there; more groups read the index more often.  So scatters go in groups of 2 rows
// from 9 rows on, and of 4 above 64, where the groups' own reads weigh more; gathers in groups
// of 4 above 16 rows.
// (Measured, us: threads that go through all rows in launch order; groups of 4 rows; as here.
// A set's order after a few steps from cells in row order, 4.19 M slots: 1 row gathered 18, 14
// and 12, scattered 17, 18 and 13; 9 rows gathered 109, 62 and 59, scattered 186, 103 and 97; 12
// rows scattered 275, 131 and 123; 24 rows gathered 300, 223 and 223, scattered 409, 269 and 251;
// 81 rows gathered 1037 and 750, scattered 1427 and 912.  In random order, scattered: 4 rows 202,
// 400 and 202; 12 rows of 1.77 M slots 333, 492 and 262; 81 rows 3918 and 2679.  In no change of
// order, where only the index and the launch differ, 4.19 M slots: 1 row gathered 11, 14 and 11,
// scattered 11, 17 and 11; 9 rows gathered 49, 58 and 46, scattered 52, 60 and 73; 24 rows
// scattered 173, 142 and 185; 81 rows gathered 500 and 553, scattered 547 and 488.)
int gather_group(int64_t rows) { return rows <= 16 ? 0 : 4; }
int scatter_group(int64_t rows) { return rows <= 8 ? 0 : rows <= 64 ? 2 : 4; }

struct PermSlot {
  int64_t i, p;  // slot, and the particle it indexes
};
template <int BS>
__device__ __forceinline__ bool perm_slot(const int32_t* __restrict__ idx, int64_t P, PermSlot& s) {
  s.i = block_chunks(kSchedXcd, gridDim.x).begin * BS + threadIdx.x;
  if (s.i >= P) return false;
  // an index outside [0, P) is clamped: a bad one gives wrong results, never a fault
  s.p = min(max((int64_t)idx[s.i], (int64_t)0), P - 1);
  return true;
}

// dst[r][i] = src[r][idx[i]]: indexed reads, coalesced writes.
template <int PR>
__global__ __launch_bounds__(kPermBlock<PR>) void gather_rows_kernel(const uint32_t* __restrict__ src,
                                                                 uint32_t* __restrict__ dst,
                                                                 const int32_t* __restrict__ idx,
                                                                 int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot<kPermBlock<PR>>(idx, P, at)) return;
  if constexpr (PR > 0) {
    for (int64_t r = (int64_t)blockIdx.y * PR; r < rows; r += (int64_t)gridDim.y * PR) {
      uint32_t v[PR];
#pragma unroll
      for (int k = 0; k < PR; ++k)
        if (r + k < rows) v[k] = src[(r + k) * P + at.p];
#pragma unroll
      for (int k = 0; k < PR; ++k)
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
template <int PR>
__global__ __launch_bounds__(kPermBlock<PR>) void scatter_rows_kernel(const uint32_t* __restrict__ src,
                                                                  uint32_t* __restrict__ dst,
                                                                  const int32_t* __restrict__ idx,
                                                                  int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot<kPermBlock<PR>>(idx, P, at)) return;
  if constexpr (PR > 0) {
    for (int64_t r = (int64_t)blockIdx.y * PR; r < rows; r += (int64_t)gridDim.y * PR) {
      uint32_t v[PR];
#pragma unroll
      for (int k = 0; k < PR; ++k)
        if (r + k < rows) v[k] = __builtin_nontemporal_load(src + (r + k) * P + at.i);
#pragma unroll
      for (int k = 0; k < PR; ++k)
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

template <int PR>
dim3 perm_grid(int64_t rows, int64_t P) {
  constexpr int BS = kPermBlock<PR>;
  const int64_t groups = PR > 0 ? (rows + PR - 1) / (PR > 0 ? PR : 1) : 1;
  return dim3((unsigned)((P + BS - 1) / BS), (unsigned)(groups < 65535 ? groups : 65535));
}

constexpr int kInvertBlock = 256;
__global__ __launch_bounds__(kInvertBlock) void invert_permutation_kernel(
    const int32_t* __restrict__ perm, int32_t* __restrict__ inv, int64_t P) {
  const int64_t i = (int64_t)blockIdx.x * kInvertBlock + threadIdx.x;
  if (i >= P) return;
  const int64_t p = min(max((int64_t)perm[i], (int64_t)0), P - 1);
  inv[p] = (int32_t)i;
}

}  // namespace

hipError_t launch_gather_rows(const void* src, void* dst, const int32_t* idx, int64_t rows,
                              int64_t P, hipStream_t stream) {
  if (P == 0 || rows == 0) return hipSuccess;
  const uint32_t* const s = static_cast<const uint32_t*>(src);
  uint32_t* const d = static_cast<uint32_t*>(dst);
  auto launch = [&](auto group) {
    constexpr int PR = group;
    gather_rows_kernel<PR><<<perm_grid<PR>(rows, P), kPermBlock<PR>, 0, stream>>>(s, d, idx, rows, P);
  };
  switch (gather_group(rows)) {
    case 0: launch(std::integral_constant<int, 0>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_scatter_rows(const void* src, void* dst, const int32_t* idx, int64_t rows,
                               int64_t P, hipStream_t stream) {
  if (P == 0 || rows == 0) return hipSuccess;
  const uint32_t* const s = static_cast<const uint32_t*>(src);
  uint32_t* const d = static_cast<uint32_t*>(dst);
  auto launch = [&](auto group) {
    constexpr int PR = group;
    scatter_rows_kernel<PR><<<perm_grid<PR>(rows, P), kPermBlock<PR>, 0, stream>>>(s, d, idx, rows, P);
  };
  switch (scatter_group(rows)) {
    case 0: launch(std::integral_constant<int, 0>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_invert_permutation(const int32_t* perm, int32_t* inv, int64_t P,
                                     hipStream_t stream) {
  if (P == 0) return hipSuccess;
  invert_permutation_kernel<<<(unsigned)((P + kInvertBlock - 1) / kInvertBlock), kInvertBlock, 0,
                              stream>>>(perm, inv, P);
  return hipGetLastError();
}

}  // namespace polypic
