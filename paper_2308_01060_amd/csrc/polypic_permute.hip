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

constexpr int kPermBlock = 512;
constexpr int kPermRows = 4;  // rows of a workgroup, in flight together

// One thread per slot of kPermRows rows.  The launch sweeps the slots of one group of rows
// before the next (blockIdx.y), with the slots in XCD-contiguous order: the indexed side of
// neighbouring slots shares lines, which then meet in one L2, and few rows are open at a
// time.  The coalesced side is streamed past the caches, which the indexed side uses.
// (Measured, 3 x 27 rows of 1.77 M in a sort's order, gather and scatter: 250 and 500 us
// with every thread going through all rows in launch order; 230 and 490 with groups of 4
// rows; 210 and 290 in XCD order as well.)
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
__global__ __launch_bounds__(kPermBlock) void gather_rows_kernel(const uint32_t* __restrict__ src,
                                                                 uint32_t* __restrict__ dst,
                                                                 const int32_t* __restrict__ idx,
                                                                 int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot(idx, P, at)) return;
  for (int64_t r = (int64_t)blockIdx.y * kPermRows; r < rows; r += (int64_t)gridDim.y * kPermRows) {
    uint32_t v[kPermRows];
#pragma unroll
    for (int k = 0; k < kPermRows; ++k)
      if (r + k < rows) v[k] = src[(r + k) * P + at.p];
#pragma unroll
    for (int k = 0; k < kPermRows; ++k)
      if (r + k < rows) __builtin_nontemporal_store(v[k], dst + (r + k) * P + at.i);
  }
}

// dst[r][idx[i]] = src[r][i]: coalesced reads, indexed writes.
__global__ __launch_bounds__(kPermBlock) void scatter_rows_kernel(const uint32_t* __restrict__ src,
                                                                  uint32_t* __restrict__ dst,
                                                                  const int32_t* __restrict__ idx,
                                                                  int64_t rows, int64_t P) {
  PermSlot at;
  if (!perm_slot(idx, P, at)) return;
  for (int64_t r = (int64_t)blockIdx.y * kPermRows; r < rows; r += (int64_t)gridDim.y * kPermRows) {
    uint32_t v[kPermRows];
#pragma unroll
    for (int k = 0; k < kPermRows; ++k)
      if (r + k < rows) v[k] = __builtin_nontemporal_load(src + (r + k) * P + at.i);
#pragma unroll
    for (int k = 0; k < kPermRows; ++k)
      if (r + k < rows) dst[(r + k) * P + at.p] = v[k];
  }
}

dim3 perm_grid(int64_t rows, int64_t P) {
  const int64_t groups = (rows + kPermRows - 1) / kPermRows;
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
  gather_rows_kernel<<<perm_grid(rows, P), kPermBlock, 0, stream>>>(
      static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), idx, rows, P);
  return hipGetLastError();
}

hipError_t launch_scatter_rows(const void* src, void* dst, const int32_t* idx, int64_t rows,
                               int64_t P, hipStream_t stream) {
  if (P == 0 || rows == 0) return hipSuccess;
  scatter_rows_kernel<<<perm_grid(rows, P), kPermBlock, 0, stream>>>(
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
