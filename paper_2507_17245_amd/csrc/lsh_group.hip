// LSH hash-and-group kernel (arXiv 2507.17245, Sec. 3.2 "similar columns identification" and Fig. 5; once per
// block as in Sec. 3.3). One workgroup per (batch, head, block of rows).
//
// For every channel column of the block: projection onto n_planes random directions -> sign bits -> Gray
// map -> integer hash; then the d hashes are ranked (ascending, ties by channel index) and the inverse of
// the rank is the block's channel permutation.
//
// The sign of a projection decides an integer, so its sum has a defining order that a CPU can repeat bit for
// bit: float, one fused multiply-add per row, rows ascending, starting at +0.
//
// Bound: the latency of reading the block (there are often fewer blocks than compute units). All of its rows
// are asked for at once by direct global->LDS loads, and the projection table is generated while they travel.
//   bf16   the projections are taken on the matrix pipe, from R split into two bf16 pieces (an entry is an integer of
//          17 bits times 2^-16: r1 = R rounded to bf16 and r2 = R - r1 hold it exactly), next to sum |q| |r1|,
//          which bounds how far that sum can be from the defining one; only sums inside the bound are
//          taken again the defining way.
//   float  the defining sums on the vector ALUs, from LDS.
// Measured (rows walked column by column in global memory, four at a time | now): bf16 H16 N200 d128 Br128
// 21.5 | 6.9 us, H16 N2048 d64 Br256 17 | 9.0, float H8 N2048 d64 Br128 13.8 | 5.7 us, float H8 N2048 d64 blocks of 64 rows
// 6.4 | 4.9 us.
#include "lsh_block.h"

namespace da {

// PARTS: not a table, but in a tensor like q the block's row of it at every part of part_rows rows.
template <typename T, int D, int BR, int THREADS, bool PARTS>
__global__ __launch_bounds__(THREADS) void lsh_group_kernel(
    const T* __restrict__ q, uint8_t* __restrict__ perm_out, uint32_t* __restrict__ hash_out,
    int N, int Tq, int n_planes, int gray_mode, uint64_t seed, int part_rows) {
  __shared__ LshLds<T, D, BR> lds;
  const int t = blockIdx.x % Tq;
  const size_t bh = blockIdx.x / Tq;
  const size_t at = PARTS ? (bh * N + (size_t)t * BR) * (D * sizeof(T)) : (size_t)blockIdx.x * D;
  lsh_block<T, D, BR, THREADS>(q + (bh * N + (size_t)t * BR) * D, min(BR, N - t * BR), n_planes, gray_mode, seed,
                      perm_out ? perm_out + at : nullptr, hash_out ? hash_out + at : nullptr, lds);
  if (PARTS && threadIdx.x < D)
    for (int r = part_rows; r < min(BR, N - t * BR); r += part_rows) perm_out[at + (size_t)r * (D * sizeof(T)) + threadIdx.x] = lds.perm[threadIdx.x];
}

template <typename T, int D, bool PARTS>
static hipError_t launch_rows(const T* q, const Problem& pb, uint8_t* perm_out, uint32_t* hash_out, int part_rows, hipStream_t stream) {
  const int Tq = (pb.N + pb.Br - 1) / pb.Br;
  const long long units = (long long)pb.B * pb.H * Tq;
#define DA_LSH_T(BR, THREADS)                                                                                                       \
  hipLaunchKernelGGL((lsh_group_kernel<T, D, BR, THREADS, PARTS>), dim3((unsigned)units), dim3(THREADS), 0, stream, q, perm_out, hash_out, \
                     pb.N, Tq, pb.n_planes, pb.gray_mode, pb.seed, part_rows)
#define DA_LSH(BR)                                                      \
  do {                                                                  \
    if constexpr (sizeof(T) == 2 || D == 128) {                         \
      if (wide) DA_LSH_T(BR, 512);                                      \
    }                                                                   \
    if constexpr (sizeof(T) == 2 || D == 64) {                          \
      if (!wide) DA_LSH_T(BR, 256);                                     \
    }                                                                   \
  } while (0)
  // Q blocks of 64, 128, 256 rows, K blocks (mirrored form) of 32, 64, 128. A sequence shorter than its block takes the
  // kernel of the shortest block that holds it: less LDS, so more workgroups on a CU (N44 Br256 d128 bf16 with 17
  // projections, 576 heads: 11 us as a block of 64, 15 walked in global memory).
  int rows = pb.Br;
  while (rows > 32 && pb.N <= rows / 2) rows /= 2;
  // Threads of a workgroup: 512 where the chip is not full without them, and for the float sums of 128 channels at any size
  // (four projections a thread, not eight; at 64 channels 256 threads have four each already, and barriers
  // of more waves cost more). us, 256 | 512 threads: bf16 d128 H16 N200 Br128 8.2 | 6.9, H16 N2048 Br256 15.8 | 10.9,
  // 1000 rows of 48 heads in blocks of 64 8.7 | 10.0; bf16 d64 H16 N2048 Br128 6.6 | 6.2, 1024 blocks 10.7 | 12.5; float d128
  // H8 N2048 Br128 8.8 | 6.6, 8192 blocks 154 | 139; float d64 H8 N2048 Br128 5.4 | 5.9.
  const bool wide = sizeof(T) == 2 ? units <= kComputeUnits : D == 128;
  switch (rows) {
    case 32: DA_LSH(32); break;
    case 64: DA_LSH(64); break;
    case 128: DA_LSH(128); break;
    case 256: DA_LSH(256); break;
    default: return hipErrorInvalidValue;
  }
#undef DA_LSH
#undef DA_LSH_T
  return hipGetLastError();
}

hipError_t launch_lsh_group(const void* q, int dtype, const Problem& pb, uint8_t* perm_out,
                            uint32_t* hash_out, hipStream_t stream, int part_rows) {
  if (part_rows && dtype == 0 && pb.d == 64) return launch_rows<bf16, 64, true>((const bf16*)q, pb, perm_out, hash_out, part_rows, stream);
  if (part_rows && dtype == 0 && pb.d == 128) return launch_rows<bf16, 128, true>((const bf16*)q, pb, perm_out, hash_out, part_rows, stream);
  if (part_rows) return hipErrorInvalidValue;
  if (dtype == 0 && pb.d == 64) return launch_rows<bf16, 64, false>((const bf16*)q, pb, perm_out, hash_out, 0, stream);
  if (dtype == 0 && pb.d == 128) return launch_rows<bf16, 128, false>((const bf16*)q, pb, perm_out, hash_out, 0, stream);
  if (dtype == 1 && pb.d == 64) return launch_rows<float, 64, false>((const float*)q, pb, perm_out, hash_out, 0, stream);
  if (dtype == 1 && pb.d == 128) return launch_rows<float, 128, false>((const float*)q, pb, perm_out, hash_out, 0, stream);
  return hipErrorInvalidValue;
}

}  // namespace da
