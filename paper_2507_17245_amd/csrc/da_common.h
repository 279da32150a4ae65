// Shared declarations of the gfx950 DistrAttention library (device helpers + kernel launchers).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <numeric>

namespace da {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr int kBc = 64;          // key/value rows per tile of the key pre-pass and the default of the attention kernels
constexpr int kKtPad = 128;      // K^T rows are padded to a multiple of the largest key tile
constexpr int kMaxPlanes = 32;   // sign bits per hash

// Projection matrix entry (plane p, row r) of the LSH stage (Sec. 3.2: a fixed random matrix).
// Counter-based: mix a 64-bit counter, add its four 16-bit fields, centre. The value is an
// integer in [-131070, 131070] times 2^-16, so float holds it exactly on host and device.
__host__ __device__ inline float hyperplane_entry(uint64_t seed, uint32_t p, uint32_t r) {
  uint64_t z = seed + 0x9E3779B97F4A7C15ULL * (((uint64_t)p << 32) + (uint64_t)r + 1ULL);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  z ^= z >> 31;
  int sum = (int)(z & 0xFFFF) + (int)((z >> 16) & 0xFFFF) + (int)((z >> 32) & 0xFFFF) + (int)(z >> 48);
  return (float)(sum - 131070) * (1.0f / 65536.0f);
}

// Hash of a channel from the sign word of its projections (Sec. 3.2). gray_mode 1: the Gray code
// of the sign word (literal table lookup); otherwise the position of the sign word in the Gray
// sequence, so that hashes differing by one belong to sign words differing in one projection.
__host__ __device__ inline uint32_t lsh_hash_of_code(uint32_t code, int gray_mode) {
  if (gray_mode == 1) return code ^ (code >> 1);
  uint32_t h = code;
  h ^= h >> 1; h ^= h >> 2; h ^= h >> 4; h ^= h >> 8; h ^= h >> 16;
  return h;
}

// Projections whose sign the matrix pipe leaves in doubt: taken again by their defining sum (float, one fused multiply-add
// per row, rows ascending, from +0). Lane `who` doubts the sign of channel 4*(who/16) + i of the wave's 16, projection
// who%16, if doubt[i]. x_at(row, channel of the 16) is the block's entry; a projection's entries are r1 + r2 (exact),
// [projection][rpad]. Usually there are one to three in a wave:
//   one, of 64 rows   is summed by the whole wave: lane = row while the entries are read, the chain takes them lane by lane.
//                     Three instructions a row, half of what follows (short forward H12 N197 B64 28.3 -> 26.8 us).
//   a few             go to a lane each and are summed at once (by the whole wave, 4.2 us for each at 256 rows).
//   many              come with channels of zeros, which leave every projection in doubt: each lane walks the rows for its
//                     own four channels (by the whole wave, a block of zeros took a millisecond).
template <typename X>
__device__ inline void settle_doubts(const bool (&doubt)[4], bool (&positive)[4], int rows, const bf16* r1, const bf16* r2, int rpad, X x_at) {
  const int lane = threadIdx.x & 63;
  uint64_t masks[4];
  int count = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    masks[i] = __builtin_amdgcn_ballot_w64(doubt[i]);
    count += __builtin_popcountll(masks[i]);
  }
  auto entries = [&](int at, float (&r)[8]) {
    const s16x8 a = *(const s16x8*)(r1 + at), b = *(const s16x8*)(r2 + at);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      r[j] = __builtin_bit_cast(float, (uint32_t)(uint16_t)a[j] << 16) + __builtin_bit_cast(float, (uint32_t)(uint16_t)b[j] << 16);
  };
  if (count > 12) {
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int r0 = 0; r0 < rows; r0 += 8) {
      float r[8];
      entries((lane & 15) * rpad + r0, r);
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = __builtin_fmaf((float)x_at(r0 + j, 4 * (lane >> 4) + i), r[j], sum[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (doubt[i]) positive[i] = sum[i] > 0.0f;
    return;
  }
  if (count == 1 && rows == 64) {
    const int i = masks[0] != 0 ? 0 : masks[1] != 0 ? 1 : masks[2] != 0 ? 2 : 3;
    const int who = __builtin_ctzll(masks[0] | masks[1] | masks[2] | masks[3]);
    const int xi = __builtin_bit_cast(int, (float)x_at(lane, 4 * (who >> 4) + i));
    const int ri = __builtin_bit_cast(int, (float)r1[(who & 15) * rpad + lane] + (float)r2[(who & 15) * rpad + lane]);
    float sum = 0.0f;
#pragma unroll 1
    for (int k0 = 0; k0 < 64; k0 += 16) {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        sum = __builtin_fmaf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, k0 + j)),
                             __builtin_bit_cast(float, __builtin_amdgcn_readlane(ri, k0 + j)), sum);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (doubt[j]) positive[j] = sum > 0.0f;
    return;
  }
  int mine = 0, n = 0;   // the n-th doubt goes to lane n (the others repeat something)
#pragma unroll
  for (int i = 0; i < 4; ++i)
    for (uint64_t left = masks[i]; left != 0; left &= left - 1, ++n) mine = lane == n ? __builtin_ctzll(left) << 2 | i : mine;
  const int who = mine >> 2, ch = 4 * (who >> 4) + (mine & 3);
  float sum = 0.0f;
#pragma unroll 1
  for (int r0 = 0; r0 < rows; r0 += 32) {
    float r[4][8], x[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) x[j] = (float)x_at(r0 + j, ch);
#pragma unroll
    for (int j = 0; j < 4; ++j) entries((who & 15) * rpad + r0 + 8 * j, r[j]);
#pragma unroll
    for (int j = 0; j < 32; ++j) sum = __builtin_fmaf(x[j], r[j >> 3][j & 7], sum);
  }
  uint64_t up = __builtin_amdgcn_ballot_w64(sum > 0.0f);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    for (uint64_t left = masks[i]; left != 0; left &= left - 1, up >>= 1)
      if (lane == __builtin_ctzll(left)) positive[i] = up & 1;
}

// Causal tiles issued longest first over all heads: which tile (0 = the longest) comes at place `at` of a head's `tiles`
// ones, with the second round of workgroups (one per compute unit) in the opposite order: the compute unit that got the
// longest tile of the first round gets the shortest of the second, where it would otherwise get the longest again. The units'
// sums then differ by a round's spread instead of twice that, which is more than the workgroups that follow even out (at
// 1024 of them the third and fourth round are a third of the work, at 512 there is none). With more heads than half the
// compute units a round holds one tile of a head and nothing is reversed.
constexpr int kComputeUnits = 256;
__device__ inline int paired_tile(int at, int heads, int tiles) {
  const int round = heads < kComputeUnits ? kComputeUnits / heads : 1;
  return at >= round && at < 2 * round ? min(2 * round, tiles) - 1 - (at - round) : at;
}

// Exchange between the wave halves: v_permlane32_swap swaps the upper 32 lanes of its first
// operand with the lower 32 lanes of its second; fed the same value twice it leaves, in every
// lane, the values of lanes l % 32 (first operand) and l % 32 + 32 (second operand). Written as
// inline asm with both registers read-write: the builtin's second result was dropped by the
// compiler when both inputs were the same value. The s_nop covers the VALU-write -> permlane
// read hazard, which the compiler cannot see inside an asm block.
__device__ inline void half_pair(float x, float& lo, float& hi) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  lo = a;
  hi = b;
}
__device__ inline float half_swap_max(float x) {
  float lo, hi;
  half_pair(x, lo, hi);
  return fmaxf(lo, hi);
}
__device__ inline float half_swap_sum(float x) {
  float lo, hi;
  half_pair(x, lo, hi);
  return lo + hi;
}

// Behind the K^T copy the key pre-pass leaves the projection matrix of the LSH stage (Sec. 3.2),
// split into two bf16 pieces r1 + r2 = R, for the attention kernel's own LSH stage at d = 64,
// which otherwise generates it again in every workgroup: a header (seed, projections, block rows)
// at offset 0 and, from offset kRtabHead on, the two pieces [16][Br + 8] bf16, each padded to a
// whole number of 1 KB blocks (the unit of a direct load into LDS).
struct RtabHeader {
  uint64_t seed;
  int32_t n_planes, Br;
};
constexpr int kRtabHead = 1024;
constexpr int rtab_piece_bytes(int Br) { return (16 * (Br + 8) * 2 + 1023) / 1024 * 1024; }
constexpr int kRtabBytes = kRtabHead + 2 * rtab_piece_bytes(256);
// bytes of the K^T copy itself: [B][Hkv][d][Npad] half
inline size_t kt_copy_bytes(int B, int Hkv, int d, int Nk) {
  const size_t npad = (size_t)((Nk + kKtPad - 1) / kKtPad) * kKtPad;
  return ((size_t)B * Hkv * d * npad * 2 + 255) & ~(size_t)255;
}

// A barrier for what the waves have written to LDS and read from it themselves. __syncthreads waits for every load in flight
// besides, those into LDS for later among them (so does a fence for LDS alone).
__device__ inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Problem {
  int B, H, Hkv, N, d, Br, n_groups, causal, n_planes, gray_mode;
  uint64_t seed;
  float scale;
  int Nk;     // keys / values per head (N is the number of queries); causal: key n is visible
              // to query i iff n <= i + (Nk - N)
  int side;   // 0: sample Q, fuse K, one grouping per Q block; 1: sample K, fuse Q, one grouping
              // per K block of Bc rows (float-arithmetic kernel)
  int Bc;     // rows of a K block (only side 1 depends on it)
  float* lse; // optional device [B][H][N]: log-sum-exp of every row's visible scores (natural log)
  uint8_t* perm_w = nullptr;   // optional device [B][H][Tq][d]: where the attention kernel's own LSH
                               // stage leaves its table
  bool group_in_kernel = false;   // float forward: the attention kernel groups its Q blocks itself (attn_f32_groups)
  // bf16 forward with the key tiles of a Q block dealt out to n_split workgroups: their sums, float
  // [n_split][B][H][N][d], and (reference, row sum) pairs, float [n_split][B][H][N][2], exp2 domain
  int n_split = 1;
  int rows = 0;   // query rows of a workgroup where the table is given and they are not a Q block's (Q~ K^T; attn_bf16_shared_rows, attn_bf16_grouped_rows)
  bool table_in_o = false;   // the LSH kernel has left every such workgroup its row of the table in o, at its first output row
  float* part_o = nullptr;
  float* part_stat = nullptr;
};

// Q blocks that read the same keys, per XCD and in eighths (12: one and a half), in a bf16 forward of up to 8 blocks per compute
// unit: workgroup ids go round-robin over the 8 XCDs, causal blocks one after the other over all heads, others in a
// range of heads per XCD where there are a multiple of 8 of them. Two or more find each other's tiles in the L2.
inline int blocks_sharing_l2(const Problem& pb, int rows) {
  const int Tq = (pb.N + rows - 1) / rows, heads = pb.B * pb.H, mine = pb.H / pb.Hkv * Tq;
  if (!pb.causal) return (long long)heads * Tq % 8 == 0 ? 8 * mine : mine;
  return std::max(mine, Tq * std::gcd(heads, 8));
}

// Launchers (defined next to their kernels). All return hipError_t of the launch.
// part_rows (bf16): perm_out is no table but a tensor like q, where every part_rows rows of a block begin with its row of the table.
hipError_t launch_lsh_group(const void* q, int dtype, const Problem& pb, uint8_t* perm_out,
                            uint32_t* hash_out, hipStream_t stream, int part_rows = 0);
// K [B][Hkv][Nk][d] bf16 -> K^T [B][Hkv][d][Npad] half (Npad = Nk rounded up to kKtPad), for the distr path,
// followed at kt_copy_bytes() by the projection-matrix table (kRtabBytes) for pb's seed, n_planes and Br.
hipError_t launch_kt_prepass(const void* k, void* kt, const Problem& pb, hipStream_t stream);
// distr != 0: S^ with the per-block permutation table `perm` [B][H][Tq][d] (null: grouped in the kernel),
// as Q_r K_f^T from the transposed keys `kt` written by launch_kt_prepass (k itself is then unused; the
// table behind the copy is used when its header matches the call), or, without `kt`, as Q~ K^T.
// With pb.n_split > 1 (never with kt) launch_attn_bf16_combine follows.
hipError_t launch_attn_bf16(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                            const void* kt, const Problem& pb, int distr, hipStream_t stream);
hipError_t launch_attn_f32(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                           const Problem& pb, int dtype, int distr, hipStream_t stream);
bool attn_f32_groups(const Problem& pb, int dtype);   // float forward: the kernel can group its Q blocks itself
bool attn_bf16_supported(const Problem& pb, int distr);
// The rules of the bf16 forward (attn_bf16.hip): whether S^ is taken as Q~ K^T (have_kt: the transposed keys are at
// hand; n_split: the shares it would be cut into), and into how many shares the keys of a Q block are cut when the
// product is that one or the exact one.
bool attn_bf16_replicated(const Problem& pb, bool have_kt, int n_split);
bool attn_bf16_light(const Problem& pb);   // Q~ K^T is good enough to run where there is no room for the transposed copy
int attn_bf16_splits(const Problem& pb, int distr);
int attn_bf16_shared_rows(const Problem& pb);   // query rows of a grouped call's workgroups when its keys are dealt out
int attn_bf16_grouped_rows(const Problem& pb);  // the same when they stay together, fewer than a Q block's (0: a Q block's)
int attn_bf16_exact_rows(const Problem& pb);   // query rows of an exact call's workgroups, in the place of Br
// Few query rows against many keys (decoding): a kernel of its own, with its own number of shares.
bool attn_bf16_few_rows(const Problem& pb, int distr);
int attn_bf16_few_splits(const Problem& pb);
hipError_t launch_attn_bf16_few(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                                const Problem& pb, int distr, hipStream_t stream);
// Short sequences at d = 64: a workgroup per head.
bool attn_bf16_short(const Problem& pb, int distr);
hipError_t launch_attn_bf16_short(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                                  const Problem& pb, int distr, hipStream_t stream);
hipError_t launch_attn_bf16_combine(void* o, const Problem& pb, hipStream_t stream);
// Backward in float arithmetic (float tensors): dq [B][H][N][d], dk and dv
// [B][Hkv][Nk][d] from the forward's inputs, its output o, the output gradient dout and the
// forward's row statistics lse; perm as in launch_attn_f32.
hipError_t launch_attn_f32_bwd(const void* q, const void* k, const void* v, const void* o, const void* dout,
                               const float* lse, void* dq, void* dk, void* dv, const uint8_t* perm,
                               const Problem& pb, int distr, hipStream_t stream);
// The same for bf16 tensors on the matrix cores; `scratch` (256-byte aligned,
// attn_bf16_bwd_scratch_bytes) carries D_i and the channel-replicated Q between its kernels.
size_t attn_bf16_bwd_scratch_bytes(const Problem& pb, int distr);
hipError_t launch_attn_bf16_bwd(const void* q, const void* k, const void* v, const void* o, const void* dout,
                                const float* lse, void* dq, void* dk, void* dv, const uint8_t* perm, void* scratch,
                                const Problem& pb, int distr, hipStream_t stream);

}  // namespace da
