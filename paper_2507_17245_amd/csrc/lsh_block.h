// The LSH hash-and-group stage of one block of rows, as device code: the kernel of its own (lsh_group.hip, which says what bounds it)
// and the prologue of the float forward (attn_f32.hip) run it.
#pragma once
#include <type_traits>

#include "da_common.h"

namespace da {

// LDS of one workgroup
template <typename T, int D, int BR>
struct LshLds {
  static constexpr bool MATRIX = sizeof(T) == 2;
  static constexpr int CR = MATRIX || BR < 128 ? BR : 128;   // rows staged at a time
  static constexpr int RPAD = BR + 8;                        // bf16 pieces: 16 lanes read 16 rows of the table at once
  __attribute__((aligned(1024))) char rows[CR * D * sizeof(T)];
  __attribute__((aligned(16))) char table[MATRIX ? 2 * 16 * RPAD * 2 : BR * 16 * 4];
  __attribute__((aligned(16))) uint32_t code[D];
  __attribute__((aligned(16))) uint32_t hash[D];
  uint8_t perm[D];
};

// Position of a 16-byte chunk inside its staged bf16 row: the transposing reads address, per 32 lanes, the same
// two chunks of rows r..r+3 and r+8..r+11, which this spreads over all banks.
template <int D>
__device__ inline int lsh_chunk_swz(int row) {
  return D == 128 ? (((row & 3) | ((row >> 1) & 4)) << 1) : ((((row >> 1) & 1) | ((row >> 2) & 2)) << 1);
}

// Rows r0 .. of `block` (`rows` of them exist, the rest reads as zeros) into LDS.
template <typename T, int D, int CR, bool SWZ, int THREADS>
__device__ __forceinline__ void lsh_stage_rows(const T* block, int rows, int r0, char* dst) {
  typedef __attribute__((address_space(3))) void lds_void;
  constexpr int CH = D * (int)sizeof(T) / 16, N = (CR * CH + THREADS - 1) / THREADS;
  static_assert(CR * CH % 64 == 0, "whole loads per wave");
  if (((uintptr_t)block & 15) != 0) {   // (a tensor of the stand-alone entry, which asks for no alignment)
    for (int i = threadIdx.x; i < CR * D; i += THREADS) {
      const int row = i / D, at = i % D * (int)sizeof(T), chunk = at / 16;
      *(T*)(dst + row * (D * (int)sizeof(T)) + (SWZ ? chunk ^ lsh_chunk_swz<D>(row) : chunk) * 16 + at % 16) =
          r0 + row < rows ? block[(size_t)(r0 + row) * D + i % D] : (T)0.0f;
    }
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)block, 0, (unsigned)rows * D * sizeof(T), 0x00020000);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int blk = j * (THREADS / 64) + wave, slot = blk * 64 + lane;
    if (CR * CH % THREADS != 0 && blk * 64 >= CR * CH) break;   // (more waves than 1 KB blocks)
    const int row = slot / CH, pc = slot % CH;
    const int chunk = SWZ ? pc ^ lsh_chunk_swz<D>(row) : pc;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + blk * 1024), 16, row * (D * (int)sizeof(T)) + chunk * 16,
                                             r0 * (D * (int)sizeof(T)), 0, 0);
  }
}

// Sign codes of the bf16 block's channels, projections p0 .. p0 + 15, into lds.code. `rows`: a multiple of 32, the rest of
// the block is zeros.
template <int D, int BR, int THREADS>
__device__ __forceinline__ void lsh_codes_matrix(LshLds<bf16, D, BR>& lds, int rows, int p0, int n_planes) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  constexpr int RPAD = LshLds<bf16, D, BR>::RPAD, ROWB = D * 2;
  const bf16* rp1 = (const bf16*)lds.table;
  const bf16* rp2 = rp1 + 16 * RPAD;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int np = min(16, n_planes - p0);
  // v_mfma_f32_16x16x32_bf16: 16 channels x 16 projections per product, 32 rows of the block per step;
  // lane = (projection pl16 = lane % 16, row group kg = lane / 16) on the R side and (channel, row
  // group) on the Q side, whose operand comes out of the staged block by transposing reads. Register i of
  // the result belongs to channel 16*ct + 4*kg + i and projection pl16.
  const int pl16 = lane & 15, kg = lane >> 4;
  // The sign of a sum is taken from the matrix pipe only if the sum is further from zero than both
  // roundings can reach, each relative to sum |q| |R| <= (1 + 2^-8) sum |q| |r1|: the pipe's, at most
  // 2*BR products and BR/16 chained accumulators added in any order with any rounding direction
  // (2 * (2*BR + BR/16) * 2^-24), and the defining chain's, BR fused multiply-adds (BR * 2^-24).
  // The absolute term covers products flushed to zero.
  constexpr float kDoubt = 3.1e-7f * BR, kTiny = 1e-30f;
  for (int ct = wave; ct < D / 16; ct += THREADS / 64) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, bnd = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < BR / 32; ++ks) {
      if (32 * ks >= rows) break;
      const int row0 = 32 * ks + 8 * kg + (pl16 >> 2), row1 = row0 + 4;
      const int chunk = 2 * ct + ((pl16 & 3) >> 1), inch = 8 * (pl16 & 1);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds.rows + row0 * ROWB + ((chunk ^ lsh_chunk_swz<D>(row0)) << 4) + inch));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds.rows + row1 * ROWB + ((chunk ^ lsh_chunk_swz<D>(row1)) << 4) + inch));
      const s16x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      const s16x8 b1 = *(const s16x8*)&rp1[pl16 * RPAD + 32 * ks + 8 * kg];
      const s16x8 b2 = *(const s16x8*)&rp2[pl16 * RPAD + 32 * ks + 8 * kg];
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b1), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b2), acc, 0, 0, 0);
      bnd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a & (short)0x7fff),
                                                    __builtin_bit_cast(bf16x8, b1 & (short)0x7fff), bnd, 0, 0, 0);
    }
    bool positive[4], doubt[4], any_doubt = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      positive[i] = acc[i] > 0.0f;
      doubt[i] = pl16 < np && !(__builtin_fabsf(acc[i]) > kDoubt * bnd[i] + kTiny);
      any_doubt |= doubt[i];
    }
    if (__builtin_amdgcn_ballot_w64(any_doubt) != 0)
      settle_doubts(doubt, positive, rows, rp1, rp2, RPAD, [&](int row, int ch) {
        return *(const bf16*)(lds.rows + row * ROWB + (((2 * ct + (ch >> 3)) ^ lsh_chunk_swz<D>(row)) << 4) + (ch & 7) * 2);
      });
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // lanes 16*kg .. 16*kg + 15 of the ballot are the projections of channel 16*ct + 4*kg + i; projection 0
      // is the top bit of the n_planes-bit code
      const uint64_t signs = __builtin_amdgcn_ballot_w64(positive[i]);
      if (pl16 == 0) {
        const uint32_t bits = __builtin_bitreverse32((uint32_t)(signs >> (16 * kg)) & 0xffffu) >> (32 - np);
        const uint32_t before = p0 ? lds.code[16 * ct + 4 * kg + i] : 0;
        lds.code[16 * ct + 4 * kg + i] = before | bits << (n_planes - p0 - np);
      }
    }
  }
}

// `rows` rows of D channels at `block`; perm and hash (either may be null): the block's table entries. With KEEP the workgroup
// has the permutation in lds.perm, too. (Inlined by force: as a function that two kernels call, bf16 H32 N4096 d64 10.2 -> 23.3 us.)
template <typename T, int D, int BR, int THREADS, bool KEEP = false>
__device__ __forceinline__ void lsh_block(const T* __restrict__ block, int rows, int n_planes, int gray_mode, uint64_t seed,
                                 uint8_t* __restrict__ perm, uint32_t* __restrict__ hash, LshLds<T, D, BR>& lds) {
  using L = LshLds<T, D, BR>;
  constexpr int NPG = THREADS / D;            // threads per channel
  const int tid = threadIdx.x, c = tid % D, pg = tid / D;
  const int taken = (rows + 31) / 32 * 32;    // (a block of few rows costs what they cost)
  for (int p0 = 0; p0 < n_planes; p0 += 16) {
    if constexpr (L::MATRIX) {
      if (p0 == 0) lsh_stage_rows<T, D, BR, true, THREADS>(block, rows, 0, lds.rows);
      else __syncthreads();                   // the last table is no longer read
      bf16* rp1 = (bf16*)lds.table;
      bf16* rp2 = rp1 + 16 * L::RPAD;
      for (int i = tid; i < BR * 16; i += THREADS) {
        const int r = i % BR, pl = i / BR;
        if (r >= taken) continue;
        const float rv = p0 + pl < n_planes ? hyperplane_entry(seed, (uint32_t)(p0 + pl), (uint32_t)r) : 0.0f;
        const bf16 r1 = (bf16)rv;
        rp1[pl * L::RPAD + r] = r1;
        rp2[pl * L::RPAD + r] = (bf16)(rv - (float)r1);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      lsh_codes_matrix<D, BR, THREADS>(lds, taken, p0, n_planes);
    } else {
      // A thread takes PPT projections, pg*PPT .. pg*PPT + PPT - 1: as few as there are for everyone.
      float* R = (float*)lds.table;           // [row][16]
      auto project = [&](auto ppt_c) {
        constexpr int PPT = decltype(ppt_c)::value, PL = PPT * NPG;   // PL: projections of the table that are generated
        float acc[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j) acc[j] = 0.0f;
        for (int r0 = 0; r0 < rows; r0 += L::CR) {
          if (p0 + r0 > 0) __syncthreads();   // the staged rows are no longer read
          lsh_stage_rows<T, D, L::CR, false, THREADS>(block, rows, r0, lds.rows);
          if (r0 == 0) {
            for (int i = tid; i < min(rows, BR) * PL; i += THREADS) {
              const int p = p0 + (i & (PL - 1)), r = i / PL;
              R[PL == 16 ? i : r * 16 + (i & (PL - 1))] = p < n_planes ? hyperplane_entry(seed, (uint32_t)p, (uint32_t)r) : 0.0f;
            }
            if (p0 == 0 && tid < D) lds.code[tid] = 0;
          }
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          __syncthreads();
          const float* x = (const float*)lds.rows + c;
          const float* Rt = R + r0 * 16 + pg * PPT;
          const int n = min(L::CR, rows - r0);
#pragma unroll 8
          for (int r = 0; r < n; ++r) {
            const float xr = x[r * D];
#pragma unroll
            for (int j = 0; j < PPT; ++j) acc[j] = __builtin_fmaf(xr, Rt[r * 16 + j], acc[j]);
          }
        }
        // (n_planes and p0 are at hand; their difference is one register more, which at 64 rows and d = 128 left the loop above the rows of one step
        // in flight instead of eight: 4.8 -> 5.8 us)
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
          const int p = p0 + pg * PPT + j;
          if (p < n_planes && acc[j] > 0.0f) bits |= 1u << (n_planes - 1 - p);   // projection 0 = top bit
        }
        if (bits) atomicOr(&lds.code[c], bits);
      };
      // (four projections at a workgroup of four threads a channel: tiny calls, whose workgroups all wait for this; H1 N256 11.3 | 10.6 us)
      if (KEEP && NPG == 4 && n_planes - p0 <= 4) project(std::integral_constant<int, KEEP ? 1 : 16 / NPG>());
      else project(std::integral_constant<int, 16 / NPG>());
    }
  }
  __syncthreads();
  if (tid < D) {
    const uint32_t h = lsh_hash_of_code(lds.code[tid], gray_mode);
    lds.hash[tid] = h;
    lds.code[tid] = 0;   // from here on the channel's rank is counted in this word
    if (hash) hash[tid] = h;
  }
  __syncthreads();
  // Rank by counting = stable ascending sort; perm = inverse of the rank. Every thread counts a slice of
  // the other channels for its own (hashes read four at a time); the slices meet in an integer LDS add.
  constexpr int SL = D / NPG;
  const int first = pg * SL;
  const uint32_t mine = lds.hash[c];
  uint32_t cnt = 0;
#pragma unroll
  for (int o4 = 0; o4 < SL; o4 += 4) {
    const u32x4 h = *(const u32x4*)&lds.hash[first + o4];
#pragma unroll
    for (int j = 0; j < 4; ++j) cnt += (h[j] < mine || (h[j] == mine && first + o4 + j < c)) ? 1u : 0u;
  }
  if (cnt) atomicAdd(&lds.code[c], cnt);
  __syncthreads();
  if (!KEEP && !perm) return;
  if (tid < D) lds.perm[lds.code[tid]] = (uint8_t)tid;
  __syncthreads();
  if (perm && tid < D) perm[tid] = lds.perm[tid];
}

}  // namespace da
