// Tiled bf16 attention forward for gfx950 (CDNA4): exact attention (Sec. 2.1, tiled as in
// Sec. 2.2.2) and DistrAttention (Sec. 3.1 Eq. 2, Sec. 3.2 sampling and fusion, Sec. 3.3
// block-wise grouping) from one template.
//
// Work split. One workgroup owns one Q block of BR rows of one (batch, head); each of its
// BR/32 wavefronts owns 32 query rows for the whole inner loop over K/V tiles of BC rows
// (the paper's l and m: BR in {64, 128, 256}, BC in {32, 64, 128}). Launches that leave SIMDs
// without a wave, or with one, take twice the wavefronts per workgroup (KS = 2): each half of them has
// tile buffers of its own and walks half of the block's tiles, the two softmax states meet in LDS at the end.
//
// Matrix-core mapping (v_mfma_f32_32x32x16_bf16, fp32 accumulate). Both products are taken
// transposed so that one lane owns one query row's softmax state:
//   S^T[kv][q] = sum_c  Kx[kv][c] * Qx[q][c]      A = Kx tile rows from LDS, B = Qx in registers
//   O^T[ch][q] = sum_kv V[kv][ch] * P^T[kv][q]    A = V^T via LDS transpose reads, B = P^T in registers
// The accumulator layout of the first product (lane = q, registers = kv) is, after conversion
// to bf16, exactly the B-operand layout of the second, so P never leaves registers; the
// contraction index kv is enumerated in the accumulator's order on both operands.
//   exact:  Kx = K tile,  Qx = Q,    contraction over d channels
//   distr:  Kx = K_f tile (Sec. 3.2 fusion: sum of the group's K channels, built once per
//           (Q block, K tile) by all waves together: packed half adds in registers on pieces of
//           a transposed half-precision copy of K, result in LDS), Qx = Q_r (sampling: the
//           group's first channel in sorted order, gathered once per Q block), contraction over
//           n_groups = d / G*, on the f16 matrix path. The grouping itself (Sec. 3.2 LSH, sort,
//           groups) is either read from a table or computed by the workgroup in its prologue.
// Online softmax (reference max, row sum, rescaled accumulator) follows the block-wise scheme of
// Sec. 2.2.2 in the exp2 domain.
//
// Pipeline (one barrier per tile): K (exact) and V tiles reach LDS by direct global->LDS loads
// two tiles (K) / one tile (V) ahead, the K^T pieces of the fusion reach registers one tile
// ahead of their use; while the vector ALUs exponentiate tile i the matrix pipe computes the
// scores of tile i+1; P.V of tile i follows with its V operands read four ahead of their MFMAs.
// The reference of the online softmax moves only when a tile's row sum says it must (no row
// maximum per tile).
#pragma once
#include <type_traits>

#include "da_common.h"

namespace da {

namespace {

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef _Float16 f16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

// Largest finite half; sampled queries and fused keys of the distr path are clamped to it.
constexpr float kHalfMax = 65504.0f;
__device__ inline f16 to_half_sat(float x) { return (f16)__builtin_amdgcn_fmed3f(x, -kHalfMax, kHalfMax); }

__device__ inline f32x16 mfma_32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ inline f32x16 mfma_32x32x16(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Two transposing LDS reads (ds_read_b64_tr_b16): within each group of 16 lanes, lane i
// receives element (i % 4) of the 8-byte chunks addressed by lanes 4j + i/4, j = 0..3.
template <typename V8>
__device__ inline V8 lds_read_tr_pair(const void* p0, const void* p1) {
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p0);
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p1);
  s16x8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(V8, r);
}

// Swizzle of the 32-byte segments of a tile that is read with transposing accesses
// (ds_read_b64_tr_b16): the LDS serves 32 lanes of such a read per cycle, which address the rows
// r..r+3 (r a multiple of 4) at two adjacent 32-byte segments, 4 lanes x 8 bytes per row and
// segment. v_swizzle spreads those 4 rows x 2 segments over all 64 banks (no conflict cycles in
// the hardware counters): with 256-byte rows the row picks one of four segment pairs, with
// 128-byte rows two consecutive rows already sit in opposite bank halves and only rows of equal
// parity need separating.
template <int ROW_BYTES>
__device__ inline int v_swizzle(int row) {
  static_assert(ROW_BYTES == 256 || ROW_BYTES == 128, "row length");
  return ROW_BYTES == 256 ? ((row & 3) << 1) : (row & 2);
}
// The fused tile K_f^T (rows of 2*BC bytes, one per group) is read with the same transposing
// accesses and takes the same swizzle as a V tile with rows of that length; rows of 64 bytes
// (BC = 32) hold two segments, exchanged on every second pair of rows.
template <int BC>
__device__ inline int kf_swizzle(int row) {
  if constexpr (BC == 64) return v_swizzle<128>(row);
  else if constexpr (BC == 128) return v_swizzle<256>(row);
  else return (row >> 1) & 1;
}

// What the score product is taken of.
//   kExact       Q and K.
//   kFused       Q_r and K_f, on the f16 matrix path, contraction over the groups.
//   kReplicated  Q~ and K: Q~ is Q with every channel replaced by its group's sampled channel, so
//                S^ = Q_r K_f^T = Q~ K^T (a sum over groups of sums over members). The exact kernel's
//                loop with the grouping in the prologue: d / n_groups times the products, but no
//                transposed copy of K to make first and no fusion (rule: attn_bf16.hip).
enum ScoreMode { kExact, kFused, kReplicated };

// KRED: contraction length of the score product (a multiple of the MFMA step, 16). NG: number of
// channel groups; smaller than KRED only for n_groups 4 and 8, whose operands are zero-padded to 16
// (kFused; the other modes are built once for every n_groups, NG = KRED = D). KS: shares of a block's tiles.
template <int D, int BR, int BC, int KRED, int MODE, int NG = KRED, int KS = 1>
struct Cfg {
  static constexpr bool FUSED = MODE == kFused;
  static constexpr bool GROUPED = MODE != kExact;
  static constexpr int RW = BR / 32;              // wavefronts side by side over the block's rows
  static constexpr int NW = RW * KS;              // wavefronts per workgroup
  static constexpr int TH = RW * 64;              // threads that share a stream of tiles
  static constexpr int T = NW * 64;               // threads
  static constexpr int G = D / NG;                // channels per group
  static constexpr int CH = D / 8;                // 16-byte chunks per row
  static constexpr int MB = BC / 32;              // 32-key blocks of the score product per tile
  static constexpr int TT = BC / 16;              // 16-key steps of P.V per tile
  static constexpr int NBLK = BC * CH / 64;       // 1 KB blocks (one wave-level direct load each) per tile
  static constexpr int CPT = (NBLK + RW - 1) / RW;  // direct loads each wave issues per tile
  // LDS layouts.
  //  * V tiles, and K tiles of the exact path, arrive by direct global->LDS loads (each
  //    wave-level load drops 64 x 16 bytes contiguously), so rows are unpadded (D*2 bytes) and
  //    bank conflicts are avoided by swizzling where a 16-byte chunk sits inside its row:
  //      K (read with 16-byte accesses, 16 lanes = 16 rows at one logical chunk):
  //          chunk' = chunk ^ (row & 15)            (D = 128: 16 chunks per row)
  //          chunk' = chunk ^ ((row >> 1) & 7)      (D = 64: 8 chunks per row, two rows per 256 B)
  //      V (read with transposing 8-byte accesses; the LDS serves 32 lanes per cycle, which
  //      address 4 rows x 2 adjacent 32-byte segments and must cover all 256 bytes of banks):
  //          32-byte segment' = segment ^ 2*(row & 3)       (D = 128: 8 segments per row)
  //          32-byte segment' = segment ^ (row & 2)         (D = 64: 4 segments per row, rows of
  //                                                          opposite parity sit in opposite bank halves)
  //    The loading lane fetches the global chunk that belongs at its LDS position.
  //  * distr path: the keys arrive transposed and in half precision (K^T in global memory, one
  //    row of BC keys = 2*BC bytes per channel and tile, written once per forward by the key
  //    pre-pass). Only the fused tile K_f^T (one such row per group) lives in LDS: written by
  //    the waves, read back with transposing accesses, segments swizzled by kf_swizzle.
  static constexpr int ROWB = D * 2;              // bytes of an unpadded K / V row
  static constexpr int TILEB = BC * ROWB;         // bytes of an unpadded tile
  static constexpr int KTROWB = BC * 2;           // bytes of a K^T / K_f^T row (BC keys)
  static constexpr int PPR = BC / 8;              // 16-byte pieces (8 keys) per K^T / K_f^T row
  static constexpr int KX_BYTES = FUSED ? KRED * KTROWB : TILEB;   // one Kx buffer: K_f^T or K
  static constexpr int FUSE_OUT = (NG * PPR + TH - 1) / TH;   // 16-byte fused outputs per thread and tile
  static constexpr int KSTEPS = KRED / 16;        // MFMA steps of the score product
  // Register budget: two waves per SIMD, except the widest tile at d = 128, whose two score sets
  // (128 registers) leave room for one.
  static constexpr int WAVES_PER_SIMD = (BC == 128 && D == 128) ? 1 : 2;
};

// Lazy reference maximum. A row keeps its reference until one of its scores runs more than kTau
// (log2 units) ahead of it and the test finds it: numerator and denominator share the
// reference, so the result is the same ratio, and the accumulator rescale (one multiply per
// accumulator register) almost never runs. The test needs no row maximum: a lane's row sum over
// the BC/2 keys it owns in a tile exceeds (BC/2) * 2^kTau only if one of them exceeds 2^kTau (an
// overflowed or NaN sum fails the comparison too), and the sum is needed anyway. One that exceeds 2^kTau alone
// may stay below it: P is at most (BC/2) * 2^kTau. Over all BC keys the test would let twice that pass and the largest weight would be the
// exact P = 1 less often (exact H4 N1500 d64, queries of four times the scale: error against 64 bits 2.6 % larger, of the row statistics 27 %).
constexpr float kTau = 8.0f;

// Row sums of P, the B operands of P.V (lane = row lane % 32, either half of the wave its half of the keys). They are taken over the
// rounded P, the values P.V really uses: numerator and denominator then carry the same rounding, which cancels for rows dominated
// by few keys. On the matrix pipe: v_mfma_f32_16x16x32_bf16 takes lanes 16 g .. 16 g + 15 as rows 8 g .. of a 32 x 16 operand;
// the left operand has ones where the group is that of the result's lane and zeros elsewhere, so that every lane receives the sum of
// its own values. 16 cycles of the pipe for eight values a lane. (v_dot2c_f32_bf16 against (1, 1), one for two values, is no vector instruction like the others: it waits for the
// matrix pipe and holds it up, 13 cycles each between products. 8 exponentials with 3, 4, 6, 8 products beside them,
// cycles by dot products | by this one, two waves per SIMD: 177 | 136, 209 | 160, 256 | 214, 310 | 273.)
// An infinity or a NaN in a lane makes the sums of the lanes 16, 32 and 48 away NaN, too (zero times it): a tile with sums that are not finite takes
// them again by_lanes, with dot products. (Keeping the matrix pipe's sums of the other rows there, to the last bit, cost every call 1-2 %.)
struct RowSum {
  bf16x8 own;
  __device__ explicit RowSum(int lane) {
    const bf16 x = (bf16)(((lane >> 2 ^ lane >> 4) & 3) == 0 ? 1.0f : 0.0f);
#pragma unroll
    for (int j = 0; j < 8; ++j) own[j] = x;
  }
  template <int TT>
  __device__ float operator()(const bf16x8 (&pop)[TT]) const {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(own, pop[tt], acc, 0, 0, 0);
    return acc[0];
  }
  template <int TT>
  static __device__ float by_lanes(const bf16x8 (&pop)[TT]) {
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
    float rs0 = 0.0f, rs1 = 0.0f;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int j = 0; j < 8; j += 4) {
        rs0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pop[tt][j], pop[tt][j + 1]}, ones, rs0, false);
        rs1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pop[tt][j + 2], pop[tt][j + 3]}, ones, rs1, false);
      }
    return rs0 + rs1;
  }
};

// Sums of P on the matrix pipe (RowSum) where they take no registers that the wave has not got: fused kernels hold ten more
// than with dot products, which costs a wave per SIMD or spills, and at d = 128 (blocks of 128 rows, one long wave) what the clock falls by. us, dot products | this:
//   exact and Q~ K^T, d64 Br256 N3000 46.0 | 45.1, Q~ K^T 42.5 | 41.4, Br64 N200 on 30000 keys 43.0 | 42.6, Br128 45.4 | 44.8;
//   exact d64 Br128 in halves N300 on 16000 keys 33.6 | 32.8, N200 on 30000 40.6 | 40.2; Q~ K^T d64 Br128 H32 N1000 18.5 | 18.5, B2 H32 N530 on 4000 58.8 | 58.5;
//   d128 H16 N8192 causal 266 | 262, Br256 N3000 77.1 | 71.0; fused d64 N16384 490 | 502; d128 N32768 3182 | 3240, but Br256 N3000 88.6 | 82.5.
// One wave per SIMD waits for its sums itself: not at d = 64 with tiles of 128 keys and 64 rows (exact N2034 on 4337 keys 49.8 | 51.4), and by the launch (launch_ks)
// at d = 128 with 64 rows and in exact blocks of 128 at d = 64.
template <int D, int BR, int BC, int MODE, int NG, int KS>
constexpr bool kMatrixSum = MODE == kFused ? D == 128 && BR == 256 && BC == 64 && NG >= 16
                            : D == 64      ? BR != 64 || BC != 128
                                           : BC != 128;

template <int D, int BR, int BC, int KRED, int MODE, int NG, int KS, bool MATRIX_SUM>
__global__ __launch_bounds__(BR * 2 * KS, (Cfg<D, BR, BC, KRED, MODE, NG, KS>::WAVES_PER_SIMD)) void attn_bf16_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v,
    bf16* __restrict__ o, const uint8_t* __restrict__ perm, const f16* __restrict__ kt, int Npad,
    int H, int Hkv, int N, int Nk, int Tq, int causal, float scale_log2e, int total_units, int n_planes,
    int gray_mode, uint64_t lsh_seed, float* __restrict__ lse, const char* __restrict__ rtab,
    uint8_t* __restrict__ perm_w, int n_groups, int Br_log2, int table_in_o, int n_split, float* __restrict__ part_o, f32x2* __restrict__ part_stat) {
  using C = Cfg<D, BR, BC, KRED, MODE, NG, KS>;
  constexpr bool FUSED = C::FUSED, GROUPED = C::GROUPED;
  constexpr float kSumTrigger = (BC / 2) * 256.0f;   // BC/2 keys per lane and tile, each at most 2^kTau
  // A row whose first tile holds only scores of -infinity (masked keys; those of a share or half that the causal mask hides)
  // takes its first score above that as its reference: against 0, scores of -150 and less would be lost. The fused product has no such
  // scores (its operands are clamped), and undivided keys begin with one that every row sees.
  constexpr bool LATE_FIRST = KS > 1 || !FUSED;
  float trigger = kSumTrigger;                       // (LATE_FIRST: below zero until the row has met such a score)
  using kx8 = typename std::conditional<FUSED, f16x8, bf16x8>::type;
  // Kx and V tiles are double-buffered: while tile i multiplies, tile i+1 (V) / i+2 (K) lands.
  // Each buffer is a separate LDS object: the compiler can then tell that the operand reads of
  // one buffer do not depend on the direct loads still in flight into the other.
  __shared__ __attribute__((aligned(1024))) char kx_lds0[KS * C::KX_BYTES];
  __shared__ __attribute__((aligned(1024))) char kx_lds1[KS * C::KX_BYTES];
  __shared__ __attribute__((aligned(1024))) char v_lds0[KS * C::TILEB];
  __shared__ __attribute__((aligned(1024))) char v_lds1[KS * C::TILEB];
  // The block's permutation is only needed while the prologue builds the sampled-query operands
  // and the fusion offsets: it borrows the head of the second V buffer, which receives its
  // first tile in the first loop iteration (after the prologue's barriers).
  uint8_t* perm_lds = (uint8_t*)v_lds1;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = KS == 1 ? wave : wave % C::RW, half = KS == 1 ? 0 : wave / C::RW;   // which 32 rows, and which half of the block's tiles
  const int tid_h = tid - half * C::TH;
  const int lq = lane & 31;   // query row of this lane inside the wave's 32 rows
  const int hh = lane >> 5;   // which half of each 8-wide contraction chunk this lane feeds
  auto kx_buf = [&](int par) -> char* { return (par ? kx_lds1 : kx_lds0) + half * C::KX_BYTES; };
  auto v_buf = [&](int par) -> char* { return (par ? v_lds1 : v_lds0) + half * C::TILEB; };

  // Workgroup -> (batch*head, Q block). Consecutive workgroup ids go round-robin over the 8 XCDs.
  // n_split > 1: the unit's key tiles are dealt out to that many workgroups (below).
  int unit = n_split > 1 ? (int)blockIdx.x % total_units : (int)blockIdx.x;
  int bh, t;
  if (causal >= 2) {
    // Causal blocks differ up to Tq-fold in length. When (nearly) all of them are resident at
    // once, head after head would leave whole compute units with only long or only short
    // blocks: take them longest first over all heads, so that every round of the dispatcher
    // spreads one length class over the chip and the short blocks fill the slots that free up
    // last. With a head count that is a multiple of 8 a head still stays on one XCD.
    const int n_bh = total_units / Tq;
    t = unit / n_bh;
    t = Tq - 1 - (causal == 3 ? paired_tile(t, n_bh, Tq) : t);
    bh = unit % n_bh;
  } else {
    // Each XCD walks a contiguous range of units, so the Q blocks of one head run together
    // and share that XCD's L2 for K and V; the causal blocks of a head longest first.
    if ((total_units & 7) == 0) unit = (unit & 7) * (total_units >> 3) + (unit >> 3);
    bh = unit / Tq;
    t = unit % Tq;
    if (causal) t = Tq - 1 - t;
  }
  const int b = bh / H, h = bh % H;
  const int hk = h / (H / Hkv);
  const int r0 = t * BR;

  const bf16* qh = q + (size_t)bh * N * D;
  const bf16* kh = k + (size_t)(b * Hkv + hk) * Nk * D;
  const bf16* vh = v + (size_t)(b * Hkv + hk) * Nk * D;
  // N queries against Nk keys; under the causal mask the last query is aligned with the last
  // key: key n is visible to query i iff n <= i + shift.
  int shift = Nk - N;

  int n_end = causal ? min(Nk, r0 + BR + shift) : Nk;
  int n_tiles = (n_end + BC - 1) / BC;
  if (n_split > 1) {
    // This workgroup's share of the tiles: the head's keys from its first tile on become the keys
    // it knows. It leaves sums relative to its own reference for the combine kernel; a workgroup
    // without tiles leaves an empty share.
    const int part = (int)blockIdx.x / total_units;
    const int t0 = (int)((long long)n_tiles * part / n_split), t1 = (int)((long long)n_tiles * (part + 1) / n_split);
    part_stat += ((size_t)part * (total_units / Tq) + bh) * N;
    part_o += ((size_t)part * (total_units / Tq) + bh) * N * D;
    if (t0 == t1) {
      for (int i = r0 + tid; i < min(r0 + BR, N); i += C::T) part_stat[i] = f32x2{0.0f, 0.0f};
      return;
    }
    kh += (size_t)t0 * BC * D;
    vh += (size_t)t0 * BC * D;
    Nk -= t0 * BC;
    shift -= t0 * BC;
    n_tiles = t1 - t0;
  }
  // KS = 2: the first half of the tiles goes to one half of the waves, the second to the other; the two meet in LDS
  // at the end. A share without tiles walks one past the last key: zeros (range check), masked out.
  int tile0 = 0, n_most = n_tiles;
  if constexpr (KS == 2) {
    n_most = (n_tiles + 1) / 2;
    if (half) {
      tile0 = n_tiles > 1 ? n_most : (Nk + BC - 1) / BC;
      n_tiles = max(n_tiles - n_most, 1);
      kh += (size_t)tile0 * BC * D;
      vh += (size_t)tile0 * BC * D;
      Nk = max(Nk - tile0 * BC, 0);
      shift -= tile0 * BC;
    } else {
      n_tiles = n_most;
    }
  }

  const int qw0 = r0 + rw * 32;              // first query row of this wave
  const int q_abs = qw0 + lq;                  // this lane's query row
  const int q_ld = min(q_abs, N - 1);          // ragged block: load a valid row, never store it

  // grouped at d = 64: the Q block first lands in LDS by direct loads, all in flight at once
  // (16-byte chunks, rows past N zero-filled by the range check); the LSH stage and the sampling
  // then read its columns from there. Walking the columns in global memory instead costs the
  // workgroup one memory round trip per 16 rows and another for the sampled columns, which at
  // d = 64, where a block only has a few short tiles of work, is a large part of its lifetime.
  // (At d = 128 the stage is a percent of the block's time and the 32 KB are not spent.)
  constexpr bool QSTAGE = GROUPED && D == 64;
  __shared__ __attribute__((aligned(1024))) char q_stage[QSTAGE ? BR * C::ROWB : 16];
  // The 16-byte chunks of a staged row are exchanged by the row index (chunk ^ ((row >> 1) & 7);
  // two rows of 128 bytes share a line of banks): the sampling reads one column of 32 different
  // rows at once and the LSH stage's transposing reads four rows per 16 lanes, which would
  // otherwise fall into one or two banks; reading along a row is conflict-free either way.
  auto q_swz = [](int row) { return (row >> 1) & 7; };
  auto q_staged = [&](int row, int ch) -> bf16 {
    return *(const bf16*)(q_stage + row * C::ROWB + (((ch >> 3) ^ q_swz(row)) << 4) + (ch & 7) * 2);
  };
  // (a generic lambda, like the other direct loads below: the builtins exist for the device only,
  // and a template is not checked against the host's builtin set)
  auto stage_q_block = [&](auto n_c, char* dst) {
    typedef __attribute__((address_space(3))) void lds_void_q;
    const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)qh, 0, (unsigned)N * D * 2, 0x00020000);
#pragma unroll
    for (int j = 0; j < decltype(n_c)::value; ++j) {
      const int blk = j * C::NW + wave;
      const int slot = blk * 64 + lane;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(q_rsrc, (lds_void_q*)(dst + blk * 1024), 16,
                                               (slot / (D / 8)) * (D * 2) + ((slot % (D / 8)) ^ (((slot / (D / 8)) >> 1) & 7)) * 16,
                                               r0 * (D * 2), 0, 0);
    }
  };
  // The two pieces of the projection table (each a whole number of 1 KB blocks) from the table in
  // global memory into d1 and d2: block j of the 2 * PB blocks goes to wave j % NW.
  auto load_rtab = [&](auto n_c, char* d1, char* d2) {
    typedef __attribute__((address_space(3))) void lds_void_r;
    constexpr int PB = ((16 * (BR + 8) * 2 + 1023) / 1024);
    const __amdgpu_buffer_rsrc_t r_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)(rtab + 1024), 0, 2 * PB * 1024, 0x00020000);
#pragma unroll
    for (int j = 0; j < decltype(n_c)::value; ++j) {
      const int blk = j * C::NW + wave;
      if (blk < 2 * PB) {
        char* dst = blk < PB ? d1 + blk * 1024 : d2 + (blk - PB) * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_rsrc, (lds_void_r*)dst, 16, lane * 16, blk * 1024, 0, 0);
      }
    }
  };
  if constexpr (QSTAGE) {
    constexpr int QBLK = BR * C::ROWB / 1024;      // 1 KB blocks of the Q block
    static_assert(QBLK % C::NW == 0, "whole blocks per wave");
    stage_q_block(std::integral_constant<int, QBLK / C::NW>(), q_stage);
  }
  // Q blocks of 1 << log2_rows rows (kReplicated: not always the workgroup's), and the entries of the tables its rows are in: of one
  // block, or of two of 64 rows at d = 128. Constants where they can be: divided and looked up for every launch, the maps of a block that
  // no other shares its workgroup with took H32 N1400 d64 from 22.3 to 22.7 us (now 22.5), and fused kernels one more register.
  const int log2_rows = MODE == kReplicated ? Br_log2 : __builtin_ctz(BR);
  const int n_maps = MODE == kReplicated && D == 128 && BR == 128 ? max(BR >> log2_rows, 1) * D : D;
  if constexpr (GROUPED) {
    if (perm != nullptr) {
      // One row of the table for each of the workgroup's Q blocks (kReplicated: several, or a part of one). D is a power
      // of two: an out-of-range entry of a caller's table cannot index past a row. table_in_o: the row lies in o, where the workgroup's first
      // output row will.
      const int blocks = ((N - 1) >> log2_rows) + 1, first = r0 >> log2_rows;
      const uint8_t* rows = MODE == kReplicated && table_in_o ? (const uint8_t*)(o + ((size_t)bh * N + r0) * D) : perm + ((size_t)bh * blocks + first) * D;
      for (int i = tid; i < n_maps; i += C::T)
        perm_lds[i] = first + i / D < blocks ? rows[i] & (D - 1) : (uint8_t)(i % D);
    } else {
      // ---- LSH hash-and-group of this Q block inside the workgroup (Sec. 3.2, 3.3) -------------
      // The table equals the stand-alone LSH kernel's bit for bit: a projection's sign is that of
      // the float sum with one fused multiply-add per row, rows ascending, from +0. At d = 128 the
      // sums are taken exactly that way; at d = 64 the matrix pipe takes them first and the defining
      // sum is only redone where the pipe's result is too close to zero to decide (below). Here the
      // stage costs no launch and no table in HBM, and runs while the CU's other workgroups keep
      // the matrix pipes busy. Up to 16 projections: R[row][16] (d = 128) or its two bf16 pieces
      // (d = 64) borrow the V buffers, the codes and hashes the first Kx buffer; all are filled
      // only after the barriers below.
      constexpr int NPG = C::T / D;             // threads per channel
      constexpr int PPT = 16 / NPG;             // projections per thread: pg*PPT .. pg*PPT+PPT-1
      static_assert(C::T % D == 0, "whole threads per channel");
      // (small tiles: the borrowed buffers are too short and the stage gets arrays of its own)
      constexpr bool R_BORROWS = BR * 16 * 4 <= C::TILEB, CODE_BORROWS = 2 * D * 4 <= C::KX_BYTES;
      __shared__ float R_own[(R_BORROWS || QSTAGE) ? 1 : BR * 16];
      __shared__ uint32_t code_own[CODE_BORROWS ? 1 : 2 * D];
      float* R_lds = R_BORROWS ? (float*)v_lds0 : R_own;
      uint32_t* code_lds = CODE_BORROWS ? (uint32_t*)kx_lds0 : code_own;
      uint32_t* hash_lds = code_lds + D;
      // Staged block: the projections are first taken on the matrix pipe, from R split into two
      // bf16 pieces (an entry is an integer of 17 bits times 2^-16: r1 = R rounded to bf16 and
      // r2 = R - r1 hold it exactly, and r1 + r2 gives it back exactly in float), next to
      // sum |q| |r1|, which bounds how far that sum can be from the float sum that defines the
      // sign. Only sums inside the bound are taken again the defining way (below). The pieces,
      // [projection][row] with rows padded by 16 bytes (16 lanes read 16 rows at once), borrow
      // the two V buffers where they fit.
      // The pieces come from the table the key pre-pass left behind the K^T copy when its header
      // names this call's seed, projection count and block rows (direct loads into LDS, no vector
      // work); otherwise the workgroup generates them.
      constexpr int RPAD = BR + 8;
      constexpr int RP_BYTES = rtab_piece_bytes(BR);
      constexpr bool RP_BORROWS = RP_BYTES <= C::TILEB;
      __shared__ __attribute__((aligned(1024))) char rp_own[(QSTAGE && !RP_BORROWS) ? 2 : 1][(QSTAGE && !RP_BORROWS) ? RP_BYTES : 16];
      bf16* rp1 = RP_BORROWS ? (bf16*)v_lds0 : (bf16*)rp_own[0];
      bf16* rp2 = RP_BORROWS ? (bf16*)v_lds1 : (bf16*)rp_own[(QSTAGE && !RP_BORROWS) ? 1 : 0];
      if constexpr (QSTAGE) {
        bool have_table = false;
        if (rtab != nullptr) {
          const RtabHeader hd = *(const RtabHeader*)rtab;
          have_table = hd.seed == lsh_seed && hd.n_planes == n_planes && hd.Br == BR;
        }
        if (have_table) {
          load_rtab(std::integral_constant<int, (2 * (RP_BYTES / 1024) + C::NW - 1) / C::NW>(), (char*)rp1, (char*)rp2);
        } else {
          for (int i = tid; i < BR * 16; i += C::T) {
            const int r = i % BR, pl = i / BR;
            const float rv = pl < n_planes ? hyperplane_entry(lsh_seed, (uint32_t)pl, (uint32_t)r) : 0.0f;
            const bf16 r1 = (bf16)rv;
            rp1[pl * RPAD + r] = r1;
            rp2[pl * RPAD + r] = (bf16)(rv - (float)r1);
          }
        }
      } else {
        // (H16 N120 Br128 took 15.3 us where the code in front had put this loop, 14.6 on a 64-byte instruction line)
        asm volatile(".p2align 6");
        for (int i = tid; i < BR * 16; i += C::T)
          R_lds[i] = (i & 15) < n_planes ? hyperplane_entry(lsh_seed, (uint32_t)(i & 15), (uint32_t)(i >> 4)) : 0.0f;
      }
      if (tid < D) code_lds[tid] = 0;
      if constexpr (QSTAGE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the Q block has landed
      __syncthreads();
      const int c = tid % D, pg = tid / D;
      const int rows = min(BR, N - r0);
      const bf16* qcol = qh + (size_t)r0 * D + c;
      if constexpr (QSTAGE) {
        // v_mfma_f32_16x16x32_bf16: 16 channels x 16 projections per product, 32 rows of the block
        // per step; lane = (projection pl16 = lane % 16, row group kg = lane / 16) on the R side
        // and (channel, row group) on the Q side, whose operand comes out of the staged block by
        // transposing reads (rows past N are zeros there). Register i of the result belongs to
        // channel 16*ct + 4*kg + i and projection pl16.
        const int pl16 = lane & 15, kg = lane >> 4;
        // The sign of a sum is taken from the matrix pipe only if the sum is further from zero
        // than both roundings can reach, each relative to sum |q| |R| <= (1 + 2^-8) sum |q| |r1|:
        // the pipe's, at most 2*BR products and BR/16 chained accumulators added in any order with
        // any rounding direction (2 * (2*BR + BR/16) * 2^-24), and the defining float chain's,
        // BR fused multiply-adds (BR * 2^-24). The absolute term covers products flushed to zero.
        constexpr float kDoubt = 3.1e-7f * BR, kTiny = 1e-30f;
        for (int ct = wave; ct < D / 16; ct += C::NW) {
          f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, bnd = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int ks = 0; ks < BR / 32; ++ks) {
            const int row0 = 32 * ks + 8 * kg + (pl16 >> 2), row1 = row0 + 4;
            const int chunk = 2 * ct + ((pl16 & 3) >> 1), inch = 8 * (pl16 & 1);
            const s16x8 a = lds_read_tr_pair<s16x8>(q_stage + row0 * C::ROWB + ((chunk ^ q_swz(row0)) << 4) + inch,
                                                    q_stage + row1 * C::ROWB + ((chunk ^ q_swz(row1)) << 4) + inch);
            const int roff = 32 * ks + 8 * kg;
            const s16x8 b1 = *(const s16x8*)&rp1[pl16 * RPAD + roff];
            const s16x8 b2 = *(const s16x8*)&rp2[pl16 * RPAD + roff];
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b1), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b2), acc, 0, 0, 0);
            bnd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a & (short)0x7fff),
                                                          __builtin_bit_cast(bf16x8, b1 & (short)0x7fff), bnd, 0, 0, 0);
          }
          bool positive[4], doubt[4], any_doubt = false;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            positive[i] = acc[i] > 0.0f;
            doubt[i] = pl16 < n_planes && !(__builtin_fabsf(acc[i]) > kDoubt * bnd[i] + kTiny);
            any_doubt |= doubt[i];
          }
          if (__builtin_amdgcn_ballot_w64(any_doubt) != 0)
            settle_doubts(doubt, positive, BR, rp1, rp2, RPAD, [&](int row, int ch) { return q_staged(row, 16 * ct + ch); });
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // lanes 16*kg .. 16*kg + 15 of the ballot are projections 0..15 of channel 16*ct + 4*kg + i;
            // projection 0 is the top bit of the n_planes-bit code
            const uint64_t signs = __builtin_amdgcn_ballot_w64(positive[i]);
            if (pl16 == 0)
              code_lds[16 * ct + 4 * kg + i] = __builtin_bitreverse32((uint32_t)(signs >> (16 * kg)) & 0xffffu) >> (32 - n_planes);
          }
        }
      } else {
        // (not staged: 16 column loads in flight per thread, because with two workgroups per CU
        // nothing else hides their latency here)
        float acc[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j) acc[j] = 0.0f;
#pragma unroll 16
        for (int r = 0; r < rows; ++r) {
          const float x = (float)qcol[(size_t)r * D];
#pragma unroll
          for (int j = 0; j < PPT; ++j) acc[j] = __builtin_fmaf(x, R_lds[r * 16 + pg * PPT + j], acc[j]);
        }
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
          const int pl = pg * PPT + j;
          if (pl < n_planes && acc[j] > 0.0f) bits |= 1u << (n_planes - 1 - pl);   // projection 0 = top bit
        }
        if (NPG == 1) code_lds[c] = bits;
        else if (bits) atomicOr(&code_lds[c], bits);
      }
      __syncthreads();
      if (tid < D) {
        // (at most 16 bits: hash and channel make one key)
        hash_lds[tid] = lsh_hash_of_code(code_lds[tid], gray_mode) << 7 | tid;
        code_lds[tid] = 0;   // from here on the channel's rank is counted in this word
      }
      __syncthreads();
      {
        // Rank by counting = stable ascending sort; perm = inverse of the rank. Every thread
        // counts a slice of the other channels for its own (NPG threads per channel, the hashes
        // read four at a time), the slices meet in an integer LDS add.
        constexpr int SL = D / NPG;
        static_assert(SL % 4 == 0, "whole 16-byte reads per slice");
        uint32_t* rank_lds = code_lds;
        const int first = pg * SL;
        const uint32_t mine = hash_lds[c];
        uint32_t cnt = 0;
#pragma unroll
        for (int o4 = 0; o4 < SL; o4 += 4) {
          const u32x4 h = *(const u32x4*)&hash_lds[first + o4];
#pragma unroll
          for (int j = 0; j < 4; ++j) cnt += h[j] < mine ? 1u : 0u;
        }
        if (NPG == 1) rank_lds[c] = cnt;
        else if (cnt) atomicAdd(&rank_lds[c], cnt);
        __syncthreads();
        if (tid < D) perm_lds[rank_lds[tid]] = (uint8_t)tid;
      }
    }
    if constexpr (QSTAGE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // the table of the workgroup's own LSH stage, for a caller that wants it (e.g. to hand it to
    // the backward pass)
    if (perm == nullptr && perm_w != nullptr)
      for (int i = tid; i < D; i += C::T) perm_w[((size_t)bh * Tq + t) * D + i] = perm_lds[i];
    if constexpr (NG < KRED) {
      // Rows NG..KRED-1 of K_f^T pad the contraction: zeroed once (after the LSH stage, which may
      // have borrowed them), the fusion never writes them; visible to every wave after the
      // barrier that ends the prologue.
      const f16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      for (int i = NG * C::KTROWB / 16 + tid_h; i < C::KX_BYTES / 16; i += C::TH) {
        ((f16x8*)kx_buf(0))[i] = zero;
        ((f16x8*)kx_buf(1))[i] = zero;
      }
    }
  }

  // ---- Q operands, held for the whole inner loop ------------------------------------------
  // distr: the reduced product runs on the f16 matrix path. A bf16 value converts to half
  // exactly (8 vs 11 significand bits) inside half's exponent range, and the fused keys, rounded
  // to half from the sum of such values, keep 3 more bits than bf16 would: with bf16 K_f the logit error
  // on inputs with heavy-tailed channel scales exceeds what the output tolerance allows.
  // distr: Q_r carries the factor softmax_scale * log2(e), rounded once more to half (11 bits:
  // the rounding is 8 times finer than the bf16 grid the inputs come from). The score
  // accumulators then hold the exponent of 2 directly. The exact path keeps Q as it is: scaling
  // and re-rounding to bf16 would cost accuracy on rows with close top scores, so there the
  // factor is applied to the float scores, one fused multiply-add per score.
  kx8 qop[C::KSTEPS];
  if constexpr (MODE == kReplicated) {
    // Q~: the sampled channel of every channel's group, by way of a map in LDS
    const int group = D / n_groups;
    uint8_t* from_lds = perm_lds + n_maps;
    const uint8_t* from = D == 128 && BR == 128 ? from_lds + (rw * 32 >> log2_rows) * D : from_lds;   // the map of this wave's Q block
    if constexpr (QSTAGE) {
      if (tid < D) from_lds[perm_lds[tid]] = perm_lds[tid / group * group];
      __syncthreads();
#pragma unroll
      for (int s = 0; s < C::KSTEPS; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) qop[s][j] = q_staged(rw * 32 + lq, from[16 * s + 8 * hh + j] & (D - 1));
    } else {
      // The wave's rows pass through its part of the K buffers, RPR at a time (16-byte chunks exchanged by the row; its
      // LDS accesses take effect in its order): gathered from global memory, two bytes per load and lane, they cost a
      // launch of few blocks several microseconds (H8 N852 causal Br256 45 -> 35 us, H16 N1024 Br128 32 -> 27). The map holds byte offsets; chunk ^ x is offset ^ 16 x.
      constexpr int PART = KS * C::KX_BYTES / (C::NW / 2), RPR = PART / C::ROWB < 32 ? PART / C::ROWB : 32;
      static_assert(RPR >= 4 && 32 % RPR == 0 && D == 128, "whole loads per round");
      u32x4 x[8];                          // load j: rows 4*j .. 4*j + 3
#pragma unroll
      for (int j = 0; j < 8; ++j)
        x[j] = *(const u32x4*)(qh + (size_t)min(qw0 + 4 * j + (lane >> 4), N - 1) * D + (lane & 15) * 8);
      for (int i = tid; i < n_maps; i += C::T) from_lds[i / D * D + perm_lds[i]] = (uint8_t)(2 * perm_lds[i / group * group]);
      __syncthreads();
      char* mine = (wave & 1 ? kx_lds1 : kx_lds0) + (wave >> 1) * (RPR * C::ROWB);
      const int row = lq % RPR;
      const uint32_t flip = (row & 15) * 0x10101010u;
#pragma unroll
      for (int r = 0; r < 32 / RPR; ++r) {
#pragma unroll
        for (int j = 0; j < RPR / 4; ++j) {
          const int dst = 4 * j + (lane >> 4);
          *(u32x4*)(mine + dst * C::ROWB + (((lane & 15) ^ (dst & 15)) << 4)) = x[r * (RPR / 4) + j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < C::KSTEPS; ++s) {
          const u32x2 f = *(const u32x2*)&from[16 * s + 8 * hh];
          const uint32_t at[2] = {(f[0] & 0xfefefefeu) ^ flip, (f[1] & 0xfefefefeu) ^ flip};
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const bf16 y = *(const bf16*)(mine + row * C::ROWB + ((at[j >> 2] >> (8 * (j & 3))) & 255));
            qop[s][j] = RPR == 32 || lq / RPR == r ? y : qop[s][j];
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      __syncthreads();                     // K tiles may land
    }
  } else if constexpr (FUSED) {
    // (staged block: a row past N reads as zeros and is never stored)
    const bf16* qrow = qh + (size_t)q_ld * D;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (NG == KRED || 16 * s + 8 * hh + j < NG)
          qop[s][j] = to_half_sat((QSTAGE ? (float)q_staged(rw * 32 + lq, perm_lds[(16 * s + 8 * hh + j) * C::G])
                                          : (float)qrow[perm_lds[(16 * s + 8 * hh + j) * C::G]]) * scale_log2e);
        else
          qop[s][j] = (f16)0.0f;   // padding of the contraction: no group there
    }
  } else {
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s)
      qop[s] = *(const bf16x8*)(qh + (size_t)q_ld * D + 16 * s + 8 * hh);
  }
  // The Q operands must have landed before the loop starts: otherwise the compiler's wait-count
  // bookkeeping carries "Q loads pending" into the loop and the MFMAs also wait for the K/V
  // prefetch of later tiles.
#pragma unroll
  for (int s = 0; s < C::KSTEPS; ++s) asm volatile("" : "+v"(qop[s]));

  // ---- fusion bookkeeping, fixed for the Q block ------------------------------------------------
  // Fused output u of this thread is the 16-byte piece (8 keys) number idx % 8 of group
  // idx / PPR, idx = tid_h + u*TH: it sums the same piece of the group's G channel rows of K^T
  // (f_src: byte offset of the piece inside the head's K^T, tile 0) and lands in row idx / 8 of
  // K_f^T at the swizzled position (f_dst).
  int f_src[FUSED ? C::FUSE_OUT : 1][FUSED ? C::G : 1];
  int f_dst[FUSED ? C::FUSE_OUT : 1];
  if constexpr (FUSED) {
#pragma unroll
    for (int u = 0; u < C::FUSE_OUT; ++u) {
      const int idx = min(tid_h + u * C::TH, NG * C::PPR - 1);
      const int j = idx / C::PPR, c8 = idx % C::PPR;
#pragma unroll
      for (int g = 0; g < C::G; ++g)
        f_src[u][g] = perm_lds[j * C::G + g] * Npad * 2 + tile0 * C::KTROWB + c8 * 16;
      f_dst[u] = j * C::KTROWB + ((((c8 >> 1) ^ kf_swizzle<BC>(j)) << 1) | (c8 & 1)) * 16;
    }
  }

  // tiles [0, n_full) need no masking for any row of the block
  const int n_full = min(causal ? max(0, min(r0 + shift, Nk)) / BC : Nk / BC, n_tiles);

  // ---- tile loads: global -> LDS ---------------------------------------------------------------
  // K and V rows are fetched through buffer descriptors: the per-lane byte offset inside a
  // tile is fixed, the tile advances through the scalar offset, and rows past the end of the
  // head read as zero (hardware range check), so a tile costs no address arithmetic.
  const unsigned head_bytes = (unsigned)Nk * D * 2;
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)kh, 0, head_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)vh, 0, head_bytes, 0x00020000);

  // Direct global->LDS tile loads. Wave-level load j of this wave fills the 1 KB block
  // j*RW + rw of the tile; lane i owns the 16 bytes at offset 16*i of that block, i.e. LDS
  // row (slot / CH), chunk position (slot % CH) with slot = 64*block + i, and fetches the global
  // chunk the swizzle assigns to that position.
  int dma_k[FUSED ? 1 : C::CPT], dma_v[C::CPT];
#pragma unroll
  for (int j = 0; j < C::CPT; ++j) {
    const int slot = (j * C::RW + rw) * 64 + lane;
    const int row = slot / C::CH, pc = slot % C::CH;
    if constexpr (!FUSED) dma_k[j] = row * C::ROWB + (pc ^ (D == 128 ? (row & 15) : ((row >> 1) & 7))) * 16;
    const int lseg = (pc >> 1) ^ v_swizzle<C::ROWB>(row);
    dma_v[j] = row * C::ROWB + (lseg * 2 + (pc & 1)) * 16;
  }
  typedef __attribute__((address_space(3))) void lds_void;
  auto dma_blocks = [&](auto n_c, __amdgpu_buffer_rsrc_t rsrc, int soff, const int* voff, char* dst) {
#pragma unroll
    for (int j = 0; j < decltype(n_c)::value; ++j)
      if (C::NBLK % C::RW == 0 || j * C::RW + rw < C::NBLK)   // (more waves than 1 KB blocks: the rest sit out)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + (j * C::RW + rw) * 1024), 16,
                                                 voff[j], soff, 0, 0);
  };
  auto dma_tile = [&](__amdgpu_buffer_rsrc_t rsrc, int tile, const int* voff, char* dst) {
    dma_blocks(std::integral_constant<int, C::CPT>(), rsrc, tile * C::TILEB, voff, dst);
  };
  auto dma_wait = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

  // distr: K^T of this kv head, [D channel rows][Npad keys] half.
  const __amdgpu_buffer_rsrc_t kt_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(FUSED ? kt + (size_t)(b * Hkv + hk) * D * Npad : nullptr), 0, (unsigned)D * Npad * 2, 0x00020000);
  // ---- fusion (Sec. 3.2): K_f^T[j][n] = sum over the group's channels c of K^T[c][n], eight keys
  // at a time with packed half adds (for G* = 2 the sum of two bf16-valued halves is rounded to
  // half once; larger groups add one channel after the other). Every thread loads the 16-byte
  // pieces it sums straight from K^T in global memory (8 lanes cover one 128-byte channel row)
  // one tile iteration before it adds them, so the LDS only sees K_f^T (8-16 KB per tile): with
  // the raw tile staged in LDS and summed from there (direct load, 16 KB read, K_f^T written)
  // the kernel was bound by LDS traffic and 2-12 % slower.
    typedef f16x8 Pieces[FUSED ? C::FUSE_OUT : 1][FUSED ? C::G : 1];
  Pieces piece;   // the set the main loop carries from one iteration to the next
  auto load_pieces = [&](int tile, Pieces& pc) {
    if constexpr (FUSED) {
#pragma unroll
      for (int u = 0; u < C::FUSE_OUT; ++u)
#pragma unroll
        for (int g = 0; g < C::G; ++g)
          pc[u][g] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(kt_rsrc, f_src[u][g], tile * C::KTROWB, 0));
    }
  };
  auto fuse_pieces = [&](int buf, const Pieces& pc) {   // loaded pieces -> K_f^T in kx_buf(buf)
    if constexpr (FUSED) {
      char* dst = kx_buf(buf);
#pragma unroll
      for (int u = 0; u < C::FUSE_OUT; ++u) {
        f16x8 acc = pc[u][0];
#pragma unroll
        for (int g = 1; g < C::G; ++g) acc += pc[u][g];
        if (NG * C::PPR % C::TH == 0 || tid_h + u * C::TH < NG * C::PPR) *(f16x8*)(dst + f_dst[u]) = acc;
      }
    }
  };

  // ---- accumulators and softmax state ---------------------------------------------------------
  f32x16 oacc[D / 32];
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[mb][i] = 0.0f;
  // Softmax state of this lane's query row, in the exp2 domain: the negated reference maximum
  // and the row sum relative to it. distr: the negated reference also sits in all 16 registers
  // of neg_ref, which the first MFMA of every score chain takes as its addend, so the
  // accumulators come out as (scaled score - m_ref) and go straight into exp2.
  constexpr bool PRESCALED = FUSED;
  float nref = 0.0f;
  f32x16 neg_ref;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_ref[i] = 0.0f;
  float l_run = 0.0f;        // over this lane's half of the keys

  // LDS byte offsets of this lane's operands inside a buffer.
  // Score product, A operand (exact): row lq (+32 per key block), logical chunk 2*s + hh.
  int ka_off[FUSED ? 2 * C::MB : C::KSTEPS];
  if constexpr (FUSED) {
    // K_f^T is read like V: lane addresses group row 8*hh + 4*half + (lane%16)/4 (+16*s), 32-byte
    // segment 2*mb + (lane/16)%2 (keys 32*mb + 16*((lane/16)%2) ..), 8-byte piece lane%4.
    const int r4 = (lane & 15) >> 2;
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
        ka_off[mb * 2 + hf] = (8 * hh + 4 * hf + r4) * C::KTROWB +
                              ((2 * mb + ((lane >> 4) & 1)) ^ kf_swizzle<BC>(4 * hf + r4)) * 32 + 8 * (lane & 3);
  } else {
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s)
      ka_off[s] = lq * C::ROWB + ((2 * s + hh) ^ (D == 128 ? (lq & 15) : ((lq >> 1) & 7))) * 16;
  }
  // P.V, A operand via transposing reads: lane addresses row 4*hh + (lane%16)/4 (+8, +16*tt),
  // logical 32-byte segment 2*mb + (lane/16)%2, 8-byte piece lane%4 of it.
  int va_off[D / 32];
  {
    const int row_l = 4 * hh + ((lane & 15) >> 2);
    const int swz = v_swizzle<C::ROWB>(row_l);
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
      va_off[mb] = row_l * C::ROWB + ((2 * mb + ((lane >> 4) & 1)) ^ swz) * 32 + 8 * (lane & 3);
  }

  // S^T = Kx . Qx^T for the Kx tile in buffer `buf`: register i of block mb holds key
  // 32*mb + 8*(i/4) + 4*hh + i%4 of the tile.
  auto qk = [&](int buf, f32x16 (&sacc)[C::MB]) {
    const char* base = kx_buf(buf);
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) {
#pragma unroll
      for (int s = 0; s < C::KSTEPS; ++s) {
        kx8 a;
        if constexpr (FUSED)
          a = lds_read_tr_pair<kx8>(base + ka_off[mb * 2] + s * 16 * C::KTROWB,
                                    base + ka_off[mb * 2 + 1] + s * 16 * C::KTROWB);
        else
          a = *(const kx8*)(base + ka_off[s] + mb * 32 * C::ROWB);
        if (s == 0) {
          if constexpr (PRESCALED) sacc[mb] = neg_ref;
          else
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[mb][i] = 0.0f;
        }
        sacc[mb] = mfma_32x32x16(a, qop[s], sacc[mb]);
      }
    }
  };

  // Causal / ragged-tail mask of the scores of tile `tile`.
  auto apply_mask = [&](int tile, f32x16 (&sc)[C::MB]) {
    const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;  // last visible key of this row
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int kv = tile * BC + 32 * mb + 8 * (i >> 2) + 4 * hh + (i & 3);
        if (kv > lim) sc[mb][i] = -INFINITY;
      }
  };
  // Row maximum of a tile's scores (relative to the current reference), the same in both lanes
  // of a row.
  auto tile_max = [&](const f32x16 (&sc)[C::MB]) -> float {
    float mt = sc[0][0];
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mt = fmaxf(mt, sc[mb][i]);
    mt = half_swap_max(mt);
    return PRESCALED ? mt : __builtin_fmaf(mt, scale_log2e, nref);
  };
  // P = exp2(scores) rounded to bf16, as the B operands of P.V; with sum_c returns this lane's row sum, by dot products.
  auto exp_tile = [&](const f32x16 (&sc)[C::MB], bf16x8 (&pop)[C::TT], auto sum_c) -> float {
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
    float rs0 = 0.0f, rs1 = 0.0f;
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        float x0 = sc[mb][i], x1 = sc[mb][i + 1];
        if constexpr (!PRESCALED) {
          x0 = __builtin_fmaf(x0, scale_log2e, nref);
          x1 = __builtin_fmaf(x1, scale_log2e, nref);
        }
        const bf16x2 pr = {(bf16)__builtin_amdgcn_exp2f(x0), (bf16)__builtin_amdgcn_exp2f(x1)};
        pop[mb * 2 + (i >> 3)][i & 7] = pr[0];
        pop[mb * 2 + (i >> 3)][(i & 7) + 1] = pr[1];
        if constexpr (decltype(sum_c)::value) {
          if (i & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs1, false);
          else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs0, false);
        }
      }
    return rs0 + rs1;
  };
  const RowSum row_sum(lane);
  const std::integral_constant<bool, !MATRIX_SUM> sum_here;
  // The reference of this lane's row moves up by `delta`: everything that is relative to it
  // follows (row sum, output accumulator, the scores already computed against the old one).
  auto shift_reference = [&](float delta, auto rescale_c, f32x16 (&sc)[C::MB], auto next_c, f32x16 (&sn)[C::MB]) {
    nref -= delta;
    if constexpr (PRESCALED) {
#pragma unroll
      for (int i = 0; i < 16; ++i) neg_ref[i] -= delta;
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sc[mb][i] -= delta;
          if constexpr (decltype(next_c)::value) sn[mb][i] -= delta;
        }
    }
    if constexpr (decltype(rescale_c)::value) {
      const float alpha = __builtin_amdgcn_exp2f(LATE_FIRST ? fminf(-delta, 0.0f) : -delta);   // (a first reference has no sums)
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mb][i] *= alpha;
    }
  };

  // What tile `it` brings in. The buffers these loads fill were last read in the previous iteration, which every wave
  // has left (barrier): K(it+2) replaces K(it), V(it+1) replaces V(it-1).
  auto feed = [&](int it, int par) {
    // distr: the pieces of K^T(it+2), loaded during the previous iteration, are summed now
    // into the buffer K_f^T(it) has left, and the loads of K^T(it+3) take their registers.
    // Nothing in this iteration depends on the fusion: it runs beside the MFMAs.
    if constexpr (FUSED) {
      fuse_pieces(par, piece);       // K^T(it+2), loaded during the previous iteration
      load_pieces(it + 3, piece);
    }
    if constexpr (!FUSED) dma_tile(k_rsrc, it + 2, dma_k, kx_buf(par));
    dma_tile(v_rsrc, it + 1, dma_v, v_buf(par ^ 1));
  };
  // One tile `it`, whose scores `sc` are masked and relative to the row's reference:
  //   scores of tile it+1 into `sn` (matrix pipe)  ||  exp2, bf16 P, row sum of `sc` (vector ALUs)
  //   the rare reference move, then O^T += V^T . P^T for tile it (matrix pipe), the mask of
  //   tile it+1 where it needs one, one barrier.
  auto body = [&](auto mask_next_c, auto next_c, int it, int par, f32x16 (&sc)[C::MB], f32x16 (&sn)[C::MB]) {
    constexpr bool HAS_NEXT = decltype(next_c)::value;
    if constexpr (HAS_NEXT) {
      feed(it, par);
      qk(par ^ 1, sn);
    }
    bf16x8 pop[C::TT];
    float rs = exp_tile(sc, pop, sum_here);
    if constexpr (MATRIX_SUM) rs = row_sum(pop);
    if (__builtin_amdgcn_ballot_w64(!(rs <= (LATE_FIRST ? trigger : kSumTrigger))) != 0) {
      // Some row of this wave met a score more than kTau above its reference, or its first one above -infinity: such rows take the
      // tile's maximum as their new reference and the tile's P is computed again.
      const float mt = tile_max(sc);
      const bool first = LATE_FIRST && trigger < 0.0f && mt > -INFINITY;
      if (first) trigger = kSumTrigger;
      shift_reference(mt > kTau || first ? mt : 0.0f, std::true_type(), sc, next_c, sn);
      rs = exp_tile(sc, pop, sum_here);
      if constexpr (MATRIX_SUM) rs = RowSum::by_lanes(pop);
    }
    l_run += rs;
    // ---- O^T += V^T . P^T: step tt covers keys 16*tt + {8*(j/4) + 4*hh + j%4} of the tile,
    // i.e. V rows 16*tt + 4*hh + 0..3 and 16*tt + 8 + 4*hh + 0..3.
    const char* vb = v_buf(par);
    // The V operands are read PF steps (four operands) ahead of the MFMA that takes them, and the
    // scheduler is told to keep that order: left alone it issues an operand's reads right in
    // front of its MFMA, which then waits out the LDS latency 4 * TT times per tile.
    constexpr int NMB = D / 32;
    constexpr int PF = (4 / NMB < C::TT) ? 4 / NMB : C::TT - 1;
    auto v_operand = [&](int tt, int mb) {
      const char* p0 = vb + va_off[mb] + 16 * tt * C::ROWB;
      return lds_read_tr_pair<bf16x8>(p0, p0 + 8 * C::ROWB);
    };
    bf16x8 va[PF + 1][NMB];
#pragma unroll
    for (int t0 = 0; t0 < PF; ++t0)
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) va[t0][mb] = v_operand(t0, mb);
#pragma unroll
    for (int tt = 0; tt < C::TT; ++tt) {
      if (tt + PF < C::TT) {
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) va[(tt + PF) % (PF + 1)][mb] = v_operand(tt + PF, mb);
      }
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
        oacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[tt % (PF + 1)][mb], pop[tt], oacc[mb], 0, 0, 0);
    }
    // instruction order: the reads of the first PF steps, then every MFMA followed by the two
    // reads of one operand PF steps ahead (0x100 = LDS reads, 0x008 = MFMA)
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * NMB * PF, 0);
#pragma unroll
    for (int i = 0; i < (C::TT - PF) * NMB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, PF * NMB, 0);
    if constexpr (HAS_NEXT) {
      if constexpr (decltype(mask_next_c)::value) apply_mask(it + 1, sn);
      dma_wait();              // this wave's direct loads have landed
    }
    __syncthreads();
  };

  // ---- prologue: tiles 0 (K, V) and 1 (K) into LDS, scores of tile 0 ---------------------------
  dma_tile(v_rsrc, 0, dma_v, v_buf(0));
  if constexpr (FUSED) {
    Pieces first;        // tiles 0 and 1 travel together (registers are plentiful before the loop)
    load_pieces(0, first);
    load_pieces(1, piece);
    fuse_pieces(0, first);
    fuse_pieces(1, piece);
    load_pieces(2, piece);
    dma_wait();          // V(0) has landed (and, with it, the pieces of tile 2)
    __syncthreads();     // K_f^T(0), K_f^T(1) and V(0) are visible
  } else {
    dma_tile(k_rsrc, 0, dma_k, kx_buf(0));
    if (n_tiles > 1) dma_tile(k_rsrc, 1, dma_k, kx_buf(1));
    dma_wait();
    __syncthreads();
  }

  // A wave without rows (of a head's last block) brings its part of the tiles in and takes no products: what its SIMD and the power
  // allow is the other waves' (200 rows on 32768 keys, H16 d128 86.0 -> 82.2 us, H32 N300 on 16000 130 -> 122, d64 H16 47.1 -> 44.9; tiles of 128 keys, Br256
  // d64 B2 H32 N2122 59.2 -> 56.4). Not in exact blocks of 256 rows with tiles of 128 keys at d = 128, where the addresses that this loop keeps double what the other
  // waves spill (35 registers -> 77; H16 N3072 not causal 140 -> 187, for B2 H8 N420 28.1 -> 24.0).
  if (MODE != kFused && !(MODE == kExact && D == 128 && BR == 256 && BC == 128) && qw0 >= N) {
    __syncthreads();
    for (int it = 0; it < n_tiles - 1; ++it) {
      feed(it, it & 1);
      dma_wait();
      __syncthreads();
    }
    __syncthreads();
    if constexpr (KS == 2) {
      if (n_tiles < n_most) __syncthreads();
      __syncthreads();
    }
    return;
  }
  const std::true_type yes;
  const std::false_type no;
  f32x16 s0[C::MB], s1[C::MB];
  qk(0, s0);             // against the initial reference 0
  apply_mask(0, s0);
  // The first tile sets the reference to its row maximum; nothing has been accumulated yet, so nothing is rescaled. Where that is
  // -infinity the reference stays 0 until a later tile has a score above it, for good if none has.
  const float first_max = tile_max(s0);
  shift_reference(first_max > -INFINITY ? first_max : 0.0f, no, s0, no, s1);
  if (LATE_FIRST && !(first_max > -INFINITY)) trigger = -1.0f;
  // The first iteration refills the buffer of tile 0 (direct load of K(2), or the fusion of
  // K_f^T(2)): every wave must have read its scores of tile 0 out of it first.
  __syncthreads();

  // Tile it+1 needs no mask while it+1 < n_full. The main loop is unrolled by two so that the
  // two score register sets swap roles without copies.
  int it = 0;
  // (at d = 128 blocks of 64 rows run one wave per SIMD, which waits for its instructions itself: by where the loop lies in the 64-byte lines
  // H8 N4000 Nk5000 took 91 to 103 us; exact d64 Br128 H32 N2048 26.95 | 26.80, H16 N4096 46.16 | 46.04; fused d64 Br256 with tiles of 32 keys H12 N5276
  // 117.9 | 115.6)
  if constexpr ((FUSED && D == 64 && BR == 256 && BC == 32) || (D == 128 && BR == 64 && KS == 1) || (D == 64 && BR == 128 && KS == 1 && MODE == kExact)) asm volatile(".p2align 6");
  for (; it + 2 < n_full; it += 2) {
    body(no, yes, it, 0, s0, s1);
    body(no, yes, it + 1, 1, s1, s0);
  }
  for (; it < n_tiles - 1; ++it) {   // at most two unmasked leftovers plus the masked tiles
    body(yes, yes, it, it & 1, s0, s1);
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) s0[mb] = s1[mb];
  }
  body(no, no, it, it & 1, s0, s1);

  // ---- epilogue: O = O_acc / l, bf16, 8-byte stores ---------------------------------------------
  float l_tot = half_swap_sum(l_run);
  constexpr int OB = D / 32 / KS;            // 32-channel blocks of the output that this wave finishes
  const int c0 = KS == 2 ? half * (D / 2) : 0;
  f32x16 out[OB];
  if constexpr (KS == 2) {
    // Each half hands the other one half of the channels and finishes the rest; a lane has the same row in both. The references
    // are the rounded ones that the halves' P were taken against, so that a weight has the rounding of one subtraction.
    if (n_tiles < n_most) __syncthreads();   // (the other half's last tile)
    static_assert(C::RW * OB * 4096 <= KS * C::TILEB && KS * C::RW * 32 * 8 <= KS * C::KX_BYTES, "the exchange fits the tile buffers");
    f32x2* stat = (f32x2*)kx_lds0;
    f32x4* give = (f32x4*)(half ? v_lds1 : v_lds0) + rw * (OB * 256) + lane;
    const f32x4* take = (const f32x4*)(half ? v_lds0 : v_lds1) + rw * (OB * 256) + lane;
    if (hh == 0) stat[wave * 32 + lq] = f32x2{-nref, l_tot};
#pragma unroll
    for (int mb = 0; mb < OB; ++mb) {
      f32x16 theirs;
      if (half) {
        theirs = oacc[mb];
        out[mb] = oacc[mb + OB];
      } else {
        theirs = oacc[mb + OB];
        out[mb] = oacc[mb];
      }
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) give[(mb * 4 + i4) * 64] = f32x4{theirs[4 * i4], theirs[4 * i4 + 1], theirs[4 * i4 + 2], theirs[4 * i4 + 3]};
    }
    __syncthreads();
    // (a half that saw nothing of a row has sum 0 and no reference; a NaN sum makes the row NaN)
    const f32x2 st = stat[(wave ^ C::RW) * 32 + lq];
    const float mine_ref = l_tot > 0.0f ? -nref : -INFINITY, other_ref = st[1] > 0.0f ? st[0] : -INFINITY;
    const float ref = fmaxf(mine_ref, other_ref);
    const float wm = mine_ref > -INFINITY ? __builtin_amdgcn_exp2f(mine_ref - ref) : 0.0f;
    const float wo = other_ref > -INFINITY ? __builtin_amdgcn_exp2f(other_ref - ref) : 0.0f;
    l_tot = __builtin_fmaf(wm, l_tot, wo * st[1]);
    nref = ref > -INFINITY ? -ref : 0.0f;   // (an empty share of n_split)
#pragma unroll
    for (int mb = 0; mb < OB; ++mb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 x = take[(mb * 4 + i4) * 64];
#pragma unroll
        for (int j = 0; j < 4; ++j) out[mb][4 * i4 + j] = __builtin_fmaf(wm, out[mb][4 * i4 + j], wo * x[j]);
      }
  } else {
#pragma unroll
    for (int mb = 0; mb < OB; ++mb) out[mb] = oacc[mb];
  }
  if (n_split > 1) {
    if (q_abs < N) {
      if (hh == 0 && half == 0) part_stat[q_abs] = f32x2{-nref, l_tot};
      float* prow = part_o + (size_t)q_abs * D + c0;
#pragma unroll
      for (int mb = 0; mb < OB; ++mb)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *(f32x4*)(prow + 32 * mb + 8 * i4 + 4 * hh) =
              f32x4{out[mb][4 * i4], out[mb][4 * i4 + 1], out[mb][4 * i4 + 2], out[mb][4 * i4 + 3]};
    }
    return;
  }
  const float inv = 1.0f / l_tot;
  // row statistics for a backward pass: ln(sum of exp(score)) = ln 2 * (reference + log2(l))
  if (lse && q_abs < N && hh == 0 && half == 0) lse[(size_t)bh * N + q_abs] = 0.6931471805599453f * (__builtin_log2f(l_tot) - nref);
  if (q_abs < N) {
    bf16* orow = o + ((size_t)bh * N + q_abs) * D + c0;
#pragma unroll
    for (int mb = 0; mb < OB; ++mb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        bf16x4 pk;
#pragma unroll
        for (int j = 0; j < 4; ++j) pk[j] = (bf16)(out[mb][4 * i4 + j] * inv);
        *(bf16x4*)(orow + 32 * mb + 8 * i4 + 4 * hh) = pk;
      }
  }
}

template <int D, int BR, int BC, int KRED, int MODE, int NG, int KS, bool MATRIX_SUM>
hipError_t launch_sum(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                      const void* kt, const Problem& pb, hipStream_t stream) {
  const int Tq = (pb.N + BR - 1) / BR;
  const long long units = (long long)pb.B * pb.H * Tq;
  const float scale_log2e = pb.scale * 1.4426950408889634f;
  // causal_mode 2 = blocks issued longest first over all heads (see the kernel): for problems
  // of up to 8 workgroups per compute unit, where load balance matters more than L2 locality
  // (with more blocks the dispatcher balances by itself and the head-major order fetches half
  // as many bytes from HBM). 3 = the second round of them reversed: where two workgroups share a compute unit (blocks
  // of 256 rows fill one: H16 N8192 d128 exact 249 us, 287 reversed) and, fused at d = 64, up to three rounds (three
  // fit there, beyond them it is even: N7500 H16 120 | 119, N3700 H32 66 | 67). Measured, 2 | 3, exact and fused:
  //   d64   H32 N2048 30.0 | 28.6, 35.7 | 33.4; H32 N2500 40.0 | 36.2, 42.5 | 39.5; H24 N4096 67.4 | 62.5, 68.3 | 63.4
  //         exact, more rounds: H32 N4096 79.1 | 76.4, H16 N7500 132 | 123, H32 N6000 155.3 | 154.8
  //   d128  H32 N2048 47.9 | 44.4, 53.3 | 50.6; H16 N4096 82.3 | 75.9, 88.7 | 82.3; H16 N8192 264 | 253, 253 | 242
  const bool paired = BR <= 128 && (MODE != kFused || D == 128 || units <= 3 * kComputeUnits);
  const int causal_mode = pb.causal ? (units <= 8 * kComputeUnits ? (paired ? 3 : 2) : 1) : 0;
  hipLaunchKernelGGL((attn_bf16_kernel<D, BR, BC, KRED, MODE, NG, KS, MATRIX_SUM>), dim3((unsigned)(units * pb.n_split)), dim3(BR * 2 * KS), 0,
                     stream, (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, perm, (const f16*)kt,
                     (pb.Nk + kKtPad - 1) / kKtPad * kKtPad, pb.H, pb.Hkv, pb.N, pb.Nk, Tq, causal_mode,
                     scale_log2e, (int)units, pb.n_planes, pb.gray_mode, pb.seed, pb.lse,
                     kt ? (const char*)kt + kt_copy_bytes(pb.B, pb.Hkv, pb.d, pb.Nk) : nullptr,
                     MODE != kExact ? pb.perm_w : nullptr, pb.n_groups, __builtin_ctz(pb.Br), pb.table_in_o, pb.n_split, pb.part_o, (f32x2*)pb.part_stat);
  return hipGetLastError();
}

template <int D, int BR, int BC, int KRED, int MODE, int NG, int KS>
hipError_t launch_ks(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                     const void* kt, const Problem& pb, hipStream_t stream) {
  constexpr bool kSum = kMatrixSum<D, BR, BC, MODE, NG, KS>;
  // Blocks of 64 rows at d = 128 (one wave per SIMD) take their row sums by dot products on long walks that keep the whole chip busy: 24 tiles and
  // more, but for the prompts of a causal call, whose blocks differ in length. us, dot products | matrix pipe: H16 Hkv4 N563 on 15710 keys 95.5 |
  // 103.9, H32 N922 on 8710 148.9 | 156.6, H16 N318 on 13807 57.2 | 59.7, H8 N4000 not causal 77.3 | 84.0, H12 N1847 41.3 | 43.1, H16 N189 on 17275 48.5 | 49.5; but
  // causal H16 N1500 33.5 | 32.6, N3000 59.0 | 57.0, H8 N4000 on 5000 81.7 | 80.0, exact H16 N1000 15.6 | 14.9, N150 on 3000 (5 tiles) 18.4 | 17.4, N944 on 2865 (22) 32.3 | 30.5.
  // Exact blocks of 128 rows at d = 64 that walk all keys: by dot products under the mask while blocks go longest first over all heads, where the last of them leave a
  // wave to a SIMD (H32 N2048 25.3 | 25.9, H16 N4096 44.0 | 44.5, H32 Hkv8 N4096 81.9 | 81.9; but B4 H32 N2500 132.9 | 130.7, not causal 206.5 | 203.6, B16 H12 N412 19.0 | 18.3).
  if constexpr (D == 128 && BR == 64 && BC == 64 && kSum) {
    if (!(pb.causal && pb.Nk < 2LL * pb.N) && (pb.Nk + BC - 1) / BC / pb.n_split / KS >= 24)
      return launch_sum<D, BR, BC, KRED, MODE, NG, KS, false>(q, k, v, o, perm, kt, pb, stream);
  }
  if constexpr (D == 64 && BR == 128 && MODE == kExact && KS == 1) {
    if (pb.causal && (long long)pb.B * pb.H * ((pb.N + BR - 1) / BR) <= 8 * kComputeUnits)
      return launch_sum<D, BR, BC, KRED, MODE, NG, KS, false>(q, k, v, o, perm, kt, pb, stream);
  }
  return launch_sum<D, BR, BC, KRED, MODE, NG, KS, kSum>(q, k, v, o, perm, kt, pb, stream);
}

template <int D, int BR, int BC, int KRED, int MODE, int NG = KRED>
hipError_t launch_one(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                      const void* kt, const Problem& pb, hipStream_t stream) {
  // Two halves of the keys per workgroup (KS = 2) where workgroups of one half each would leave SIMDs with a wave or none:
  // the longest block's walk is halved, and the prologue's grouping has twice the threads. Blocks of 64 rows: as many workgroups as
  // are resident with twice the waves. Blocks of 128 rows, whose eight waves then fill a compute unit and meet at every
  // tile's barrier: one for each, and walks long enough to pay for the exchange at the end. Where blocks find no tiles of each other in an
  // L2 the walk waits for memory, in halves for the later of two loads (waves wait 41 % of their cycles, whole 27 %): long shares of
  // 64-row blocks at d = 64 stay whole there, and at d = 128 middling ones of 128-row blocks. us, KS 1 | 2, exact and distr:
  //   Br64  d64  B2 H32 Hkv8 N200 Nk8000 63 | 47, 68 | 52; H16 Hkv4 N700 Nk12000 86 | 57, 94 | 62; H32 N1000 Nk4000 52 | 39, 57 | 42;
  //              H12 N400 8.2 | 7.6, 12.2 | 10.5; 672 workgroups (B8 H12 N400) 12.8 | 15.1, 17.2 | 20.6
  //              nothing shared, causal: H11 N700 (4 shares) Nk16000 64.2 | 70.5, 69.9 | 75.8, but B3 H9 Hkv3 N300 Nk16000 (15 blocks on 8 XCDs)
  //              81 | 59, 86 | 63, and H250 N50 Nk8000 (2 shares) 1.06 | 1; 4 tiles a share, H13 N64 Nk8000, 1.05 | 1
  //         d128 H12 N400 11.4 | 10.3, 18.4 | 15.0; H16 N1024 21.5 | 16.5, 27.8 | 21.2; 512 workgroups 59 | 69, 65 | 78
  //   Br128 causal, d64 H8 N4096 40.1 | 35.0, 43.1 | 37.9; d128 59.8 | 54.4, 66.4 | 60.1; H16 N2048 33.5 | 31.9, 40.3 | 37.4;
  //         16 tiles and fewer (N1024, N512) 0-9 % slower; 512 workgroups (H32 N2048) 29.6 | 29.5, 36.0 | 39.4; not causal d128
  //         exact H16 N2048 38.4 | 39.2; 24 tiles, one block a head: H16 N54 Nk1500 KS 2 7 % faster, H250 N60 4 % slower, from 62 on 5 % faster
  //         d128, nothing shared, tiles per share: H11 N700 Nk5000 (26) 34.9 | 36.6, H32 Hkv8 N100 Nk16000 (31) 1 | 1.09, H25 N200 Nk16000 (50)
  //         68.8 | 71.2, but H100 N100 Nk8000 (62) 99 | 92, Nk16000 (125) 176 | 160, H28 N180 Nk30000 (117) 149 | 135
  if constexpr (BC == 64 && BR <= 128) {
    constexpr bool GROUPED = MODE != kExact;
    const long long wgs = (long long)pb.B * pb.H * ((pb.N + BR - 1) / BR) * pb.n_split;
    const int tiles = (pb.Nk + BC - 1) / BC / pb.n_split;
    const bool halves =
        BR == 64 ? wgs <= (D == 64 ? 2 : 1) * kComputeUnits && tiles >= 4 &&
                       (D == 128 || pb.n_split <= 2 || tiles < 12 || blocks_sharing_l2(pb, BR) > (pb.causal ? 11 : 8))
                 : wgs <= kComputeUnits && tiles >= (pb.N <= BR && pb.n_split == 1 && wgs > kComputeUnits / 2 ? 32 : 24) &&
                       (D == 64 || ((GROUPED || pb.causal) && (pb.n_split == 1 || tiles > 64 || (pb.N > BR && blocks_sharing_l2(pb, BR) >= 12))));
    if (halves)
      return launch_ks<D, BR, BC, KRED, MODE, NG, 2>(q, k, v, o, perm, kt, pb, stream);
  }
  return launch_ks<D, BR, BC, KRED, MODE, NG, 1>(q, k, v, o, perm, kt, pb, stream);
}

// Group counts built for a K/V tile of BC rows: every supported one for the default tile of
// 64 rows, the common ones (16, 32, 64 groups) for the tiles of the block-size study.
constexpr bool attn_bf16_groups_built(int BC, int d, int n_groups) {
  if (n_groups > d || d % n_groups != 0 || d / n_groups > 16) return false;
  if (n_groups == d) return true;   // exact product
  if (BC == 64) return n_groups == 4 || n_groups == 8 || n_groups == 16 || n_groups == 32 || n_groups == 64;
  return n_groups == 16 || n_groups == 32 || n_groups == 64;
}

template <int D, int BR, int BC>
hipError_t dispatch_kred(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                         const void* kt, const Problem& pb, int distr, hipStream_t stream) {
  if (!distr) return launch_one<D, BR, BC, D, kExact>(q, k, v, o, nullptr, nullptr, pb, stream);
  if (!kt) return launch_one<D, BR, BC, D, kReplicated>(q, k, v, o, perm, nullptr, pb, stream);
  switch (pb.n_groups) {   // n_groups = d (groups of one channel) is the exact product: dispatched by the caller
    case 4:                // fewer groups than one MFMA step: contraction zero-padded to 16
      if constexpr (D == 64 && BC == 64) return launch_one<D, BR, BC, 16, kFused, 4>(q, k, v, o, perm, kt, pb, stream);
      return hipErrorInvalidValue;
    case 8:
      if constexpr (BC == 64) return launch_one<D, BR, BC, 16, kFused, 8>(q, k, v, o, perm, kt, pb, stream);
      return hipErrorInvalidValue;
    case 16: return launch_one<D, BR, BC, 16, kFused>(q, k, v, o, perm, kt, pb, stream);
    case 32: return launch_one<D, BR, BC, 32, kFused>(q, k, v, o, perm, kt, pb, stream);
    case 64:
      if constexpr (D == 128) return launch_one<D, BR, BC, 64, kFused>(q, k, v, o, perm, kt, pb, stream);
      [[fallthrough]];
    default: return hipErrorInvalidValue;
  }
}

// Every (head dim, Q block rows) pair for one K/V tile size; one translation unit per tile size.
template <int BC>
hipError_t dispatch_shape(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                          const void* kt, const Problem& pb, int distr, hipStream_t stream) {
  const int rows = pb.rows ? pb.rows : pb.Br;
  if (pb.d == 64 && rows == 64) return dispatch_kred<64, 64, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.d == 64 && rows == 128) return dispatch_kred<64, 128, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.d == 64 && rows == 256) return dispatch_kred<64, 256, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.d == 128 && rows == 64) return dispatch_kred<128, 64, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.d == 128 && rows == 128) return dispatch_kred<128, 128, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.d == 128 && rows == 256) return dispatch_kred<128, 256, BC>(q, k, v, o, perm, kt, pb, distr, stream);
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace da
