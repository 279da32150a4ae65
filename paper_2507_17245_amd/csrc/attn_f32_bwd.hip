// Backward of the attention forward (exact and DistrAttention) for gfx950 in float arithmetic: the
// reference-precision path, for float tensors (bf16 tensors take the matrix-core kernels of
// attn_bf16_bwd.hip). Products on v_mfma_f32_32x32x2_f32 (float operands and sums), in groups of two and four channels at d = 64
// most of them by bf16 pieces (f32_tiles.h), no atomics (results do not depend on the run), no scratch.
//
// The paper trains through the approximation (Sec. 4.3, 4.4) and gives no gradient. Computed
// here: the derivative of the forward with every Q block's grouping held fixed (the permutation
// is a piecewise-constant function of Q). With P = softmax(S^) rebuilt from the saved row
// statistics, dP = dO V^T, D_i = sum_c dO_ic O_ic and dS^ = P o (dP - D):
//   dV = P^T dO
//   dQ[:, first channel of group j] = scale * (dS^ K_f)[:, j]; the other columns of the block 0
//   dK[:, c] = scale * sum over Q blocks of (dS^T Q_r)[:, group of c in that block]
// (Eq. 2 with Q_r the sampled and K_f the fused columns of Sec. 3.2; one grouping per Q block,
// Sec. 3.3). Exact attention is the case of one channel per group.
//
//   bwd_delta_kernel  D_i of every row, left at the head of dq, which the last kernel overwrites
//   bwd_dkv_kernel    one workgroup per (kv head, 32 keys), lane = key, K and V rows resident; its waves deal the 32-row query tiles of all query heads of the kv head
//                     out among themselves. Groups of 2 and 4 channels: a wave takes a run of tiles, sums K_f of its keys once for
//                     every Q block it enters and reads Q_r (gathered from global memory, groups' order) for S^ and
//                     dK_f, both over n_groups; dK_f of a Q block meets the channels by way of LDS when the wave leaves it.
//                     Other group sizes: Q~ = Q whose channels are replaced by their group's sampled one (dK =
//                     scale dS^T Q~: every member of a group receives its group's column).
//   bwd_dq_kernel     one workgroup per 32 query rows, lane = query row, waves deal the key tiles
//                     out. Groups of 2 and 4 channels: the K tile lies in LDS in sorted channel order,
//                     members adjacent and summed as they are read, S^ and dQ_r contract over
//                     n_groups; other group sizes take Q~ and sum dQ~ over the members at the end.
//   bwd_dkv_pieces_kernel, bwd_dq_pieces_kernel   the same by pieces, for calls that float_by_pieces names
// The waves' partial sums meet in LDS once, at the end, in a fixed order: as in the forward no wave waits
// for another before that, and few rows still give every SIMD work. Bound: the matrix
// instruction (64 cycles for 4096 FLOP): 7 products over d per (query, key) pair, 5 with groups of two, 4 with groups
// of four. Measured on it (B1 H8 N2048 d64 n_groups 32; by pieces 126 and 75 us): delta 4, dK/dV 144, dQ 91 us; the matrix pipes are busy 60 and 62 % of the launch
// (67 and 71 % of the cycles in which their CU has work), the waves wait for them to take an instruction 57 and 68 % of their cycles
// and for memory, LDS and barriers 23 and 14 %; tiles hit the L2 (95 %). (dK/dV with S^ and dK over the groups' members, K_f summed for every tile anew: 176 us; backward d128 642 -> 504 us, groups of four
// 572 -> 411; float multiply-adds on the vector ALUs: dK/dV 2740, dQ 1980 us).
#include <type_traits>

#include "f32_tiles.h"

namespace da {

namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr float kLog2e = 1.4426950408889634f;

typedef Quad<float> Q4;

typedef __attribute__((address_space(3))) void lds_void;

// A row of 32-row tile registers: piece u of a lane is row (u*64 + lane) / (D/4) of the tile, channels
// 4*((u*64 + lane) % (D/4)) ..; rows past the end of the head read as zeros.
template <int D>
struct Tile {
  static constexpr int KU = kTile * D / 4 / 64;
  static constexpr int RS = D + 4;   // LDS row length: 16-byte aligned rows whose starts are 4 banks apart
  static constexpr int BYTES = kTile * D * 4;
  u32x4 x[KU];
  __device__ void load(__amdgpu_buffer_rsrc_t rsrc, int tile, int lane) {
#pragma unroll
    for (int u = 0; u < KU; ++u) x[u] = Q4::load(rsrc, (u * 64 + lane) * 16, tile * BYTES);
  }
  // every channel replaced by `from` (the lane's four channels, the same in all its pieces)
  __device__ void gather(__amdgpu_buffer_rsrc_t rsrc, int tile, int lane, uint32_t from) {
#pragma unroll
    for (int u = 0; u < KU; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        x[u][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (u * 64 + lane) / (D / 4) * (D * 4) + ((from >> (8 * e)) & (D - 1)) * 4, tile * BYTES, 0);
  }
  __device__ void store(float* lds, int lane) const {
#pragma unroll
    for (int u = 0; u < KU; ++u) *(u32x4*)&lds[(u * 64 + lane) / (D / 4) * RS + (u * 64 + lane) % (D / 4) * 4] = x[u];
  }
  __device__ void scatter(float* lds, int lane, const int (&to)[4]) const {
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const f32x4 y = Q4::values(x[u]);
#pragma unroll
      for (int e = 0; e < 4; ++e) lds[(u * 64 + lane) / (D / 4) * RS + to[e]] = y[e];
    }
  }
};

// The tile straight into LDS, rows of D floats with 16 bytes behind every 256 floats (what was read there has arrived).
template <int D>
struct TileToLds {
  static constexpr int KU = Tile<D>::KU, BYTES = Tile<D>::BYTES, FLOATS = KU * 260;
  // Float c of a row: one instruction leaves 256 floats in a row (four rows at D = 64), 16 bytes lie between two instructions'.
  static __device__ int at(int row, int c) { return row / (256 / D) * 260 + row % (256 / D) * D + c; }
  int voff;
  __device__ explicit TileToLds(int lane) : voff(lane * 16) {}
  __device__ void load(__amdgpu_buffer_rsrc_t rsrc, int tile, float* dst) const {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < KU; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + u * 260), 16, voff, tile * BYTES + u * 1024, 0, 0);
  }
};

// dP = dO V^T. (64 channels: one chain is precise enough, and the chains' joints cost 2 % of the backward.)
template <int D>
using DpSum = typename std::conditional<D == 64, OneChain, ChannelSum<D / 2>>::type;

// (tile rows as lanes) x (operand b): contraction over the channels hh*D/2 + s of step s
template <int D, typename SUM = ChannelSum<D / 2>>
__device__ inline f32x16 row_product(const float* row, int hh, const float (&b)[D / 2]) {
  SUM acc;
#pragma unroll
  for (int c = 0; c < D / 2; c += 4) {
    const f32x4 x = *(const f32x4*)&row[hh * (D / 2) + c];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc.step(c + e, x[e], b[c + e]);
  }
  return acc.sum();
}
// the same with the operand b as a row in LDS
template <int D, typename SUM = ChannelSum<D / 2>>
__device__ inline f32x16 row_product(const float* row, int hh, const float* b) {
  SUM acc;
#pragma unroll
  for (int c = 0; c < D / 2; c += 4) {
    const f32x4 x = *(const f32x4*)&row[hh * (D / 2) + c], y = *(const f32x4*)&b[hh * (D / 2) + c];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc.step(c + e, x[e], y[e]);
  }
  return acc.sum();
}
// (rows of KRED floats, HS = KRED/2 of them from either half of the wave) x (operand b)
template <int HS>
__device__ inline f32x16 group_product(const float* row, int hh, const float (&b)[HS]) {
  ChannelSum<HS> acc;
#pragma unroll
  for (int c = 0; c < HS; c += 4) {
    const f32x4 x = *(const f32x4*)&row[hh * HS + c];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc.step(c + e, x[e], b[c + e]);
  }
  return acc.sum();
}
// acc[mb] += (tile transposed) x (accumulator p as operand): lane m owns channels NB*m .. NB*m + NB-1
template <int D>
__device__ inline void column_product(const float* tile, int lq, int hh, const f32x16& p, f32x16 (&acc)[D / 32]) {
  constexpr int NB = D / 32, RS = Tile<D>::RS;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float* src = &tile[acc_row(i, hh) * RS + lq * NB];
    float x[NB];
    if constexpr (NB == 2) {
      const f32x2 y = *(const f32x2*)src;
      x[0] = y[0], x[1] = y[1];
    } else {
      const f32x4 y = *(const f32x4*)src;
      x[0] = y[0], x[1] = y[1], x[2] = y[2], x[3] = y[3];
    }
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = mfma(x[mb], p[i], acc[mb]);
  }
}
// the accumulators of column_product into LDS rows (row = lane's own)
template <int D>
__device__ inline void store_columns(float* row, int hh, const f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = acc_row(i, hh);
    if constexpr (D == 64) *(f32x2*)&row[m * 2] = f32x2{acc[0][i], acc[1][i]};
    else *(f32x4*)&row[m * 4] = f32x4{acc[0][i], acc[1][i], acc[D / 32 - 2][i], acc[D / 32 - 1][i]};
  }
}

// ------------------------------------------------------------------------------------------------
// D_i of 256 / (D/4) rows per workgroup.
template <int D>
__global__ __launch_bounds__(kThreads) void bwd_delta_kernel(const float* __restrict__ o, const float* __restrict__ dout,
                                                             float* __restrict__ delta, size_t rows) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;   // 4-channel piece
  float s = 0.0f;
  if (i < rows * (D / 4)) {
    const f32x4 a = *(const f32x4*)(o + i * 4), b = *(const f32x4*)(dout + i * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) s = __builtin_fmaf(a[e], b[e], s);
  }
#pragma unroll
  for (int m = 1; m < D / 4; m <<= 1) s += __shfl_xor(s, m);
  if (i % (D / 4) == 0 && i < rows * (D / 4)) delta[i / (D / 4)] = s;
}

// ------------------------------------------------------------------------------------------------
// W waves. Eight at d = 64, two per SIMD, with the K and V rows that all of them multiply by in LDS; four, with V in
// registers, at d = 128, where their tiles fill the LDS but for K's, and for fewer than eight query tiles, which would
// leave waves without any (backward of d = 64, four | eight waves: H8 N2048 248 | 237 us, H8 Hkv2 N1024 causal 189 | 171,
// H8 N256 29.1 | 27.9, H1 N64 17.2 | 17.7). K in registers at d = 128 spilled 97 of them (backward, exact,
// H8 N1024: 203 us; in LDS 151).
// G: channels per group where the scores are summed over the groups, as the forward sums them (2, 4); 1: over the
// channels, with Q~. P = exp(S - lse) then rests on the bits of S that lse was taken of: with S over the channels and lse
// of sums over groups, scores of 25 put dK and dV 2.6 times as far from 64 bits.
template <int D, int W, int G>
__global__ __launch_bounds__(W * 64, W / 4) void bwd_dkv_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dk, float* __restrict__ dv,
    const uint8_t* __restrict__ perm, int H, int Hkv, int N, int Nk, int Br, int Tq, int n_groups, int causal, float scale) {
  constexpr int NB = D / 32, RS = Tile<D>::RS;
  constexpr bool SHARED = W == 8, K_LDS = SHARED || G > 1 || D == 128;
  __shared__ __attribute__((aligned(16))) float q_lds[W][kTile * RS];    // Q~ tile of each wave, at the end its dK
  __shared__ __attribute__((aligned(16))) float do_lds[W][kTile * RS];   // dO tile, at the end dV
  __shared__ __attribute__((aligned(16))) float k_lds[K_LDS ? kTile * RS : 4];
  __shared__ __attribute__((aligned(16))) float v_lds[SHARED ? kTile * RS : 4];
  __shared__ __attribute__((aligned(16))) float stat_lds[W][2][kTile];   // lse, D_i
  // G = 1: sorted order, sampled channel of a channel's group. G > 1: of this Q block and the one before or after it, sorted
  // order and the channels' groups
  __shared__ __attribute__((aligned(16))) uint8_t map_lds[W][G > 1 ? 4 : 2][D];
  // G > 1: Q_r, KRED sampled channels a row, in groups' order; ROWS of its rows per load
  constexpr int KRED = D / G, HS = KRED / 2, RQ = KRED + 4, NG = (KRED + 31) / 32, ROWS = G > 1 ? 64 / KRED : 1, QL = kTile / ROWS;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  // causal: the keys that most queries see come first; the tile index is the slow one, so that a
  // kv head stays on one XCD when their number is a multiple of 8
  const int n_bk = gridDim.x / ((Nk + kTile - 1) / kTile);
  const int t = blockIdx.x / n_bk, bk = blockIdx.x % n_bk;
  const int b = bk / Hkv, hk = bk % Hkv, rep = H / Hkv;
  const int n0 = t * kTile, key = n0 + lq;
  const int shift = Nk - N;   // causal: query i sees key n iff n <= i + shift
  const int group = G > 1 ? G : D / n_groups;

  const int first = causal ? max(0, n0 - shift) / kTile : 0;   // first tile with a row that sees key n0
  const int tiles = (N + kTile - 1) / kTile - first;           // per query head
  const int n_it = tiles * rep;
  auto head_of = [&](int it) { return (size_t)b * H + hk * rep + it / tiles; };
  auto tile_of = [&](int it) { return first + it % tiles; };

  // The sampled channels of the lane's four channels in the block of iteration `it` (0, 1, 2, 3 .. for
  // exact attention), from the bytes of its table row.
  uint8_t map_reg[D / 64];
  auto load_map = [&](int it) {
    const uint8_t* pr = perm + (head_of(it) * Tq + tile_of(it) * kTile / Br) * D;
#pragma unroll
    for (int u = 0; u < D / 64; ++u) map_reg[u] = pr[u * 64 + lane];
  };
  auto sampled = [&]() -> uint32_t {
    uint8_t* order = map_lds[w][0];
    uint8_t* from = map_lds[w][1];
    wave_order();
#pragma unroll
    for (int u = 0; u < D / 64; ++u) order[u * 64 + lane] = map_reg[u] & (D - 1);
    wave_order();
#pragma unroll
    for (int u = 0; u < D / 64; ++u) from[order[u * 64 + lane]] = order[(u * 64 + lane) / group * group];
    wave_order();
    return *(const uint32_t*)&from[lane % (D / 4) * 4];
  };
  typename std::conditional<G == 1, Tile<D>, char>::type qt;
  float qr[QL];
  Tile<D> dt;
  float lse_reg, delta_reg;
  // G > 1: the table of iteration it's Q block into place `slot`; map_reg holds it
  auto block_of = [&](int it) { return (int)(head_of(it) * Tq) + tile_of(it) * kTile / Br; };
  auto store_map = [&](int slot) {
    uint8_t* order = map_lds[w][2 * slot];
    uint8_t* groups = map_lds[w][2 * slot + 1];
    wave_order();
#pragma unroll
    for (int u = 0; u < D / 64; ++u) {
      const int i = u * 64 + lane, c = map_reg[u] & (D - 1);
      order[i] = (uint8_t)c;
      groups[c] = (uint8_t)(i / G);
    }
    wave_order();
  };
  auto load_q = [&](int it, int slot) {
    const size_t bh = head_of(it);
    const int i0 = tile_of(it);
    const __amdgpu_buffer_rsrc_t q_rsrc = head_rsrc(q + bh * N * D, (unsigned)N * D * 4);
    if constexpr (G > 1) {
      const int c = map_lds[w][2 * slot][lane % KRED * G];   // the sampled channel of this lane's group
#pragma unroll
      for (int u = 0; u < QL; ++u)
        qr[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(q_rsrc, lane / KRED * (D * 4) + c * 4, i0 * Tile<D>::BYTES + u * ROWS * (D * 4), 0));
    } else {
      if (perm) qt.gather(q_rsrc, i0, lane, sampled());
      else qt.load(q_rsrc, i0, lane);
    }
    const int row = min(i0 * kTile + lq, N - 1);
    lse_reg = lse[bh * N + row];
    delta_reg = delta[bh * N + row];
  };
  auto load_do = [&](int it) { dt.load(head_rsrc(dout + head_of(it) * N * D, (unsigned)N * D * 4), tile_of(it), lane); };
  // G = 1: the waves deal the tiles out one by one; G > 1: runs of them, so that a wave stays in a Q block
  constexpr int STEP = G > 1 ? 1 : W;
  int it = G > 1 ? n_it * w / W : w;
  const int it_end = G > 1 ? n_it * (w + 1) / W : n_it;
  int slot = 0;
  if (it < it_end) {
    if (perm) load_map(it);
    if constexpr (G > 1) store_map(0);
    load_q(it, 0);
    load_do(it);
    if (perm && it + STEP < it_end) load_map(it + STEP);
  }

  float kop[K_LDS ? 1 : D / 2], vop[SHARED ? 1 : D / 2];
  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)bk * Nk * D, (unsigned)Nk * D * 4);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)bk * Nk * D, (unsigned)Nk * D * 4);
  if constexpr (K_LDS) {
    if (w < (SHARED ? 2 : 1)) {
      Tile<D> x;
      x.load(w ? v_rsrc : k_rsrc, t, lane);
      x.store(w ? v_lds : k_lds, lane);
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int c = 0; c < D / 2; c += 4) {
      const f32x4 x = Q4::values(Q4::load(k_rsrc, (lq * D + hh * (D / 2) + c) * 4, n0 * (D * 4)));
#pragma unroll
      for (int e = 0; e < 4; ++e) kop[c + e] = x[e];
    }
  }
  if constexpr (!SHARED) {
#pragma unroll
    for (int c = 0; c < D / 2; c += 4) {
      const f32x4 y = Q4::values(Q4::load(v_rsrc, (lq * D + hh * (D / 2) + c) * 4, n0 * (D * 4)));
#pragma unroll
      for (int e = 0; e < 4; ++e) vop[c + e] = y[e];
    }
  }
  f32x16 dkacc[NB], dvacc[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) {
    zero(dkacc[mb]);
    zero(dvacc[mb]);
  }
  // G > 1: K_f of the workgroup's keys and dK_f of the Q block the wave is in
  float kf[G > 1 ? HS : 1];
  f32x16 dkf[G > 1 ? NG : 1];
  auto fuse_keys = [&]() {
    if constexpr (G > 1) {
#pragma unroll
      for (int c = 0; c < D / 2; c += 8) {
        const u32x2 e2 = *(const u32x2*)&map_lds[w][2 * slot][hh * (D / 2) + c];
#pragma unroll
        for (int e = 0; e < 8; e += G) {
          float x = k_lds[lq * RS + ((e2[e >> 2] >> (8 * (e & 3))) & (D - 1))];
#pragma unroll
          for (int m = 1; m < G; ++m) x += k_lds[lq * RS + ((e2[(e + m) >> 2] >> (8 * ((e + m) & 3))) & (D - 1))];
          kf[(c + e) / G] = x;
        }
      }
#pragma unroll
      for (int mb = 0; mb < NG; ++mb) zero(dkf[mb]);
    }
  };
  // every channel receives its group's column (register i, lane half hh: groups NG * acc_row(i) .., channels NB * acc_row(i) ..)
  auto unfuse = [&](int of) {
    if constexpr (G > 1) {
      float* mine = &q_lds[w][lq * RQ];
      wave_order();
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int mb = 0; mb < NG; ++mb)
          if (KRED >= 32 || acc_row(i, 0) < KRED) mine[acc_row(i, hh) * NG + mb] = dkf[mb][i];
      wave_order();
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
        for (int c = 0; c < 4 * NB; c += 4) {
          const uint32_t g4 = *(const uint32_t*)&map_lds[w][2 * of + 1][NB * (8 * i4 + 4 * hh) + c];
#pragma unroll
          for (int e = 0; e < 4; ++e) dkacc[(c + e) % NB][4 * i4 + (c + e) / NB] += mine[(g4 >> (8 * e)) & (KRED - 1)];
        }
    }
  };
  int block = it < it_end && G > 1 ? block_of(it) : 0;
  if constexpr (G > 1) {
    if (it < it_end) fuse_keys();
  }

  for (; it < it_end; it += STEP) {
    const int i0 = tile_of(it) * kTile;
    if constexpr (G > 1) {
      if (block_of(it) != block) {
        unfuse(slot);
        slot ^= 1;
        block = block_of(it);
        fuse_keys();
      }
    }
    wave_order();   // the reads of the previous tile come first
    if constexpr (G > 1) {
#pragma unroll
      for (int u = 0; u < QL; ++u) q_lds[w][(u * ROWS + lane / KRED) * RQ + lane % KRED] = qr[u];
    } else {
      qt.store(q_lds[w], lane);
    }
    dt.store(do_lds[w], lane);
    stat_lds[w][hh][lq] = hh ? delta_reg : lse_reg;
    if (it + STEP < it_end) {
      if constexpr (G > 1) {
        const bool same = block_of(it + 1) == block;
        if (!same) store_map(slot ^ 1);
        load_q(it + 1, same ? slot : slot ^ 1);
      } else {
        load_q(it + STEP, 0);
      }
      if (perm && it + 2 * STEP < it_end) load_map(it + 2 * STEP);
    }
    wave_order();
    f32x16 s, dp;
    if constexpr (G > 1) s = group_product<HS>(&q_lds[w][lq * RQ], hh, kf);
    else if constexpr (K_LDS) s = row_product<D>(&q_lds[w][lq * RS], hh, &k_lds[lq * RS]);
    else s = row_product<D>(&q_lds[w][lq * RS], hh, kop);
    if (it + STEP < it_end) load_do(it + STEP);   // (only now: the registers were those of the sum)
    if constexpr (SHARED) dp = row_product<D, DpSum<D>>(&do_lds[w][lq * RS], hh, &v_lds[lq * RS]);
    else dp = row_product<D, DpSum<D>>(&do_lds[w][lq * RS], hh, vop);
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 ls = *(const f32x4*)&stat_lds[w][0][8 * i4 + 4 * hh], dl = *(const f32x4*)&stat_lds[w][1][8 * i4 + 4 * hh];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * i4 + e;
        s[i] = __builtin_amdgcn_exp2f(scaled_plus(s[i], scale, -ls[e]) * kLog2e);
        dp[i] = dp[i] - dl[e];
      }
    }
    if (i0 + kTile > N || (causal && i0 + shift < n0 + kTile - 1)) {   // rows past N; the causal diagonal
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = i0 + acc_row(i, hh);
        if (row >= N || (causal && key > row + shift)) s[i] = 0.0f;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) dp[i] *= s[i];
    // (G > 1: a wave's run of tiles makes the chains of the causal mask's heavy rows long, so that a tile's dV is summed by
    // itself first, like dK; at d = 128 in groups of two, two channel blocks at a time: with four, 36 registers spilled. As it is
    // 12 do there, and 6 and 2 at d = 64 with eight waves in groups of two and four, some of them reloaded at every tile)
    if constexpr (G > 1 && (NB == 2 || G == 4)) {
      f32x16 part[NB];
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) zero(part[mb]);
      column_product<D>(do_lds[w], lq, hh, s, part);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) dvacc[mb] += part[mb];
    } else if constexpr (G > 1) {
#pragma unroll
      for (int m0 = 0; m0 < NB; m0 += 2) {
        f32x16 part[2];
        zero(part[0]);
        zero(part[1]);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const f32x2 x = *(const f32x2*)&do_lds[w][acc_row(i, hh) * RS + lq * NB + m0];
          part[0] = mfma(x[0], s[i], part[0]);
          part[1] = mfma(x[1], s[i], part[1]);
        }
        dvacc[m0] += part[0];
        dvacc[m0 + 1] += part[1];
      }
    } else {
      column_product<D>(do_lds[w], lq, hh, s, dvacc);
    }
    // (a tile's dK is summed by itself first: many heads and rows would make the chain long)
    if constexpr (G > 1) {
      // lane m owns the groups NG*m .. (with 16 groups the upper lanes repeat the lower)
      f32x16 part[NG];
#pragma unroll
      for (int mb = 0; mb < NG; ++mb) zero(part[mb]);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) part[mb] = mfma(q_lds[w][acc_row(i, hh) * RQ + lq * NG % KRED + mb], dp[i], part[mb]);
#pragma unroll
      for (int mb = 0; mb < NG; ++mb) dkf[mb] += part[mb];
    } else {
      f32x16 part[NB];
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) zero(part[mb]);
      column_product<D>(q_lds[w], lq, hh, dp, part);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) dkacc[mb] += part[mb];
    }
  }
  if constexpr (G > 1) {
    if (n_it * w / W < it_end) unfuse(slot);
  }

  wave_order();
  store_columns<D>(&q_lds[w][lq * RS], hh, dkacc);
  store_columns<D>(&do_lds[w][lq * RS], hh, dvacc);
  __syncthreads();
  for (int i = tid; i < kTile * D / 4; i += W * 64) {
    const int row = i / (D / 4), c = i % (D / 4) * 4;
    if (n0 + row < Nk) {
      f32x4 x = *(const f32x4*)&q_lds[0][row * RS + c], y = *(const f32x4*)&do_lds[0][row * RS + c];
#pragma unroll
      for (int j = 1; j < W; ++j) {
        x += *(const f32x4*)&q_lds[j][row * RS + c];
        y += *(const f32x4*)&do_lds[j][row * RS + c];
      }
      const size_t dst = ((size_t)bk * Nk + n0 + row) * D + c;
      *(f32x4*)(dk + dst) = x * scale;
      *(f32x4*)(dv + dst) = y;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Groups of two and four channels at d = 64, from more than eight key tiles on (float_by_pieces): S^ and dP by bf16 pieces (V's lie
// in LDS, K_f's in registers for a Q block), in the same order as the forward, whose lse P = exp(S^ - lse) rests on; dV and dK_f on
// the float instruction, tile by tile. By pieces these need 48 registers more: 70 spilled, and dK/dV took 244 us; with one wave per SIMD and
// none spilled 164. dO and V are raised by 2^24 before they are split (groups of four, H16 N1500: whole backward 195 -> 199 us), a second
// walk takes what pieces do not hold. The dO tile comes straight into LDS as soon as its columns have been read (through registers, 32 spilled: 148).
// Bound: issue and both matrix instructions' time. B1 H8 N2048 n_groups 32: 141 -> 126 us, 16 groups 128 -> 115.
template <int D, int W, int G>
__global__ __launch_bounds__(W * 64, W / 4) void bwd_dkv_pieces_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dk, float* __restrict__ dv,
    const uint8_t* __restrict__ perm, int H, int Hkv, int N, int Nk, int Br, int Tq, int causal, float scale) {
  constexpr int NB = D / 32, RS = Tile<D>::RS;
  constexpr int KRED = D / G, HS = KRED / 2, RQ = KRED + 4, NG = (KRED + 31) / 32, ROWS = 64 / KRED, QL = kTile / ROWS;
  __shared__ __attribute__((aligned(16))) float q_lds[W][kTile * RQ];                  // Q_r tile of each wave: KRED sampled channels a row, in groups' order
  __shared__ __attribute__((aligned(16))) float do_lds[W][TileToLds<D>::FLOATS];   // dO tile, at the end dV and dK
  __shared__ __attribute__((aligned(16))) float k_lds[kTile * RS];                        // of the workgroup's keys
  __shared__ __attribute__((aligned(16))) PieceRows<D> v_lds;
  __shared__ __attribute__((aligned(16))) float stat_lds[W][2][kTile];   // lse, D_i
  __shared__ uint32_t mark_lds[kTile + 1];   // what is known of a key's row (kRowAgain ..); whether a score's operand is beyond_pieces
  __shared__ __attribute__((aligned(16))) uint8_t map_lds[W][4][D];   // of this Q block and the one before or after it: sorted order, the channels' groups

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  // causal: the keys that most queries see come first; the tile index is the slow one, so that a
  // kv head stays on one XCD when their number is a multiple of 8
  const int n_bk = gridDim.x / ((Nk + kTile - 1) / kTile);
  const int t = blockIdx.x / n_bk, bk = blockIdx.x % n_bk;
  const int b = bk / Hkv, hk = bk % Hkv, rep = H / Hkv;
  const int n0 = t * kTile, key = n0 + lq;
  const int shift = Nk - N;   // causal: query i sees key n iff n <= i + shift
  // the rows that see this lane's key: see_from .. see_from + see_rows - 1
  const int see_from = causal ? key - shift : 0;
  const unsigned see_rows = see_from < N ? (unsigned)(N - see_from) : 0u;

  const int first = causal ? max(0, n0 - shift) / kTile : 0;   // first tile with a row that sees key n0
  const int tiles = (N + kTile - 1) / kTile - first;           // per query head
  const int n_it = tiles * rep;
  auto head_of = [&](int it) { return (size_t)b * H + hk * rep + it / tiles; };
  auto tile_of = [&](int it) { return first + it % tiles; };

  uint8_t map_reg[D / 64];   // table row of an iteration's Q block
  auto load_map = [&](int it) {
    const uint8_t* pr = perm + (head_of(it) * Tq + tile_of(it) * kTile / Br) * D;
#pragma unroll
    for (int u = 0; u < D / 64; ++u) map_reg[u] = pr[u * 64 + lane];
  };
  float qr[QL];
  float lse_reg, delta_reg;
  // the table of iteration it's Q block into place `slot`; map_reg holds it
  auto block_of = [&](int it) { return (int)(head_of(it) * Tq) + tile_of(it) * kTile / Br; };
  auto store_map = [&](int slot) {
    uint8_t* order = map_lds[w][2 * slot];
    uint8_t* groups = map_lds[w][2 * slot + 1];
    wave_order();
#pragma unroll
    for (int u = 0; u < D / 64; ++u) {
      const int i = u * 64 + lane, c = map_reg[u] & (D - 1);
      order[i] = (uint8_t)c;
      groups[c] = (uint8_t)(i / G);
    }
    wave_order();
  };
  auto load_q = [&](int it, int slot) {
    const size_t bh = head_of(it);
    const int i0 = tile_of(it);
    const __amdgpu_buffer_rsrc_t q_rsrc = head_rsrc(q + bh * N * D, (unsigned)N * D * 4);
    const int c = map_lds[w][2 * slot][lane % KRED * G];   // the sampled channel of this lane's group
#pragma unroll
    for (int u = 0; u < QL; ++u)
      qr[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(q_rsrc, lane / KRED * (D * 4) + c * 4, i0 * Tile<D>::BYTES + u * ROWS * (D * 4), 0));
    const int row = min(i0 * kTile + lq, N - 1);
    lse_reg = lse[bh * N + row];
    delta_reg = delta[bh * N + row];
  };
  // straight into LDS, behind the last reads of the tile before
  const TileToLds<D> to_lds(lane);
  auto load_do = [&](int it) {
    to_lds.load(head_rsrc(dout + head_of(it) * N * D, (unsigned)N * D * 4), tile_of(it), do_lds[w]);
  };
  auto do_at = [&](int row, int c) { return TileToLds<D>::at(row, c); };
  // the waves deal out runs of tiles, so that a wave stays in a Q block
  const int it_first = n_it * w / W, it_end = n_it * (w + 1) / W;
  int slot = 0;
  auto load_first = [&]() {
    slot = 0;
    if (it_first < it_end) {
      load_map(it_first);
      store_map(0);
      load_q(it_first, 0);
      load_do(it_first);
      if (it_first + 1 < it_end) load_map(it_first + 1);
    }
  };
  load_first();
  if (tid <= kTile) mark_lds[tid] = 0;

  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)bk * Nk * D, (unsigned)Nk * D * 4);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)bk * Nk * D, (unsigned)Nk * D * 4);
  Tile<D> kt;
  if (w == 0) {
    kt.load(k_rsrc, t, lane);
    kt.store(k_lds, lane);
  }
  for (int c = (W - 1 - w) * 8; c < D / 2; c += W * 8) {
    const int at = hh * (D / 2) + c;
    const f32x4 x = Q4::values(Q4::load(v_rsrc, (lq * D + at) * 4, n0 * (D * 4))), y = Q4::values(Q4::load(v_rsrc, (lq * D + at + 4) * 4, n0 * (D * 4)));
    v_lds.store(lq, at, split(f32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]} * kRaise));
  }
  __syncthreads();
  // The rows (keys) of the bit mask `rows`, S^ and dP by pieces or on the float instruction. By pieces, the rows to be taken again are
  // returned; a second walk takes the scores by pieces that the first took by them (beyond_pieces), and with s_again set it is for
  // the keys, too, that have other scores.
  bool s_again = false;
  auto pass = [&](auto pieces, uint32_t rows) -> uint32_t {
    constexpr bool BY_PIECES = decltype(pieces)::value;
    constexpr float raise = BY_PIECES ? kRaise : 1.0f, dp_raise = raise * raise;   // of dO and V; of dP, D_i, dS and dK_f
    const Splitter splitter(lane);
    f32x16 dkacc[NB], dvacc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
      zero(dkacc[mb]);
      zero(dvacc[mb]);
    }
    // K_f of the workgroup's keys and dK_f of the Q block the wave is in
    Pieces kf[HS / 8];
    f32x16 dkf[NG];
    uint32_t any_beyond = 0;
    uint32_t key_beyond = 0;   // of the Q block the wave is in
    auto fused_keys = [&](float (&sum)[HS]) {
#pragma unroll
      for (int c = 0; c < D / 2; c += 8) {
        const u32x2 e2 = *(const u32x2*)&map_lds[w][2 * slot][hh * (D / 2) + c];
#pragma unroll
        for (int e = 0; e < 8; e += G) {
          float x = k_lds[lq * RS + ((e2[e >> 2] >> (8 * (e & 3))) & (D - 1))];
#pragma unroll
          for (int m = 1; m < G; ++m) x += k_lds[lq * RS + ((e2[(e + m) >> 2] >> (8 * ((e + m) & 3))) & (D - 1))];
          sum[(c + e) / G] = x;
        }
      }
    };
    auto fuse_keys = [&]() {
      float sum[HS];
      fused_keys(sum);
      key_beyond = rows_of(beyond_pieces(largest(sum)));
      if constexpr (BY_PIECES) any_beyond |= key_beyond;
      split_steps<HS>(splitter, sum, [&](int s, const Pieces& p) { kf[s] = p; });
#pragma unroll
      for (int mb = 0; mb < NG; ++mb) zero(dkf[mb]);
    };
    // every channel receives its group's column (register i, lane half hh: groups NG * acc_row(i) .., channels NB * acc_row(i) ..)
    auto unfuse = [&](int of) {
      float* mine = &q_lds[w][lq * RQ];
      wave_order();
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int mb = 0; mb < NG; ++mb)
          if (KRED >= 32 || acc_row(i, 0) < KRED) mine[acc_row(i, hh) * NG + mb] = dkf[mb][i];
      wave_order();
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
        for (int c = 0; c < 4 * NB; c += 4) {
          const uint32_t g4 = *(const uint32_t*)&map_lds[w][2 * of + 1][NB * (8 * i4 + 4 * hh) + c];
#pragma unroll
          for (int e = 0; e < 4; ++e) dkacc[(c + e) % NB][4 * i4 + (c + e) / NB] += mine[(g4 >> (8 * e)) & (KRED - 1)];
        }
    };
    int it = it_first, block = it < it_end ? block_of(it) : 0;
    if (it < it_end) fuse_keys();

    for (; it < it_end; ++it) {
      const int i0 = tile_of(it) * kTile;
      if (block_of(it) != block) {
        unfuse(slot);
        slot ^= 1;
        block = block_of(it);
        fuse_keys();
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the dO tile has landed
      wave_order();   // the reads of the previous tile come first
#pragma unroll
      for (int u = 0; u < QL; ++u) q_lds[w][(u * ROWS + lane / KRED) * RQ + lane % KRED] = qr[u];
      if constexpr (BY_PIECES) any_beyond |= rows_of(beyond_pieces(largest(qr)));
      stat_lds[w][hh][lq] = hh ? delta_reg * dp_raise : lse_reg;
      if (it + 1 < it_end) {
        const bool same = block_of(it + 1) == block;
        if (!same) store_map(slot ^ 1);
        load_q(it + 1, same ? slot : slot ^ 1);
        if (it + 2 < it_end) load_map(it + 2);
      }
      wave_order();
      f32x16 s, dp;
      {
        float x[HS];
#pragma unroll
        for (int c = 0; c < HS; c += 4) {
          const f32x4 y = *(const f32x4*)&q_lds[w][lq * RQ + hh * HS + c];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[c + e] = y[e];
        }
        {
          PieceSum acc;
          split_steps<HS>(splitter, x, [&](int s, const Pieces& p) { acc.template step<true>(p, kf[s]); });
          s = acc.sum();
        }
        if constexpr (!BY_PIECES) {
          const uint32_t q_beyond = rows_of(beyond_pieces(largest(x)));
          if ((q_beyond != 0 && i0 + 31 - __builtin_clz(q_beyond) >= see_from) || (key_beyond >> lq & 1) != 0) atomicOr(&mark_lds[lq], kRowBeyond);
          if ((q_beyond | key_beyond) != 0) {
            ChannelSum<HS> acc;
            float y[HS];
            fused_keys(y);
#pragma unroll
            for (int s = 0; s < HS; ++s) acc.step(s, x[s], y[s]);
            const f32x16 z = acc.sum();
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = ((key_beyond >> lq | q_beyond >> acc_row(i, hh)) & 1) != 0 ? z[i] : s[i];
          }
        }
      }
      zero(dp);
#pragma unroll
      for (int c0 = 0; c0 < D / 2; c0 += 16) {
        float x[16];
#pragma unroll
        for (int c = 0; c < 16; c += 4) {
          const f32x4 y = *(const f32x4*)&do_lds[w][do_at(lq, hh * (D / 2) + c0 + c)];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[c + e] = y[e] * raise;
        }
        if constexpr (BY_PIECES) {
          split_steps<16>(splitter, x, [&](int s, const Pieces& p) { dp = mfma(p, v_lds.load(lq, hh * (D / 2) + c0 + 8 * s), dp); });
        } else {
#pragma unroll
          for (int c = 0; c < 16; c += 4) {
            const f32x4 y = Q4::values(Q4::load(v_rsrc, (lq * D + hh * (D / 2) + c0 + c) * 4, n0 * (D * 4)));
#pragma unroll
            for (int e = 0; e < 4; ++e) dp = mfma(x[c + e], y[e], dp);
          }
        }
      }
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 ls = *(const f32x4*)&stat_lds[w][0][8 * i4 + 4 * hh], dl = *(const f32x4*)&stat_lds[w][1][8 * i4 + 4 * hh];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          s[i] = __builtin_amdgcn_exp2f(scaled_plus(s[i], scale, -ls[e]) * kLog2e);
          dp[i] = dp[i] - dl[e];
        }
      }
      if (i0 + kTile > N || (causal && i0 + shift < n0 + kTile - 1)) {   // rows past N; the causal diagonal
        asm volatile("");   // (a branch: few tiles are masked)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = (unsigned)(i0 + acc_row(i, hh) - see_from) < see_rows ? s[i] : 0.0f;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) dp[i] *= s[i];
      {
        f32x16 part[NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) zero(part[mb]);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const f32x2 y = *(const f32x2*)&do_lds[w][do_at(acc_row(i, hh), lq * NB)];
          part[0] = mfma(y[0], s[i], part[0]);
          part[1] = mfma(y[1], s[i], part[1]);
        }
        if (it + 1 < it_end) load_do(it + 1);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) dvacc[mb] += part[mb];
      }
      {
        // lane m owns the groups NG*m .. (with 16 groups the upper lanes repeat the lower)
        f32x16 part[NG];
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) zero(part[mb]);
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int mb = 0; mb < NG; ++mb) part[mb] = mfma(q_lds[w][acc_row(i, hh) * RQ + lq * NG % KRED + mb], dp[i], part[mb]);
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) dkf[mb] += part[mb];
      }
    }
    if (it_first < it_end) unfuse(slot);

    // the waves' sums meet, dV, then dK, by way of the dO tiles
#pragma unroll
    for (int of = 0; of < 2; ++of) {
      if (of) __syncthreads();
      else wave_order();
#pragma unroll
      for (int i = 0; i < 16; ++i)
        *(f32x2*)&do_lds[w][do_at(lq, acc_row(i, hh) * 2)] = of ? f32x2{dkacc[0][i], dkacc[1][i]} : f32x2{dvacc[0][i], dvacc[1][i]};
      __syncthreads();
      for (int i = tid; i < kTile * D / 4; i += W * 64) {
        const int row = i / (D / 4), c = i % (D / 4) * 4;
        if (n0 + row < Nk && ((rows >> row & 1) != 0 || (!BY_PIECES && (mark_lds[row] & kRowBeyond) != 0))) {
          f32x4 x = *(const f32x4*)&do_lds[0][do_at(row, c)];
#pragma unroll
          for (int j = 1; j < W; ++j) x += *(const f32x4*)&do_lds[j][do_at(row, c)];
          if (BY_PIECES && of && !all_finite(x)) atomicOr(&mark_lds[row], kRowAgain);
          *(f32x4*)((of ? dk : dv) + ((size_t)bk * Nk + n0 + row) * D + c) = of ? x * (1.0f / dp_raise) * scale : x;
        }
      }
    }
    if constexpr (!BY_PIECES) return 0;
    if (any_beyond != 0) atomicOr(&mark_lds[kTile], 1u);
    __syncthreads();
    s_again = mark_lds[kTile] != 0;
    return rows_of((mark_lds[lq] & kRowAgain) != 0);
  };
  const uint32_t again = pass(std::true_type(), ~0u);
  if (again == 0 && !s_again) return;
  load_first();
  pass(std::false_type(), again);
}

// ------------------------------------------------------------------------------------------------
// G: channels per group where the score and dQ_r products contract over the groups (2, 4); 1: over the
// channels, with Q~.
template <int D, int G, int W>
__global__ __launch_bounds__(W * 64, (D == 64 ? 2 : 1)) void bwd_dq_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ o,
    const float* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ dq, const uint8_t* __restrict__ perm,
    int H, int Hkv, int N, int Nk, int Br, int Tq, int n_groups, int causal, float scale) {
  constexpr int NB = D / 32, RS = Tile<D>::RS;
  constexpr int KRED = D / G, HS = KRED / 2;
  constexpr int NG = G == 1 ? NB : (KRED + 31) / 32;   // 32-row blocks of the dQ_r accumulator
  __shared__ __attribute__((aligned(16))) float k_lds[W][kTile * RS];   // at the end the wave's dQ_r
  __shared__ __attribute__((aligned(16))) float v_lds[W][kTile * RS];
  __shared__ uint8_t order_lds[D];   // sorted order of the block's channels
  __shared__ uint8_t map_lds[D];     // G > 1: a channel's position in it; G = 1: its group's sampled channel
  __shared__ uint8_t pos_lds[D];     // (G = 1) a channel's position in the sorted order

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const int Tw = (N + kTile - 1) / kTile;
  const int n_bh = gridDim.x / Tw;
  const int t = causal ? Tw - 1 - (int)blockIdx.x / n_bh : (int)blockIdx.x / n_bh;   // longest first
  const int bh = blockIdx.x % n_bh;
  const int b = bh / H, hk = bh % H / (H / Hkv);
  const int r0 = t * kTile, q_abs = r0 + lq;
  const int shift = Nk - N;
  const int group = D / n_groups;

  const size_t head = (size_t)bh * N * D;
  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)(b * Hkv + hk) * Nk * D, (unsigned)Nk * D * 4);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)(b * Hkv + hk) * Nk * D, (unsigned)Nk * D * 4);
  const int n_end = causal ? min(Nk, r0 + kTile + shift) : Nk;
  const int n_tiles = (n_end + kTile - 1) / kTile;
  const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;   // last key this row sees

  Tile<D> kt, vt;
  if (w < n_tiles) {
    kt.load(k_rsrc, w, lane);
    vt.load(v_rsrc, w, lane);
  }
  // Q, dO and O rows pass through LDS (one tile per wave 0, 1, 2)
  {
    const float* src = w == 0 ? q : w == 1 ? dout : o;
    Tile<D> x;
    if (w < 3) {
      x.load(head_rsrc(src + head, (unsigned)N * D * 4), t, lane);
      x.store(w == 2 ? v_lds[0] : k_lds[w], lane);
    }
  }
  if (perm) {
    // D is a power of two: an out-of-range entry of a caller's table cannot index past a row
    const uint8_t* pr = perm + ((size_t)bh * Tq + r0 / Br) * D;
    for (int i = tid; i < D; i += (W * 64)) {
      order_lds[i] = pr[i] & (D - 1);
      pos_lds[pr[i] & (D - 1)] = (uint8_t)i;
      map_lds[pr[i] & (D - 1)] = G > 1 ? (uint8_t)i : (uint8_t)(pr[i / group * group] & (D - 1));
    }
  } else {
    for (int i = tid; i < D; i += (W * 64)) order_lds[i] = map_lds[i] = (uint8_t)i;
  }
  __syncthreads();
  float qop[HS], doop[D / 2], dl = 0.0f;
  int kdst[4];
#pragma unroll
  for (int s = 0; s < HS; ++s)
    qop[s] = k_lds[0][lq * RS + (G > 1 ? order_lds[(hh * HS + s) * G] : (map_lds[hh * HS + s] & (D - 1)))];
#pragma unroll
  for (int c = 0; c < D / 2; ++c) {
    doop[c] = k_lds[1][lq * RS + hh * (D / 2) + c];
    dl = __builtin_fmaf(doop[c], v_lds[0][lq * RS + hh * (D / 2) + c], dl);
  }
  dl = half_swap_sum(dl);
#pragma unroll
  for (int e = 0; e < 4; ++e) kdst[e] = map_lds[lane % (D / 4) * 4 + e] & (D - 1);
  const float lse_row = lse[(size_t)bh * N + min(q_abs, N - 1)];
  __syncthreads();   // the staged rows have been read

  f32x16 dqacc[NG];
#pragma unroll
  for (int mb = 0; mb < NG; ++mb) zero(dqacc[mb]);
  for (int tile = w; tile < n_tiles; tile += W) {
    wave_order();   // the reads of the previous tile come first
    if constexpr (G > 1) kt.scatter(k_lds[w], lane, kdst);
    else kt.store(k_lds[w], lane);
    vt.store(v_lds[w], lane);
    if (tile + W < n_tiles) {
      kt.load(k_rsrc, tile + W, lane);
      vt.load(v_rsrc, tile + W, lane);
    }
    wave_order();
    f32x16 s;
    if constexpr (G == 1) {
      s = row_product<D>(&k_lds[w][lq * RS], hh, qop);
    } else {
      ChannelSum<HS> acc;
#pragma unroll
      for (int c = 0; c < D / 2; c += 4) {
        const f32x4 x = *(const f32x4*)&k_lds[w][lq * RS + hh * (D / 2) + c];
        if constexpr (G == 2) {
          acc.step(c / 2, x[0] + x[1], qop[c / 2]);
          acc.step(c / 2 + 1, x[2] + x[3], qop[c / 2 + 1]);
        } else {
          acc.step(c / 4, ((x[0] + x[1]) + x[2]) + x[3], qop[c / 4]);
        }
      }
      s = acc.sum();
    }
    const f32x16 dp = row_product<D, DpSum<D>>(&v_lds[w][lq * RS], hh, doop);
    const int n0 = tile * kTile;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(scaled_plus(s[i], scale, -lse_row) * kLog2e);
    if (n0 + kTile > Nk || (causal && n0 + kTile - 1 > r0 + shift)) {
      asm volatile("");   // (a branch: few tiles are masked)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (n0 + acc_row(i, hh) > lim) s[i] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] *= dp[i] - dl;
    if constexpr (G == 1) {
      column_product<D>(k_lds[w], lq, hh, s, dqacc);
    } else {
      // lane m owns the groups NG*m .. (of 32 * NG slots; with 16 groups the upper lanes repeat the lower)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float* src = &k_lds[w][acc_row(i, hh) * RS + (lq * NG % KRED) * G];
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) {
          float x;
          if constexpr (G == 2) {
            const f32x2 y = *(const f32x2*)(src + mb * G);
            x = y[0] + y[1];
          } else {
            const f32x4 y = *(const f32x4*)(src + mb * G);
            x = ((y[0] + y[1]) + y[2]) + y[3];
          }
          dqacc[mb] = mfma(x, s[i], dqacc[mb]);
        }
      }
    }
  }

  wave_order();
  // dQ_r (G > 1: by group; G = 1: dQ~ by channel) of the wave, then summed over the waves
  float* mine = &k_lds[w][lq * RS];
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int mb = 0; mb < NG; ++mb)
      if (KRED >= 32 || acc_row(i, hh) < KRED) mine[acc_row(i, hh) * NG + mb] = dqacc[mb][i];
  __syncthreads();
  for (int i = tid; i < kTile * KRED / 4; i += (W * 64)) {
    const int row = i / (KRED / 4), c = i % (KRED / 4) * 4;
    f32x4 x = *(const f32x4*)&k_lds[0][row * RS + c];
#pragma unroll
    for (int j = 1; j < W; ++j) x += *(const f32x4*)&k_lds[j][row * RS + c];
    *(f32x4*)&v_lds[0][row * RS + c] = x;
  }
  __syncthreads();
  for (int i = tid; i < kTile * D / 4; i += (W * 64)) {
    const int row = i / (D / 4), c = i % (D / 4) * 4;
    if (r0 + row >= N) continue;
    f32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (G > 1) {
        const int pos = map_lds[c + e] & (D - 1);
        y[e] = pos % G == 0 ? scale * v_lds[0][row * RS + pos / G] : 0.0f;
      } else if (!perm) {
        y[e] = scale * v_lds[0][row * RS + c + e];
      } else {
        // the sampled channel of a group receives the sum over its members, the others 0
        float s = 0.0f;
        if (map_lds[c + e] == c + e) {
          const int pos = (pos_lds[c + e] & (D - 1)) / group * group;
          for (int g = 0; g < group; ++g) s += v_lds[0][row * RS + order_lds[pos + g]];
        }
        y[e] = scale * s;
      }
    }
    *(f32x4*)(dq + head + (size_t)(r0 + row) * D + c) = y;
  }
}

// The same by bf16 pieces, all three products (groups of two and four at d = 64, as bwd_dkv_pieces_kernel; Q_r's and dO's pieces lie in LDS).
// 48 products and 20 for the splitting a tile instead of 64 of twice the time. B1 H8 N2048 n_groups 32: 90 -> 75 us, 16 groups 84 -> 73.
template <int D, int G, int W>
__global__ __launch_bounds__(W * 64, (D == 64 ? 2 : 1)) void bwd_dq_pieces_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ o,
    const float* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ dq, const uint8_t* __restrict__ perm,
    int H, int Hkv, int N, int Nk, int Br, int Tq, int causal, float scale) {
  constexpr int RS = Tile<D>::RS;
  constexpr int KRED = D / G, HS = KRED / 2;
  constexpr int NG = (KRED + 31) / 32;   // 32-row blocks of the dQ_r accumulator
  __shared__ __attribute__((aligned(16))) float k_lds[W][kTile * RS];   // V, then K tile of each wave; at the end its dQ_r
  __shared__ __attribute__((aligned(16))) PieceRows<KRED> q_lds;
  __shared__ __attribute__((aligned(16))) PieceRows<D> do_lds;
  __shared__ __attribute__((aligned(16))) float sum_lds[kTile * RS];
  __shared__ uint32_t mark_lds[kTile + 1];   // what is known of a row (kRowAgain ..); whether a key is beyond_pieces
  __shared__ uint8_t order_lds[D];   // sorted order of the block's channels
  __shared__ uint8_t map_lds[D];     // a channel's position in it

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const int Tw = (N + kTile - 1) / kTile;
  const int n_bh = gridDim.x / Tw;
  const int t = causal ? Tw - 1 - (int)blockIdx.x / n_bh : (int)blockIdx.x / n_bh;   // longest first
  const int bh = blockIdx.x % n_bh;
  const int b = bh / H, hk = bh % H / (H / Hkv);
  const int r0 = t * kTile, q_abs = r0 + lq;
  const int shift = Nk - N;

  const size_t head = (size_t)bh * N * D;
  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)(b * Hkv + hk) * Nk * D, (unsigned)Nk * D * 4);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)(b * Hkv + hk) * Nk * D, (unsigned)Nk * D * 4);
  const int n_end = causal ? min(Nk, r0 + kTile + shift) : Nk;
  const int n_tiles = (n_end + kTile - 1) / kTile;
  const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;   // last key this row sees

  Tile<D> kt, vt;
  auto load_first = [&]() {
    if (w < n_tiles) {
      kt.load(k_rsrc, w, lane);
      vt.load(v_rsrc, w, lane);
    }
  };
  load_first();
  if (tid <= kTile) mark_lds[tid] = 0;
  // Q, dO and O rows pass through LDS (one tile per wave 0, 1, 2)
  {
    const float* src = w == 0 ? q : w == 1 ? dout : o;
    Tile<D> x;
    if (w < 3) {
      x.load(head_rsrc(src + head, (unsigned)N * D * 4), t, lane);
      x.store(k_lds[w], lane);
    }
  }
  {
    // D is a power of two: an out-of-range entry of a caller's table cannot index past a row
    const uint8_t* pr = perm + ((size_t)bh * Tq + r0 / Br) * D;
    for (int i = tid; i < D; i += W * 64) {
      order_lds[i] = pr[i] & (D - 1);
      map_lds[pr[i] & (D - 1)] = (uint8_t)i;
    }
  }
  __syncthreads();
  float dl = 0.0f;
  int kdst[4];
#pragma unroll
  for (int c = 0; c < D / 2; ++c) dl = __builtin_fmaf(k_lds[1][lq * RS + hh * (D / 2) + c], k_lds[2][lq * RS + hh * (D / 2) + c], dl);
  for (int s = w * 8; s < HS; s += W * 8) {
    f32x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      x[e] = k_lds[0][lq * RS + order_lds[(hh * HS + s + e) * G]];
    q_lds.store(lq, hh * HS + s, split(x));
    if (beyond_pieces(largest(largest(0.0f, x.lo), x.hi))) atomicOr(&mark_lds[lq], kRowAgain);
  }
  for (int s = w * 8; s < D / 2; s += W * 8) {
    f32x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = k_lds[1][lq * RS + hh * (D / 2) + s + e] * kRaise;
    do_lds.store(lq, hh * (D / 2) + s, split(x));
  }
  dl = half_swap_sum(dl);
#pragma unroll
  for (int e = 0; e < 4; ++e) kdst[e] = map_lds[lane % (D / 4) * 4 + e] & (D - 1);
  const float lse_row = lse[(size_t)bh * N + min(q_abs, N - 1)];
  __syncthreads();   // the staged rows have been read

  // The rows of the bit mask `rows`, products by pieces or on the float instruction. By pieces, the rows to be taken again are returned;
  // a second walk takes the scores by pieces that the first took by them (beyond_pieces), and with k_again set it is for the rows, too,
  // that see a key that is not held by pieces.
  bool k_again = false;
  auto pass = [&](auto pieces, uint32_t rows) -> uint32_t {
    constexpr bool BY_PIECES = decltype(pieces)::value;
    constexpr float raise = BY_PIECES ? kRaise : 1.0f, dp_raise = raise * raise;   // of dO, V and K_f; of dP, D and dS
    const Splitter splitter(lane);
    const float raised_dl = dl * dp_raise;
    const __amdgpu_buffer_rsrc_t q_rsrc = head_rsrc(q + head, (unsigned)N * D * 4), do_rsrc = head_rsrc(dout + head, (unsigned)N * D * 4);
    uint32_t any_beyond = 0;
    f32x16 dqacc[NG];
#pragma unroll
    for (int mb = 0; mb < NG; ++mb) zero(dqacc[mb]);
    for (int tile = w; tile < n_tiles; tile += W) {
      wave_order();   // the reads of the previous tile come first
      vt.store(k_lds[w], lane);
      wave_order();
      float x[D / 2];
#pragma unroll
      for (int c = 0; c < D / 2; c += 4) {
        const f32x4 y = *(const f32x4*)&k_lds[w][lq * RS + hh * (D / 2) + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[c + e] = y[e] * raise;
      }
      wave_order();
      kt.scatter(k_lds[w], lane, kdst);
      if (tile + W < n_tiles) {
        kt.load(k_rsrc, tile + W, lane);
        vt.load(v_rsrc, tile + W, lane);
      }
      wave_order();
      f32x16 dp;
      if constexpr (BY_PIECES) {
        zero(dp);
        split_steps<D / 2>(splitter, x, [&](int s, const Pieces& p) { dp = mfma(p, do_lds.load(lq, hh * (D / 2) + 8 * s), dp); });
      } else {
        OneChain acc;
#pragma unroll
        for (int c = 0; c < D / 2; c += 4) {
          const f32x4 y = Q4::values(Q4::load(do_rsrc, (lq * D + hh * (D / 2) + c) * 4, r0 * (D * 4)));
#pragma unroll
          for (int e = 0; e < 4; ++e) acc.step(c + e, x[c + e], y[e]);
        }
        dp = acc.sum();
      }
      float y[HS];
#pragma unroll
      for (int c = 0; c < D / 2; c += 4) {
        const f32x4 x = *(const f32x4*)&k_lds[w][lq * RS + hh * (D / 2) + c];
        if constexpr (G == 2) {
          y[c / 2] = x[0] + x[1];
          y[c / 2 + 1] = x[2] + x[3];
        } else {
          y[c / 4] = ((x[0] + x[1]) + x[2]) + x[3];
        }
      }
      const uint32_t k_beyond = rows_of(beyond_pieces(largest(y)));
      any_beyond |= k_beyond;
      f32x16 s;
      {
        PieceSum acc;
        split_steps<HS>(splitter, y, [&](int s, const Pieces& p) { acc.step(p, q_lds.load(lq, hh * HS + 8 * s)); });
        s = acc.sum();
      }
      if constexpr (!BY_PIECES) {
        float qop[HS];
#pragma unroll
        for (int c = 0; c < HS; ++c)
          qop[c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(q_rsrc, (lq * D + order_lds[(hh * HS + c) * G]) * 4, r0 * (D * 4), 0));
        const uint32_t q_beyond = rows_of(beyond_pieces(largest(qop)));
        if (k_beyond != 0 && tile * kTile + __builtin_ctz(k_beyond) <= lim) atomicOr(&mark_lds[lq], kRowBeyond);
        if ((q_beyond | k_beyond) != 0) {
          ChannelSum<HS> acc;
#pragma unroll
          for (int c = 0; c < HS; ++c) acc.step(c, y[c], qop[c]);
          const f32x16 z = acc.sum();
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = ((q_beyond >> lq | k_beyond >> acc_row(i, hh)) & 1) != 0 ? z[i] : s[i];
        }
      }
      const int n0 = tile * kTile;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(scaled_plus(s[i], scale, -lse_row) * kLog2e);
      if (n0 + kTile > Nk || (causal && n0 + kTile - 1 > r0 + shift)) {
        asm volatile("");   // (a branch: few tiles are masked)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (n0 + acc_row(i, hh) > lim) s[i] = 0.0f;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] *= dp[i] - raised_dl;
      // lane m owns the columns NG*m .. (of 32 * NG slots; with 16 groups the upper lanes repeat the lower)
      f32x16 kc[NG];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float* src = &k_lds[w][acc_row(i, hh) * RS + (lq * NG % KRED) * G];
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) {
          if constexpr (G == 2) {
            const f32x2 y = *(const f32x2*)(src + mb * G);
            kc[mb][i] = (y[0] + y[1]) * raise;
          } else {
            const f32x4 y = *(const f32x4*)(src + mb * G);
            kc[mb][i] = (((y[0] + y[1]) + y[2]) + y[3]) * raise;
          }
        }
      }
      if constexpr (BY_PIECES) {
        Pieces s0, s1, k0, k1;
        splitter(s, s0, s1);
#pragma unroll
        for (int mb = 0; mb < NG; ++mb) {
          splitter(kc[mb], k0, k1);
          dqacc[mb] = mfma(k0, s0, dqacc[mb]);
          dqacc[mb] = mfma(k1, s1, dqacc[mb]);
        }
      } else {
#pragma unroll
        for (int mb = 0; mb < NG; ++mb)
#pragma unroll
          for (int i = 0; i < 16; ++i) dqacc[mb] = mfma(kc[mb][i], s[i], dqacc[mb]);
      }
    }

    wave_order();
    // dQ_r of the wave, then summed over the waves
    float* mine = &k_lds[w][lq * RS];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int mb = 0; mb < NG; ++mb)
        if (KRED >= 32 || acc_row(i, hh) < KRED) mine[acc_row(i, hh) * NG + mb] = dqacc[mb][i];
    __syncthreads();
    for (int i = tid; i < kTile * KRED / 4; i += W * 64) {
      const int row = i / (KRED / 4), c = i % (KRED / 4) * 4;
      f32x4 x = *(const f32x4*)&k_lds[0][row * RS + c];
#pragma unroll
      for (int j = 1; j < W; ++j) x += *(const f32x4*)&k_lds[j][row * RS + c];
      *(f32x4*)&sum_lds[row * RS + c] = x * (1.0f / (dp_raise * raise));
      if (BY_PIECES && r0 + row < N && !all_finite(x)) atomicOr(&mark_lds[row], kRowAgain);
    }
    __syncthreads();
    for (int i = tid; i < kTile * D / 4; i += W * 64) {
      const int row = i / (D / 4), c = i % (D / 4) * 4;
      if (r0 + row >= N || !((rows >> row & 1) != 0 || (!BY_PIECES && (mark_lds[row] & kRowBeyond) != 0))) continue;
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pos = map_lds[c + e] & (D - 1);
        y[e] = pos % G == 0 ? scale * sum_lds[row * RS + pos / G] : 0.0f;
      }
      *(f32x4*)(dq + head + (size_t)(r0 + row) * D + c) = y;
    }
    if constexpr (!BY_PIECES) return 0;
    if (any_beyond != 0) atomicOr(&mark_lds[kTile], 1u);
    __syncthreads();
    k_again = mark_lds[kTile] != 0;
    return rows_of((mark_lds[lq] & kRowAgain) != 0);
  };
  const uint32_t again = pass(std::true_type(), ~0u);
  if (again == 0 && !k_again) return;
  load_first();
  pass(std::false_type(), again);
}

template <int D>
hipError_t launch_d(const float* q, const float* k, const float* v, const float* o, const float* dout, const float* lse,
                    float* dq, float* dk, float* dv, const uint8_t* perm, const Problem& pb, int distr, hipStream_t stream) {
  const int Tq = (pb.N + pb.Br - 1) / pb.Br;
  const size_t rows = (size_t)pb.B * pb.H * pb.N;
  const long long q_units = (long long)pb.B * pb.H * ((pb.N + kTile - 1) / kTile);
  const long long k_units = (long long)pb.B * pb.Hkv * ((pb.Nk + kTile - 1) / kTile);
  const size_t d_units = (rows * (D / 4) + kThreads - 1) / kThreads;
  if (q_units > 0x7fffffffLL || k_units > 0x7fffffffLL || d_units > 0x7fffffffULL) return hipErrorInvalidValue;
  const uint8_t* table = distr ? perm : nullptr;
  const int n_groups = distr ? pb.n_groups : D;
  float* delta = dq;   // one float per row: dq is overwritten after its last use
  hipLaunchKernelGGL((bwd_delta_kernel<D>), dim3((unsigned)d_units), dim3(kThreads), 0, stream, o, dout, delta, rows);
#define DA_DKV(W, GG)                                                                                                      \
  hipLaunchKernelGGL((bwd_dkv_kernel<D, W, GG>), dim3((unsigned)k_units), dim3(W * 64), 0, stream, q, k, v, dout, lse, delta, dk, dv, \
                     table, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq, n_groups, pb.causal, pb.scale)
  const bool eight = D == 64 && (long long)(pb.H / pb.Hkv) * ((pb.N + kTile - 1) / kTile) >= 8;
  const int G = D / n_groups;
  const bool pieces = distr && float_by_pieces(pb);
  if constexpr (D == 64) {
#define DA_DKVP(W, GG)                                                                                                      \
  hipLaunchKernelGGL((bwd_dkv_pieces_kernel<D, W, GG>), dim3((unsigned)k_units), dim3(W * 64), 0, stream, q, k, v, dout, lse, delta, dk, dv, \
                     table, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq, pb.causal, pb.scale)
    if (pieces && eight && G == 2) DA_DKVP(8, 2);
    else if (pieces && eight) DA_DKVP(8, 4);
    else if (pieces && G == 2) DA_DKVP(4, 2);
    else if (pieces) DA_DKVP(4, 4);
    else if (eight && G == 2) DA_DKV(8, 2);
    else if (eight && G == 4) DA_DKV(8, 4);
    else if (eight) DA_DKV(8, 1);
#undef DA_DKVP
  }
  if (pieces || eight) {
  } else if (G == 2) {
    DA_DKV(4, 2);
  } else if (G == 4) {
    DA_DKV(4, 4);
  } else {
    DA_DKV(4, 1);
  }
#undef DA_DKV
  // dQ: eight waves as in the forward (launch_waves in attn_f32.hip)
  const bool wide = D == 64 && q_units <= kComputeUnits && (pb.Nk + kTile - 1) / kTile > 8;
  if constexpr (D == 64) {
    if (pieces) {
#define DA_DQ(GG, W)                                                                                                       \
  hipLaunchKernelGGL((bwd_dq_pieces_kernel<D, GG, W>), dim3((unsigned)q_units), dim3(W * 64), 0, stream, q, k, v, o, dout, lse, dq, \
                     table, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq, pb.causal, pb.scale)
      if (wide && G == 2) DA_DQ(2, 8);
      else if (wide) DA_DQ(4, 8);
      else if (G == 2) DA_DQ(2, 4);
      else DA_DQ(4, 4);
#undef DA_DQ
      return hipGetLastError();
    }
  }
#define DA_DQ(GG, W)                                                                                                       \
  hipLaunchKernelGGL((bwd_dq_kernel<D, GG, W>), dim3((unsigned)q_units), dim3(W * 64), 0, stream, q, k, v, o, dout, lse, dq, \
                     table, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq, n_groups, pb.causal, pb.scale)
  if constexpr (D == 64) {
    if (wide) DA_DQ(1, 8);   // (groups of two and four take the pieces where it is wide)
  }
  if (wide) {
  } else if (G == 2) {
    DA_DQ(2, 4);
  } else if (G == 4) {
    DA_DQ(4, 4);
  } else {
    DA_DQ(1, 4);
  }
#undef DA_DQ
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32_bwd(const void* q, const void* k, const void* v, const void* o, const void* dout,
                               const float* lse, void* dq, void* dk, void* dv, const uint8_t* perm,
                               const Problem& pb, int distr, hipStream_t stream) {
  if (pb.d == 64)
    return launch_d<64>((const float*)q, (const float*)k, (const float*)v, (const float*)o, (const float*)dout, lse, (float*)dq,
                        (float*)dk, (float*)dv, perm, pb, distr, stream);
  if (pb.d == 128)
    return launch_d<128>((const float*)q, (const float*)k, (const float*)v, (const float*)o, (const float*)dout, lse, (float*)dq,
                         (float*)dk, (float*)dv, perm, pb, distr, stream);
  return hipErrorInvalidValue;
}

}  // namespace da
