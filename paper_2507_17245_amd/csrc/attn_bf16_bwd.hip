// Backward of the attention forward (exact and DistrAttention) for bf16 tensors on the gfx950
// matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate). Two kernels (and a reduction when the
// dK/dV launch is split over query heads), no atomics (results do not depend on the run).
//
// The paper trains through the approximation (Sec. 4.3, 4.4) and gives no gradient; computed here
// is the derivative of the forward with every Q block's grouping held fixed. With Q_r the sampled
// and K_f the fused columns of Sec. 3.2 (Eq. 2: S^ = Q_r K_f^T, one grouping per Q block,
// Sec. 3.3), write Q~ for Q with every channel replaced by its group's sampled channel:
//   S^ = Q_r K_f^T = Q~ K^T                       (a sum over groups of sums over members)
//   dK = scale * dS^T Q~                          (every member of a group receives dK_f's column)
//   dQ[:, sampled channel of group j] = scale * sum over the group's members c of (dS K)[:, c]
// so the backward of DistrAttention is the backward of exact attention taken on Q~, followed by a
// sum over each group's members for dQ. P = exp(S^ - lse) is rebuilt from the forward's row
// statistics, dP = dO V^T, D_i = sum_c dO_ic O_ic, dS = P o (dP - D), dV = P^T dO.
//
//   bwd_dq_kernel       one workgroup per 128 query rows, lane = query row; K and V tiles of 64
//                       rows stream through LDS:  S^T = K Q~^T, dP^T = V dO^T, dQ~^T += K^T dS^T.
//                       Takes -D_i, lse * log2(e) and Q~ (DistrAttention only) of its rows on the way
//                       and leaves them in scratch for the next kernel (a kernel of its own for it read Q, dO
//                       and O once more: backward H16 N1024 d64 52 -> 48 us, d128 90 -> 79, H32 Hkv8 N4096 d64 292 -> 287)
//   bwd_dkv_kernel      one workgroup per 128 keys of a kv head, lane = key; Q~ and dO tiles of 64
//                       rows of every query head of the group stream through LDS:
//                       S = Q~ K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q~^T dS
//   bwd_reduce_kernel   sums the float partial dK, dV of a head-split dK/dV launch
//   bwd_short_kernel    short sequences at d = 64: all of it in one workgroup per head, one launch
// In both, the accumulator layout of the first products (registers = streamed rows, lanes =
// resident rows) is the B-operand layout of the last ones, so P and dS never leave registers; the
// streamed tiles are read once row-wise (16-byte reads) and once with transposing reads. Tiles are
// double-buffered in LDS and loaded one iteration ahead (one barrier per tile).
#include <type_traits>

#include "da_common.h"

namespace da {

namespace {

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kBwdRows = 128;      // resident rows per workgroup (4 waves x 32)
constexpr int kBwdStream = 64;     // streamed rows per LDS tile
constexpr int kBwdThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Position of a 16-byte chunk inside its row of a streamed tile (rows of D bf16, unpadded). A
// tile is read two ways: 16 lanes take the same chunk of 16 consecutive rows (16-byte reads), and
// the transposing reads take, per 32 lanes, 64 consecutive bytes of 4 consecutive rows. Both are
// free of bank conflicts when the chunk index is XORed with these bits of the row.
template <int D>
__device__ inline int chunk_swz(int row) {
  if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
  else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

template <int D>
__device__ inline char* chunk_addr(char* tile, int row, int chunk) {
  return tile + row * (D * 2) + ((chunk ^ chunk_swz<D>(row)) << 4);
}

// Streamed tiles reach LDS by direct global->LDS loads (buffer_load ... lds: each wave-level load
// drops 64 x 16 bytes contiguously): wave-level load j of wave w fills the 1 KB block 4*j + w of
// the tile; the lane that owns a 16-byte position fetches the global chunk the swizzle assigns to
// it. The source is a buffer descriptor over one head, whose range check makes rows past the end
// read as zeros.
typedef __attribute__((address_space(3))) void lds_void;
template <int D>
struct TileLoader {
  static constexpr int CH = D / 8, ROWB = D * 2, TILE = kBwdStream * ROWB;
  static constexpr int CPT = TILE / 1024 / (kBwdThreads / 64);
  int voff[CPT];
  int wave;
  __device__ TileLoader(int wave_, int lane) : wave(wave_) {
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int slot = (j * (kBwdThreads / 64) + wave) * 64 + lane;
      const int row = slot / CH, pc = slot % CH;
      voff[j] = row * ROWB + ((pc ^ chunk_swz<D>(row)) << 4);
    }
  }
  __device__ void load(__amdgpu_buffer_rsrc_t rsrc, int row0, char* dst) const {
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + (j * (kBwdThreads / 64) + wave) * 1024), 16,
                                               voff[j], row0 * ROWB, 0, 0);
  }
};
__device__ inline __amdgpu_buffer_rsrc_t head_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}
__device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Per-lane byte offsets of the MFMA A operands inside a streamed tile (the swizzle depends on the
// low four bits of the row only, so a 32-row block or a 16-row step adds a multiple of the row
// length).
//  rows[s]:   row-wise operand of contraction step s: the 16-byte chunk 2*s + hh of tile row
//             lane%32 (contraction slots 8*hh .. 8*hh+7 of the step).
//  tr[cb][.]: operand of a product that contracts over the tile's rows (the tile transposed):
//             output rows are the channels 32*cb + lane%32, the contraction runs over 16 tile rows
//             in the order an accumulator enumerates them (slot j of lane half hh = row
//             8*(j/4) + 4*hh + j%4), read by two ds_read_b64_tr_b16 (within 16 lanes, lane i
//             receives element i%4 of the 8-byte pieces addressed by lanes 4j + i/4, j = 0..3):
//             this lane addresses rows 4*hh + (lane%16)/4 and that + 8.
template <int D>
struct OperandOffsets {
  int rows[D / 16];
  int tr[D / 32][2];
  __device__ OperandOffsets(int lane) {
    const int lq = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) rows[s] = (int)(chunk_addr<D>(nullptr, lq, 2 * s + hh) - (char*)nullptr);
    const int row = 4 * hh + ((lane & 15) >> 2);
    const int inb = 8 * (lane & 1);
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb) {
      const int chunk = 4 * cb + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
      tr[cb][0] = (int)(chunk_addr<D>(nullptr, row, chunk) - (char*)nullptr) + inb;
      tr[cb][1] = (int)(chunk_addr<D>(nullptr, row + 8, chunk) - (char*)nullptr) + inb;
    }
  }
};

// all row-wise operands of the 32-row block `blk` of a tile
template <int D>
__device__ inline void read_rows(const char* tile, int blk, const OperandOffsets<D>& off, bf16x8 (&a)[D / 16]) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s) a[s] = *(const bf16x8*)(tile + blk * 32 * (D * 2) + off.rows[s]);
}

// all transposed operands of the 32-row block `blk`: [channel block][16-row step]
template <int D>
__device__ inline void read_transposed(const char* tile, int blk, const OperandOffsets<D>& off,
                                       bf16x8 (&a)[D / 32][2]) {
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const char* base = tile + (blk * 32 + tt * 16) * (D * 2);
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + off.tr[cb][0]));
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + off.tr[cb][1]));
      s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      a[cb][tt] = __builtin_bit_cast(bf16x8, r);
    }
}

// Which (head, tile) a workgroup takes: `tile` counts from the longest causal tile on. Consecutive
// workgroup ids go round-robin over the 8 XCDs.
//   kHeadMajor     every XCD walks a contiguous range of units: the tiles of a head share its L2.
//   kLongestFirst  (causal, at most kBalancedUnits) tile by tile over all heads. Causal tiles differ up to
//                  Tw-fold in length; with (nearly) all of them resident at once, head after head leaves compute
//                  units with only long or only short ones. A head still stays on one XCD when the head count
//                  is a multiple of 8.
//   kPaired        the same with the second round reversed (paired_tile), where two workgroups share a compute unit: not for
//                  dK/dV at d = 128, which fills one (H16 N4096 270 us, 289 reversed). Backward, longest first | this: d64 H32
//                  N2048 93.5 | 88.9 us, H16 N4096 162 | 151, H32 Hkv8 N4096 274 | 266; d128 H16 N2048 132 | 127.
enum UnitOrder { kHeadMajor, kLongestFirst, kPaired };
constexpr int kBalancedUnits = 8 * kComputeUnits;
__device__ inline void unit_of(int id, int units, int Tw, int order, int& head, int& tile) {
  if (order != kHeadMajor) {
    const int heads = units / Tw;
    tile = order == kPaired ? paired_tile(id / heads, heads, Tw) : id / heads;
    head = id % heads;
  } else {
    if ((units & 7) == 0) id = (id & 7) * (units >> 3) + (id >> 3);
    head = id / Tw;
    tile = id % Tw;
  }
}

// nothing moves across: operand reads issued before it stay ahead of the MFMAs behind it
__device__ inline void fence() { __builtin_amdgcn_sched_barrier(0); }

// tile row that register i of a 32 x 32 accumulator block holds, for lane half hh
__device__ inline int acc_row(int i, int hh) { return 8 * (i >> 2) + 4 * hh + (i & 3); }

__device__ inline void zero(f32x16& x) {
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = 0.0f;
}

}  // namespace

// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kBwdThreads, 2) void bwd_dq_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, const bf16* __restrict__ o,
    const bf16* __restrict__ dout, const float* __restrict__ lse, bf16* __restrict__ qrep, float* __restrict__ lse2p,
    float* __restrict__ delta, bf16* __restrict__ dq, const uint8_t* __restrict__ perm, int H, int Hkv, int N, int Nk, int Br, int Tq,
    int Tw, int n_groups, int causal, int order, float scale) {
  constexpr int CH = D / 8;
  constexpr int KS = D / 16;    // MFMA steps over the channels
  constexpr int CB = D / 32;    // 32-channel blocks of the dQ~ accumulator
  constexpr int TILE = kBwdStream * D * 2;
  // separate objects: the compiler then does not make reads of one buffer wait for loads in
  // flight into another
  __shared__ __attribute__((aligned(1024))) char k_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) char k_lds1[TILE];
  __shared__ __attribute__((aligned(1024))) char v_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) char v_lds1[TILE];
  __shared__ uint8_t perm_lds[kBwdRows / 32][D];
  __shared__ uint8_t group_lds[kBwdRows / 32][D];   // group whose sampled channel c is, else 255
  __shared__ __attribute__((aligned(8))) uint8_t from_lds[kBwdRows / 32][D];   // byte offset in a row of a channel's sampled one

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lq = lane & 31, hh = lane >> 5;
  int head, t;
  unit_of((int)blockIdx.x, (int)gridDim.x, Tw, order, head, t);
  if (causal) t = Tw - 1 - t;   // the blocks with the most keys first
  const size_t bh = head;
  const int b = (int)(bh / H), h = (int)(bh % H);
  const int hk = h / (H / Hkv);
  const int r0 = t * kBwdRows;
  const int rows = min(kBwdRows, N - r0);
  const int q_abs = r0 + 32 * w + lq;
  const bool active = q_abs < N;
  const int shift = Nk - N;
  const float sl2e = scale * kLog2e;

  const unsigned head_bytes = (unsigned)Nk * D * 2;
  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)(b * Hkv + hk) * Nk * D, head_bytes);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)(b * Hkv + hk) * Nk * D, head_bytes);
  const TileLoader<D> loader(w, lane);
  const int n_end = causal ? min(Nk, r0 + rows + shift) : Nk;
  const int n_tiles = ((n_end + kBwdStream - 1) / kBwdStream + 1) & ~1;   // even
  // tiles that end at or before n_free need no mask for any row of the workgroup
  const int n_free = causal ? min(r0 + shift + 1, Nk) : Nk;
  loader.load(k_rsrc, 0, k_lds0);
  loader.load(v_rsrc, 0, v_lds0);

  const size_t row_off = (bh * N + (active ? q_abs : r0)) * D;
  bf16x8 qop[KS], doop[KS];
  // The wave's rows of Q and its table entries, asked for ahead of dO and O (used below).
  constexpr int QU = 32 * CH / 64, PU = D / 64;
  const int G = D / n_groups;
  u32x4 qx[QU];
  int entry[PU], first[PU];
  if (perm) {
    const int blk = min((r0 + 32 * w) / Br, Tq - 1);   // a wave's 32 rows lie in one Q block (Br is a multiple of 32)
    const uint8_t* pr = perm + (bh * Tq + blk) * D;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      entry[u] = pr[u * 64 + lane] & (D - 1);
      first[u] = pr[(u * 64 + lane) / G * G] & (D - 1);
    }
#pragma unroll
    for (int j = 0; j < QU; ++j) {
      const int row = min(r0 + 32 * w + (j * 64 + lane) / CH, N - 1);   // (a row past the end is never stored)
      qx[j] = *(const u32x4*)(q + (bh * N + row) * D + lane % CH * 8);
    }
    fence();
  }
  float dl = 0.0f;   // -D: dP^T accumulates from there on (the products' addend, in 16 registers: no subtraction per score)
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u}, z = {0u, 0u, 0u, 0u};
    if (active) {
      if (!perm) x = *(const u32x4*)(q + row_off + (2 * s + hh) * 8);
      y = *(const u32x4*)(dout + row_off + (2 * s + hh) * 8);
      z = *(const u32x4*)(o + row_off + (2 * s + hh) * 8);
    }
    qop[s] = __builtin_bit_cast(bf16x8, x);
    doop[s] = __builtin_bit_cast(bf16x8, y);
    const bf16x8 ov = __builtin_bit_cast(bf16x8, z);
#pragma unroll
    for (int j = 0; j < 8; ++j) dl = __builtin_fmaf((float)doop[s][j], -(float)ov[j], dl);
  }
  dl = half_swap_sum(dl);
  const float lse2 = active ? lse[bh * N + q_abs] * kLog2e : 0.0f;
  if (active && hh == 0) {
    lse2p[bh * N + q_abs] = lse2;
    delta[bh * N + q_abs] = dl;
  }
  if (perm) {
    // Q~: channel c of a row takes the value of the first channel (sorted order) of c's group in the row's Q block. The
    // wave's rows pass through its quarter of the tile buffers that stay free until the loop (16-byte chunks exchanged
    // by the row); its LDS accesses take effect in its order.
    char* rows_lds = (w & 2 ? v_lds1 : k_lds1) + (w & 1) * (32 * D * 2);
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      perm_lds[w][u * 64 + lane] = (uint8_t)entry[u];
      from_lds[w][entry[u]] = (uint8_t)(2 * first[u]);
    }
    auto swz = [](int row) { return D == 64 ? (row >> 1) & 7 : row & 15; };
#pragma unroll
    for (int j = 0; j < QU; ++j) {
      const int row = (j * 64 + lane) / CH, chunk = lane % CH;
      *(u32x4*)(rows_lds + row * (D * 2) + ((chunk ^ swz(row)) << 4)) = qx[j];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t flip = swz(lq) * 0x10101010u;       // chunk ^ x is offset ^ 16 x, for four channels at once
    const char* row = rows_lds + lq * (D * 2);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x2 f = *(const u32x2*)&from_lds[w][16 * s + 8 * hh];
      const uint32_t at[2] = {(f[0] & 0xfefefefeu) ^ flip, (f[1] & 0xfefefefeu) ^ flip};
#pragma unroll
      for (int j = 0; j < 8; ++j) qop[s][j] = *(const bf16*)(row + ((at[j >> 2] >> (8 * (j & 3))) & (2 * D - 1)));
      if (active) *(bf16x8*)(qrep + row_off + (2 * s + hh) * 8) = qop[s];
    }
  }
  f32x16 neg_d;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_d[i] = dl;
  const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;   // last key this row sees

  f32x16 dqacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) zero(dqacc[cb]);

  const OperandOffsets<D> off(lane);
  // dS^T of one 32-key block as B operands
  auto ds_operands = [&](const f32x16& sacc, const f32x16& dpacc, int kv0, auto masked_c, bf16x8 (&dsop)[2]) {
    float pv[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) pv[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], sl2e, -lse2));
    if constexpr (decltype(masked_c)::value) {
#pragma unroll
      for (int i = 0; i < 16; ++i) pv[i] = kv0 + acc_row(i, hh) <= lim ? pv[i] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) dsop[i >> 3][i & 7] = (bf16)(pv[i] * dpacc[i]);
  };
  auto dq_update = [&](const bf16x8 (&at)[CB][2], const bf16x8 (&dsop)[2]) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) dqacc[cb] = mfma(at[cb][tt], dsop[tt], dqacc[cb]);
  };

  // One tile; the loop is unrolled by two so that every buffer is a fixed object in each copy
  // (the compiler then knows that the loads in flight do not touch the tile being read). Tiles
  // that need the mask take a copy of the body of their own.
  auto tile_step = [&](auto par_c, auto masked, int n0) __attribute__((always_inline)) {
    constexpr int par = decltype(par_c)::value;
    const char* k_lds = par ? k_lds1 : k_lds0;
    const char* v_lds = par ? v_lds1 : v_lds0;
    wait_loads();
    __syncthreads();   // this tile has landed; the other buffers' readers are done
    if (n0 + kBwdStream < n_tiles * kBwdStream) {
      loader.load(k_rsrc, n0 + kBwdStream, par ? k_lds0 : k_lds1);
      loader.load(v_rsrc, n0 + kBwdStream, par ? v_lds0 : v_lds1);
    }
    // Two waves share a SIMD (a single wave cannot fill it: its LDS reads alone take as many
    // issue cycles as its MFMAs take pipe cycles), so the blocks follow one another and operands
    // are read in batches of HB contraction steps in front of their MFMAs (all of them at d = 64;
    // at d = 128 two batches: with the 96 accumulator registers the whole set does not fit beside
    // the resident operands).
    constexpr int HB = D == 128 ? KS / 2 : KS;
#pragma unroll
    for (int mb = 0; mb < kBwdStream / 32; ++mb) {
      bf16x8 ak[HB], av[HB], at[CB][2], ds[2];
      f32x16 sacc, dpacc;
      zero(sacc);
      dpacc = neg_d;
#pragma unroll
      for (int h0 = 0; h0 < KS; h0 += HB) {
#pragma unroll
        for (int s = 0; s < HB; ++s) {
          ak[s] = *(const bf16x8*)(k_lds + mb * 32 * (D * 2) + off.rows[h0 + s]);
          av[s] = *(const bf16x8*)(v_lds + mb * 32 * (D * 2) + off.rows[h0 + s]);
        }
        fence();
#pragma unroll
        for (int s = 0; s < HB; ++s) {
          sacc = mfma(ak[s], qop[h0 + s], sacc);
          dpacc = mfma(av[s], doop[h0 + s], dpacc);
        }
        fence();
      }
      ds_operands(sacc, dpacc, n0 + 32 * mb, masked, ds);
      read_transposed<D>(k_lds, mb, off, at);
      fence();
      dq_update(at, ds);
      fence();
    }
  };
  // Tiles [a, b), b - a even, with or without the mask; buffer parity = tile parity. The loop is
  // unrolled by two over fixed buffers; masked and unmasked tiles run in loops of their own (both
  // copies under a branch inside one loop cost 200 spilled registers). The tile count is rounded
  // up to an even number: a tile past the last visible key is masked out entirely.
  auto run = [&](int a, int b, auto masked_c) {
    for (int t = a; t < b; t += 2) {
      tile_step(std::integral_constant<int, 0>(), masked_c, t * kBwdStream);
      tile_step(std::integral_constant<int, 1>(), masked_c, (t + 1) * kBwdStream);
    }
  };
  const int free_tiles = min(n_free / kBwdStream, n_tiles) & ~1;
  run(0, free_tiles, std::false_type());
  run(free_tiles, n_tiles, std::true_type());

  // Epilogue: every wave puts the dQ~ of its 32 rows into LDS (float; the column index XORed
  // with the row so that a register's 32 rows fall into different banks) and sums, for every
  // group of its rows' Q block, the members' columns into the sampled channel; the other channels
  // get 0.
  __syncthreads();   // all waves are done with the tiles
  float* stage = (float*)(w == 0 ? k_lds0 : w == 1 ? k_lds1 : w == 2 ? v_lds0 : v_lds1);
  static_assert(32 * D * 4 <= TILE, "a wave's staging fits one tile buffer");
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) stage[lq * D + ((32 * cb + acc_row(i, hh)) ^ lq)] = dqacc[cb][i];
  for (int i = lane; i < D; i += 64) {
    if (!perm) perm_lds[w][i] = (uint8_t)i;
    group_lds[w][i] = 255;
  }
  __syncthreads();
  for (int j = lane; j < n_groups; j += 64) group_lds[w][perm_lds[w][j * G]] = (uint8_t)j;
  __syncthreads();
  for (int id = lane; id < 32 * CH; id += 64) {
    const int lr = id / CH, chunk = id % CH;
    const int row = r0 + 32 * w + lr;
    if (row >= N) continue;
    bf16x8 y;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = group_lds[w][chunk * 8 + e];
      float s = 0.0f;
      if (j != 255)
        for (int m = 0; m < G; ++m) s += stage[lr * D + (perm_lds[w][j * G + m] ^ lr)];
      y[e] = (bf16)(scale * s);
    }
    *(bf16x8*)(dq + (bh * N + row) * D + chunk * 8) = y;
  }
}

// What the dK/dV kernel streams: iteration `it` brings rows i_start + 64 * (it % tiles) .. of
// query head bh0 + it / tiles (Q~, dO, and the rows' statistics) into the given buffers.
template <int D>
struct QueryStream {
  const bf16 *qrep, *dout;
  const float *lse2, *delta;
  size_t bh0;   // b * H + first query head of the kv head
  int N, i_start, tiles, wave, lane;
  TileLoader<D> loader;
  __device__ void issue(int it, char* q_dst, char* do_dst, float* lse_dst, float* dl_dst) const {
    const size_t bh = bh0 + it / tiles;
    const int i0 = i_start + kBwdStream * (it % tiles);
    const unsigned head_bytes = (unsigned)N * D * 2;
    loader.load(head_rsrc(qrep + bh * N * D, head_bytes), i0, q_dst);
    loader.load(head_rsrc(dout + bh * N * D, head_bytes), i0, do_dst);
    if (wave == 0)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(head_rsrc(lse2 + bh * N, (unsigned)N * 4), (lds_void*)lse_dst, 4,
                                               lane * 4, i0 * 4, 0, 0);
    if (wave == 1)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(head_rsrc(delta + bh * N, (unsigned)N * 4), (lds_void*)dl_dst, 4,
                                               lane * 4, i0 * 4, 0, 0);
  }
};

// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kBwdThreads, (D == 64 ? 2 : 1)) void bwd_dkv_kernel(
    const bf16* __restrict__ qrep, const bf16* __restrict__ k, const bf16* __restrict__ v,
    const bf16* __restrict__ dout, const float* __restrict__ lse2p, const float* __restrict__ delta,
    bf16* __restrict__ dk, bf16* __restrict__ dv, float* __restrict__ part, int hsplit, int H, int Hkv, int N,
    int Nk, int Tw, int causal, int order, float scale) {
  constexpr int KS = D / 16;
  constexpr int CB = D / 32;
  constexpr int TILE = kBwdStream * D * 2;
  __shared__ __attribute__((aligned(1024))) char q_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) char q_lds1[TILE];
  __shared__ __attribute__((aligned(1024))) char do_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) char do_lds1[TILE];
  __shared__ __attribute__((aligned(256))) float lse_lds0[kBwdStream];   // lse * log2(e)
  __shared__ __attribute__((aligned(256))) float lse_lds1[kBwdStream];
  __shared__ __attribute__((aligned(256))) float dl_lds0[kBwdStream];
  __shared__ __attribute__((aligned(256))) float dl_lds1[kBwdStream];

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lq = lane & 31, hh = lane >> 5;
  // hsplit > 1: the query heads of the kv head are dealt out to hsplit workgroups, which leave
  // float partial sums in `part` for the reduction kernel
  int head, t;   // (kv head, share of its query heads); causal: the first keys are seen by the most rows
  unit_of((int)blockIdx.x, (int)gridDim.x, Tw, order, head, t);
  const int hs = head % hsplit;
  const size_t bk = head / hsplit;              // b * Hkv + hk
  const int b = (int)(bk / Hkv), hk = (int)(bk % Hkv);
  const int rep = H / Hkv / hsplit;             // query heads of this workgroup
  const int n0 = t * kBwdRows;
  const int key = n0 + 32 * w + lq;
  const bool valid = key < Nk;
  const int shift = Nk - N;
  const float sl2e = scale * kLog2e;

  // causal: query i sees key n iff n <= i + shift; the first tile with a row that sees key n0
  const int i_start = causal ? max(0, n0 - shift) / kBwdStream * kBwdStream : 0;
  const int tiles = ((N - i_start + kBwdStream - 1) / kBwdStream + 1) & ~1;   // per query head, even
  // the rows that see this lane's key: see_from .. see_from + see_rows - 1
  const int see_from = causal ? key - shift : 0;
  const unsigned see_rows = valid && see_from < N ? (unsigned)(N - see_from) : 0u;
  const int n_it = rep * tiles;
  const TileLoader<D> loader(w, lane);
  const QueryStream<D> ctx = {qrep, dout, lse2p, delta, (size_t)b * H + (hk * hsplit + hs) * rep, N, i_start, tiles, w, lane, loader};
  ctx.issue(0, q_lds0, do_lds0, lse_lds0, dl_lds0);

  bf16x8 kop[KS], vop[KS];
  {
    const size_t row_off = (bk * Nk + (valid ? key : n0)) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
      if (valid) {
        x = *(const u32x4*)(k + row_off + (2 * s + hh) * 8);
        y = *(const u32x4*)(v + row_off + (2 * s + hh) * 8);
      }
      kop[s] = __builtin_bit_cast(bf16x8, x);
      vop[s] = __builtin_bit_cast(bf16x8, y);
    }
  }
  f32x16 dkacc[CB], dvacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    zero(dkacc[cb]);
    zero(dvacc[cb]);
  }

  const OperandOffsets<D> off(lane);
  // One tile; the loop is unrolled by two so that every buffer is a fixed object in each copy
  // (the compiler then knows that the loads in flight do not touch the tile being read).
  auto tile_step = [&](auto par_c, auto masked_c, int it) __attribute__((always_inline)) {
    constexpr int par = decltype(par_c)::value;
    const char* q_lds = par ? q_lds1 : q_lds0;
    const char* do_lds = par ? do_lds1 : do_lds0;
    const float* lse_lds = par ? lse_lds1 : lse_lds0;
    const float* dl_lds = par ? dl_lds1 : dl_lds0;
    const int i0 = i_start + kBwdStream * (it % tiles);
    // Register classes, stated once per tile: the accumulators of dK and dV and the resident K and V
    // operands live in the accumulator half of the register file, the operands read from LDS in the vector
    // half (left to itself the allocator moved 128 accumulator registers back and forth per tile).
    if constexpr (D == 128) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+a"(dkacc[cb]), "+a"(dvacc[cb]));
#pragma unroll
      for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(kop[s]), "+a"(vop[s]));
    }
    wait_loads();
    __syncthreads();   // this tile has landed; the other buffers' readers are done
    if (it + 1 < n_it) {
      if constexpr (par) ctx.issue(it + 1, q_lds0, do_lds0, lse_lds0, dl_lds0);
      else ctx.issue(it + 1, q_lds1, do_lds1, lse_lds1, dl_lds1);
    }
    // Operands are read a phase ahead of the MFMAs that take them, into the other of two sets of registers, and the vector work
    // of a 32-row block sits beside the matrix work of the phases behind it. A lone wave (d = 128) reads them before the phase's
    // products begin: read behind most of them, every phase began by waiting for LDS (B4 H16 N8192 4.34 ms, 4.15 so). With two
    // waves (d = 64) their place in the phase is the compiler's (first: B2 H16 N4096 causal backward 248 us, 250).
    auto first = [&]() {
      if constexpr (D == 128) fence();
    };
    bf16x8 ar0[KS], ar1[KS], at0[CB][2], at1[CB][2], pop0[2], ds0[2], pop1[2], ds1[2];
    f32x16 s0, p0, s1, p1;
    f32x4 l4[4];
    auto product = [&](const bf16x8 (&a)[KS], const bf16x8 (&b)[KS], f32x16& acc) {
#pragma unroll
      for (int s = 0; s < KS; ++s) acc = mfma(a[s], b[s], acc);
    };
    // a block's row statistics come in the accumulator's order: lse for the exponent, -D straight into the
    // accumulator of dP
    auto read_lse = [&](int qb) {
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) l4[i4] = *(const f32x4*)&lse_lds[32 * qb + 8 * i4 + 4 * hh];
    };
    auto read_neg_d = [&](int qb, f32x16& acc) {
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 x = *(const f32x4*)&dl_lds[32 * qb + 8 * i4 + 4 * hh];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * i4 + e] = x[e];
      }
    };
    // S to P, in place and as an operand; dP to dS
    auto p_operands = [&](f32x16& sacc, int qb, bf16x8 (&pop)[2]) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sacc[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], sl2e, -l4[i >> 2][i & 3]));
      if constexpr (decltype(masked_c)::value) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[i] = (unsigned)(i0 + 32 * qb + acc_row(i, hh) - see_from) < see_rows ? sacc[i] : 0.0f;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) pop[i >> 3][i & 7] = (bf16)sacc[i];
    };
    auto ds_operands = [&](const f32x16& pv, const f32x16& dpacc, bf16x8 (&dsop)[2]) {
#pragma unroll
      for (int i = 0; i < 16; ++i) dsop[i >> 3][i & 7] = (bf16)(pv[i] * dpacc[i]);
    };
    auto update = [&](const bf16x8 (&at)[CB][2], const bf16x8 (&b)[2], f32x16 (&acc)[CB]) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) acc[cb] = mfma(at[cb][tt], b[tt], acc[cb]);
    };
    zero(s0);
    zero(s1);
    read_rows<D>(q_lds, 0, off, ar0);
    read_neg_d(0, p0);
    read_lse(0);
    fence();
    read_rows<D>(do_lds, 0, off, ar1);
    first();
    product(ar0, kop, s0);
    fence();
    read_rows<D>(q_lds, 1, off, ar0);
    first();
    product(ar1, vop, p0);
    p_operands(s0, 0, pop0);
    fence();
    read_rows<D>(do_lds, 1, off, ar1);
    read_neg_d(1, p1);
    read_lse(1);
    first();
    product(ar0, kop, s1);
    ds_operands(s0, p0, ds0);
    fence();
    read_transposed<D>(do_lds, 0, off, at0);
    first();
    product(ar1, vop, p1);
    p_operands(s1, 1, pop1);
    fence();
    read_transposed<D>(q_lds, 0, off, at1);
    first();
    update(at0, pop0, dvacc);
    ds_operands(s1, p1, ds1);
    fence();
    read_transposed<D>(do_lds, 1, off, at0);
    first();
    update(at1, ds0, dkacc);
    fence();
    read_transposed<D>(q_lds, 1, off, at1);
    first();
    update(at0, pop1, dvacc);
    fence();
    update(at1, ds1, dkacc);
  };
  // Iterations [a, b), b - a even, with or without the mask; buffer parity = iteration parity.
  // The loop is unrolled by two over fixed buffers, masked and unmasked tiles run in loops of
  // their own.
  auto run = [&](int a, int b, auto masked_c) {
    for (int it = a; it < b; it += 2) {
      tile_step(std::integral_constant<int, 0>(), masked_c, it);
      tile_step(std::integral_constant<int, 1>(), masked_c, it + 1);
    }
  };
  // Per query head (an even number of tiles; a tile past the last query row is masked out
  // entirely): the first m1 tiles touch the causal diagonal (all tiles, when some key of the
  // workgroup does not exist), the last two may hold rows past N; the tiles between need no
  // mask: every row is a query, every key exists and is visible to all rows.
  int m1 = 0;
  if (n0 + kBwdRows > Nk) m1 = tiles;
  else if (causal) m1 = min(tiles, (max(0, (n0 + kBwdRows - 1 - shift - i_start + kBwdStream - 1) / kBwdStream) + 1) & ~1);
  const int m2 = (i_start + tiles * kBwdStream > N && m1 < tiles) ? 2 : 0;
  for (int hh_ = 0; hh_ < rep; ++hh_) {
    const int base = hh_ * tiles;
    run(base, base + m1, std::true_type());
    run(base + m1, base + tiles - m2, std::false_type());
    run(base + tiles - m2, base + tiles, std::true_type());
  }
  if (valid && hsplit > 1) {
    // partial sums: [dK | dV][hsplit][B * Hkv * Nk][D] float
    const size_t elems = (size_t)gridDim.x / hsplit / Tw * Nk * D;
    float* dkrow = part + (size_t)hs * elems + (bk * Nk + key) * D;
    float* dvrow = dkrow + (size_t)hsplit * elems;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int c = 32 * cb + 8 * i4 + 4 * hh;
        f32x4 a, bq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = scale * dkacc[cb][4 * i4 + e];
          bq[e] = dvacc[cb][4 * i4 + e];
        }
        *(f32x4*)(dkrow + c) = a;
        *(f32x4*)(dvrow + c) = bq;
      }
  } else if (valid) {
    bf16* dkrow = dk + (bk * Nk + key) * D;
    bf16* dvrow = dv + (bk * Nk + key) * D;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int c = 32 * cb + 8 * i4 + 4 * hh;
        bf16x4 a, bq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = (bf16)(scale * dkacc[cb][4 * i4 + e]);
          bq[e] = (bf16)dvacc[cb][4 * i4 + e];
        }
        *(bf16x4*)(dkrow + c) = a;
        *(bf16x4*)(dvrow + c) = bq;
      }
  }
}

// dK and dV from the partial sums of the head-split dK/dV launch: out = sum over the hsplit parts,
// in a fixed order (results do not depend on the run), rounded once.
__global__ __launch_bounds__(256) void bwd_reduce_kernel(const float* __restrict__ part, bf16* __restrict__ dk,
                                                         bf16* __restrict__ dv, size_t elems, int hsplit) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= 2 * elems) return;
  const bool second = i >= elems;
  const size_t j = second ? i - elems : i;
  const float* src = part + (second ? (size_t)hsplit * elems : 0) + j;
  f32x4 acc = *(const f32x4*)src;
  for (int s = 1; s < hsplit; ++s) acc += *(const f32x4*)(src + (size_t)s * elems);
  bf16x4 y = {(bf16)acc[0], (bf16)acc[1], (bf16)acc[2], (bf16)acc[3]};
  *(bf16x4*)((second ? dv : dk) + j) = y;
}

// ------------------------------------------------------------------------------------------------
// Short sequences (at most 32 * NW keys), d = 64, as many kv heads as query heads: the whole backward of a
// head in one workgroup and one launch. Wave w owns the keys 32*w .. as in bwd_dkv_kernel; row tiles of 64
// pass through LDS, where they are also prepared (D_i, Q~). dS of a tile, of all keys, meets in LDS, and
// the workgroup takes dQ~^T = K^T dS^T from it: five products instead of the seven of the two kernels, Q, dO
// and O read once, nothing in scratch (the call still asks for the room of the other kernels).
//
// Bound: memory traffic (5 + 3 tensors of N rows) where there are heads to fill the chip, LDS cycles next.
// Iteration `it`, one barrier each, so that a wave's products, LDS phases and waits fall beside
// those of the SIMD's other wave:
//   S, dP, P, dS, dV, dK of tile it | rows of tile it + 1 into LDS, those of it + 2 asked for |
//   dQ~ of tile it - 1 into LDS | dQ of tile it - 2 grouped and stored
constexpr int kShortMaxGroup = 4;
template <int NW, bool GROUPED>
__global__ __launch_bounds__(NW * 64, 2) void bwd_short_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, const bf16* __restrict__ o,
    const bf16* __restrict__ dout, const float* __restrict__ lse, bf16* __restrict__ dq, bf16* __restrict__ dk,
    bf16* __restrict__ dv, const uint8_t* __restrict__ perm, int N, int Nk, int Br, int Tq, int G,
    int causal, float scale) {
  constexpr int D = 64, CH = D / 8, KS = D / 16, CB = D / 32, T = NW * 64, KEYS = NW * 32;
  constexpr int TILE = kBwdStream * D * 2, RAW = D * 2 + 16;
  constexpr int CPT = kBwdStream * CH / T;           // 16-byte chunks of a row tile per thread
  constexpr int QB = 16 / NW;                        // 16-row blocks of dQ~ per wave (16 channels each)
  constexpr int SLOTS = 8;                           // tables of the tiles in flight (it - 2 .. it + 2)
  __shared__ __attribute__((aligned(1024))) char ds_lds[2][KEYS * kBwdStream * 2];   // [key][row of the tile]
  __shared__ __attribute__((aligned(1024))) char q_lds[2][TILE];                     // Q~
  __shared__ __attribute__((aligned(1024))) char do_lds[2][TILE];
  __shared__ __attribute__((aligned(1024))) float stage_lds[2][kBwdStream][D];       // dQ~, 16-byte pieces ^ row
  __shared__ __attribute__((aligned(16))) char raw_lds[GROUPED ? kBwdStream * RAW : 16];
  __shared__ __attribute__((aligned(16))) float lse_lds[2][kBwdStream];              // lse * log2(e)
  __shared__ __attribute__((aligned(16))) float nd_lds[2][kBwdStream];               // -D
  // tables of a tile's Q block: the sampled channel of a channel's group; per sampled channel the group's other
  // members (255 in the first row for channels that are not sampled)
  __shared__ __attribute__((aligned(8))) uint8_t rep_lds[GROUPED ? SLOTS : 1][D];
  __shared__ __attribute__((aligned(8))) uint8_t mem_lds[GROUPED ? SLOTS : 1][kShortMaxGroup][D];

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const size_t bh = blockIdx.x;                      // b * H + h
  const int key0 = 32 * w, key = key0 + lq;
  const bool valid = key < Nk;
  const int shift = Nk - N;
  const float sl2e = scale * kLog2e;
  const int n_it = (N + kBwdStream - 1) / kBwdStream;
  const size_t row0 = bh * N;                        // the head's first row

  // (the thread's index, renewed for every iteration: kept from one to the next, the addresses that follow from
  // it would take the registers of the products)
  int tl = tid;

  // ---- tables: wave 0 alone, a byte per lane
  auto load_table = [&](int it) -> int {
    if (!GROUPED || w != 0 || it >= n_it) return 0;
    return perm[(bh * Tq + it * kBwdStream / Br) * D + lane] & (D - 1);
  };
  auto write_table = [&](int it, int c) {
    if constexpr (GROUPED) {
      if (w != 0 || it >= n_it) return;
      const int slot = it & (SLOTS - 1), first = lane / G * G;
      rep_lds[slot][c] = (uint8_t)__shfl(c, first);
#pragma unroll
      for (int m = 0; m < kShortMaxGroup; ++m) {
        const int other = __shfl(c, min(lane + m, D - 1));
        if (m < G) mem_lds[slot][m][c] = (uint8_t)(lane == first ? other : 255);
      }
    }
  };

  // ---- rows: this thread's chunks of a tile (and, from the first thread of a row, its statistics)
  u32x4 qx[CPT], ox[CPT], dx[CPT];
  float lx[CPT];
  auto fetch = [&](int it) {
    if (it >= n_it) return;
    const int r0 = it * kBwdStream;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int row = r0 + (u * T + tl) / CH, chunk = tl % CH;
      qx[u] = ox[u] = dx[u] = u32x4{0u, 0u, 0u, 0u};
      lx[u] = 0.0f;
      if (row < N) {
        const size_t at = (row0 + row) * D + chunk * 8;
        qx[u] = *(const u32x4*)(q + at);
        ox[u] = *(const u32x4*)(o + at);
        dx[u] = *(const u32x4*)(dout + at);
        if (chunk == 0) lx[u] = lse[row0 + row];
      }
    }
  };
  auto place = [&](int it) {                          // the fetched rows into the tile's buffers
    const int par = it & 1;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int lr = (u * T + tl) / CH, chunk = tl % CH;
      const bf16x8 a = __builtin_bit_cast(bf16x8, dx[u]), b = __builtin_bit_cast(bf16x8, ox[u]);
      float acc = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) acc = __builtin_fmaf((float)a[j], (float)b[j], acc);
#pragma unroll
      for (int m = 1; m < CH; m <<= 1) acc += __shfl_xor(acc, m);
      if (chunk == 0) {
        nd_lds[par][lr] = -acc;
        lse_lds[par][lr] = lx[u] * kLog2e;
      }
      *(u32x4*)chunk_addr<D>(do_lds[par], lr, chunk) = dx[u];
      if constexpr (GROUPED) {
        // (the eight threads of a row are lanes of one wave: their writes precede the reads in its order)
        *(u32x4*)(raw_lds + lr * RAW + chunk * 16) = qx[u];
        __builtin_amdgcn_wave_barrier();
        const u32x2 from = *(const u32x2*)&rep_lds[it & (SLOTS - 1)][chunk * 8];
        bf16x8 y;
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = *(const bf16*)(raw_lds + lr * RAW + ((from[j >> 2] >> (8 * (j & 3))) & (D - 1)) * 2);
        *(bf16x8*)chunk_addr<D>(q_lds[par], lr, chunk) = y;
        __builtin_amdgcn_wave_barrier();
      } else {
        *(u32x4*)chunk_addr<D>(q_lds[par], lr, chunk) = qx[u];
      }
    }
  };
  // dQ of tile `it` from the staged dQ~: the members' columns summed into the sampled channel
  auto store_dq = [&](int it) {
    const int r0 = it * kBwdStream;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int lr = (u * T + tl) / CH, chunk = tl % CH;
      const float* row = stage_lds[it & 1][lr];
      const f32x4 lo = *(const f32x4*)(row + (((2 * chunk) ^ (lr & 15)) << 2)), hi = *(const f32x4*)(row + (((2 * chunk + 1) ^ (lr & 15)) << 2));
      float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if constexpr (GROUPED) {
        const uint8_t(*mem)[D] = mem_lds[it & (SLOTS - 1)];
        const u32x2 own = *(const u32x2*)&mem[0][chunk * 8];
        for (int m = 1; m < G; ++m) {
          const u32x2 other = *(const u32x2*)&mem[m][chunk * 8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int c = (other[e >> 2] >> (8 * (e & 3))) & (D - 1);
            x[e] += row[(((c >> 2) ^ (lr & 15)) << 2) | (c & 3)];
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (((own[e >> 2] >> (8 * (e & 3))) & 255) == 255) x[e] = 0.0f;
      }
      if (r0 + lr < N) {
        bf16x8 y;
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = (bf16)(scale * x[e]);
        *(bf16x8*)(dq + (row0 + r0 + lr) * D + chunk * 8) = y;
      }
    }
  };

  fetch(0);
  {   // K passes through the dS buffers on its way to the operands of dQ~
    const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + bh * Nk * D, (unsigned)Nk * D * 2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int slot = (j * NW + w) * 64 + lane, row = slot / CH, pc = slot % CH;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (lds_void*)(ds_lds[0] + (j * NW + w) * 1024), 16,
                                               row * (D * 2) + ((pc ^ chunk_swz<D>(row)) << 4), 0, 0, 0);
    }
  }
  write_table(0, load_table(0));
  write_table(1, load_table(1));
  int next_table = load_table(2);
  bf16x8 kop[KS], vop[KS];
  {
    const size_t row_off = (bh * Nk + (valid ? key : 0)) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
      if (valid) {
        x = *(const u32x4*)(k + row_off + (2 * s + hh) * 8);
        y = *(const u32x4*)(v + row_off + (2 * s + hh) * 8);
      }
      kop[s] = __builtin_bit_cast(bf16x8, x);
      vop[s] = __builtin_bit_cast(bf16x8, y);
    }
  }
  f32x16 dkacc[CB], dvacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    zero(dkacc[cb]);
    zero(dvacc[cb]);
  }
  const OperandOffsets<D> off(lane);
  // dS of this wave's keys: 8-byte pieces (4 rows of the tile) of key row `key`; the tile's other 32 rows: ^ 64
  int ds_off[4];
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) ds_off[i4] = (int)(chunk_addr<D>(nullptr, key, i4) - (char*)nullptr) + 8 * hh;
  // dQ~^T[ch][row] on v_mfma_f32_16x16x32_bf16: this wave's 16 channels and QB blocks of 16 rows, all keys.
  // Transposing reads of a [key][64] buffer: lanes address keys 8*(lane/16) + (lane%16)/4 (+4), columns
  // 16*block + 4*(lane%4) ..; lane i%16 receives column 16*block + i%16 of its 8 keys.
  const int ch16 = w & 3, qb0 = (w >> 2) * QB;
  auto tr16 = [&](const char* buf, int block, int step) {
    const int ln = tl & 63, row = 8 * (ln >> 4) + ((ln & 15) >> 2), chunk = 2 * block + ((ln & 3) >> 1);
    const char* base = buf + step * 32 * (D * 2) + 8 * (ln & 1);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + row * (D * 2) + ((chunk ^ chunk_swz<D>(row)) << 4)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + (row + 4) * (D * 2) + ((chunk ^ chunk_swz<D>(row + 4)) << 4)));
    const s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, r);
  };
  wait_loads();                                      // K has landed
  __syncthreads();
  place(0);
  fetch(1);
  asm volatile("" : "+v"(tl));
  bf16x8 kt[NW];
#pragma unroll
  for (int s = 0; s < NW; ++s) kt[s] = tr16(ds_lds[0], ch16, s);
  if (key0 >= Nk) {                                  // dS of a wave without keys: zero, as its K rows in the other buffer are
#pragma unroll
    for (int u = 0; u < 4; ++u) *(u32x4*)(ds_lds[1] + w * 4096 + u * 1024 + (tid & 63) * 16) = u32x4{0u, 0u, 0u, 0u};
  }
  __syncthreads();

#pragma unroll 1
  for (int it = 0; it < n_it + 2; ++it) {
    asm volatile("" : "+v"(tl));
    if (it < n_it) {
      const int par = it & 1, r0 = it * kBwdStream;
      const char* qt = q_lds[par];
      const char* dot = do_lds[par];
      // ---- S, dP, P, dS; dV, dK; dS into LDS
      const int blocks = key0 >= Nk ? 0 : r0 + 32 < N ? 2 : 1;   // 32-row blocks of the tile that hold rows (a wave without keys: none)
#pragma unroll 1
      for (int qb = 0; qb < blocks; ++qb) {
        char* ds_dst = ds_lds[par];
        const int flip = qb << 6;
        const int q0 = r0 + 32 * qb;
        bf16x8 ar[KS], at[CB][2], pop[2], dsop[2];
        f32x16 sacc, dpacc;
        f32x4 l4[4];
        zero(sacc);
        read_rows<D>(qt, qb, off, ar);
        fence();
#pragma unroll
        for (int s = 0; s < KS; ++s) sacc = mfma(ar[s], kop[s], sacc);
        read_rows<D>(dot, qb, off, ar);
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          l4[i4] = *(const f32x4*)&lse_lds[par][32 * qb + 8 * i4 + 4 * hh];
          const f32x4 x = *(const f32x4*)&nd_lds[par][32 * qb + 8 * i4 + 4 * hh];
#pragma unroll
          for (int e = 0; e < 4; ++e) dpacc[4 * i4 + e] = x[e];
        }
        fence();
#pragma unroll
        for (int s = 0; s < KS; ++s) dpacc = mfma(ar[s], vop[s], dpacc);
        read_transposed<D>(dot, qb, off, at);
        float pv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) pv[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], sl2e, -l4[i >> 2][i & 3]));
        // (rows past N hold zeros and reach nothing; keys past Nk must not reach dQ)
        if (key0 + 32 > Nk || (causal && key0 + 31 > q0 + shift)) {
          const int first = valid ? (causal ? key - shift - q0 : 0) : 32;   // row of the block that sees this key first
#pragma unroll
          for (int i = 0; i < 16; ++i) pv[i] = acc_row(i, hh) >= first ? pv[i] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          pop[i >> 3][i & 7] = (bf16)pv[i];
          dsop[i >> 3][i & 7] = (bf16)(pv[i] * dpacc[i]);
        }
        fence();
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) dvacc[cb] = mfma(at[cb][tt], pop[tt], dvacc[cb]);
        read_transposed<D>(qt, qb, off, at);
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *(u32x2*)(ds_dst + (ds_off[i4] ^ flip)) =
              i4 & 1 ? __builtin_bit_cast(u32x2, __builtin_shufflevector(dsop[i4 >> 1], dsop[i4 >> 1], 4, 5, 6, 7))
                     : __builtin_bit_cast(u32x2, __builtin_shufflevector(dsop[i4 >> 1], dsop[i4 >> 1], 0, 1, 2, 3));
        fence();
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) dkacc[cb] = mfma(at[cb][tt], dsop[tt], dkacc[cb]);
      }
    }
    if (it + 1 < n_it) {
      place(it + 1);
      fetch(it + 2);
      write_table(it + 2, next_table);
      next_table = load_table(it + 3);
    }
    if (it > 0 && it <= n_it) {
      // ---- dQ~ of the last tile (buffers of keys past Nk hold zeros; a block of rows past N is never stored)
      const char* ds = ds_lds[(it - 1) & 1];
      const int r0 = (it - 1) * kBwdStream;
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        if (r0 + 16 * (qb0 + b) >= N) break;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s0 = 0; s0 < NW; s0 += 4) {
          bf16x8 x[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) x[s] = tr16(ds, qb0 + b, s0 + s);
          fence();
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt[s0 + s], x[s], acc, 0, 0, 0);
        }
        const int ln = tl & 63, lr = 16 * (qb0 + b) + (ln & 15);   // register i: channel 16*ch16 + 4*(lane/16) + i of this row
        *(f32x4*)&stage_lds[(it - 1) & 1][lr][((4 * ch16 + (ln >> 4)) ^ (lr & 15)) << 2] = acc;
      }
    }
    if (it > 1) store_dq(it - 2);
    __syncthreads();
  }
  // ---- dK, dV: 32 rows of a wave by way of its part of the dS buffers, whole rows to memory
  char* out = ds_lds[0] + w * 4096;
  auto store_rows = [&](const f32x16 (&acc)[CB], float factor, bf16* dst) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        bf16x4 a;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = (bf16)(factor * acc[cb][4 * i4 + e]);
        *(bf16x4*)(out + lq * (D * 2) + (((4 * cb + i4) ^ (lq & 7)) << 4) + 8 * hh) = a;
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = u * 8 + lane / CH, chunk = lane % CH;
      const u32x4 x = *(const u32x4*)(out + row * (D * 2) + ((chunk ^ (row & 7)) << 4));
      if (key0 + row < Nk) *(u32x4*)(dst + (bh * Nk + key0 + row) * D + chunk * 8) = x;
    }
    __builtin_amdgcn_wave_barrier();
  };
  store_rows(dkacc, scale, dk);
  store_rows(dvacc, 1.0f, dv);
}

// Workgroups of the dK/dV launch that share one kv head's keys but take different query heads: used
// when the launch would otherwise not fill the chip twice over (grouped-query shapes with few kv
// heads; under the causal mask its workgroups differ many-fold in length and need company).
// Every share costs a float copy of dK and dV, written here and read by bwd_reduce_kernel. Where a smaller number of
// shares fills the chip by itself (one workgroup per compute unit, two at d = 64; under the mask, d = 128, two rounds) and the
// key tiles are whole, it is taken: the resident workgroups end together. A launch that is less full, or whose heads end in
// a ragged tile (masked at every step, so its workgroup is the last), lives on many short ones, and so does the mask at d = 64.
// The line: heads dealt out by a smaller number are faster from 0.8 of a full chip on (time over that of all dealt out, at 3/4, 13/16,
// 7/8 and all of it: d128 not causal 0.93-0.95, 0.94-0.96, 0.95-0.97, 0.95-0.98; causal 0.93-1.00, 0.89-0.98, 0.89-0.95, 0.90-0.96; d64 not causal
// 1.03-1.06, 0.95-0.97, 0.96-0.97, 0.97-0.99) and lose past it (17/16: 1.11, 0.93-0.98, 1.06-1.09); 7/8 is on the safe side of that.
// Whole backward, us, all heads dealt out | the rule: d128 causal H32 Hkv8 N4096 545 | 519, N3712 465 | 444, B8 N512 215 | 168; not causal
// N2048 267 | 256, N4096 937 | 893, H24 Hkv4 N4096 708 | 688, B16 H32 Hkv8 N128 81 | 65; d64 not causal N4096 480 | 474, B4 N1024 160 | 150,
// B16 N256 85 | 74. Fewer shares elsewhere: d64 causal H32 Hkv8 N4096 284 | 297, ragged N3800 d128 859 | 975, 3/4 full (B2 H24 Hkv4
// N2048 d64) 191 | 200.
static int dkv_head_split(const Problem& pb) {
  const int rep = pb.H / pb.Hkv;
  const long long k_units = (long long)pb.B * pb.Hkv * ((pb.Nk + kBwdRows - 1) / kBwdRows);
  if (k_units >= 2 * kComputeUnits) return 1;
  const long long full = (pb.causal || pb.d == 64 ? 2 : 1) * kComputeUnits;
  for (int n = 1; n < rep && pb.Nk % kBwdRows == 0 && !(pb.causal && pb.d == 64); ++n)
    if (rep % n == 0 && k_units * n > full * 7 / 8 && k_units * n <= full) return n;
  return rep;
}

// Where the one-workgroup backward is taken: what its LDS holds (keys, and the tables of groups of up to 4
// channels), and no grouped query heads, which one workgroup would have to take one after the other.
// Measured, three kernels | one: H12 N197 B64 100 | 68 us, B8 31 | 20, B1 29 | 19; N256 B64 106 | 75; N128 B64 52 | 42; N64
// B64 40 | 26, B4 23 | 10; with the loop over grouped heads H32 Hkv8 N200 B8 48 | 62, B1 30 | 63.
static bool bwd_short(const Problem& pb, int distr) {
  return pb.d == 64 && pb.H == pb.Hkv && pb.N <= 256 && pb.Nk <= 256 && (!distr || pb.d / pb.n_groups <= kShortMaxGroup);
}

size_t attn_bf16_bwd_scratch_bytes(const Problem& pb, int distr) {
  const size_t rows = (size_t)pb.B * pb.H * pb.N;
  const size_t stat = (rows * 4 + 255) & ~(size_t)255;   // D_i, and lse * log2(e)
  const int hsplit = dkv_head_split(pb);
  const size_t part = hsplit > 1 ? ((size_t)2 * hsplit * pb.B * pb.Hkv * pb.Nk * pb.d * 4 + 255) & ~(size_t)255 : 0;
  return 2 * stat + (distr ? ((rows * pb.d * 2 + 255) & ~(size_t)255) : 0) + part;
}

hipError_t launch_attn_bf16_bwd(const void* q, const void* k, const void* v, const void* o, const void* dout,
                                const float* lse, void* dq, void* dk, void* dv, const uint8_t* perm, void* scratch,
                                const Problem& pb, int distr, hipStream_t stream) {
  const int Tq = (pb.N + pb.Br - 1) / pb.Br;
  const int Twq = (pb.N + kBwdRows - 1) / kBwdRows;
  const int Twk = (pb.Nk + kBwdRows - 1) / kBwdRows;
  const long long q_units = (long long)pb.B * pb.H * Twq;
  const long long k_units = (long long)pb.B * pb.Hkv * Twk;
  if (q_units > 0x7fffffffLL || k_units > 0x7fffffffLL / 16) return hipErrorInvalidValue;
  if ((pb.d != 64 && pb.d != 128) || pb.Br % 32 != 0 || pb.d % pb.n_groups != 0) return hipErrorInvalidValue;
  // tiles are addressed by 32-bit byte offsets inside a head
  if ((size_t)pb.N * pb.d * 2 >= 0x7fffffffULL || (size_t)pb.Nk * pb.d * 2 >= 0x7fffffffULL) return hipErrorInvalidValue;
  const size_t rows = (size_t)pb.B * pb.H * pb.N;
  const size_t stat = (rows * 4 + 255) & ~(size_t)255;
  float* delta = (float*)scratch;
  float* lse2 = (float*)((char*)scratch + stat);
  bf16* qrep = distr ? (bf16*)((char*)scratch + 2 * stat) : nullptr;
  const int hsplit = dkv_head_split(pb);
  float* part = hsplit > 1 ? (float*)((char*)scratch + 2 * stat + (distr ? ((rows * pb.d * 2 + 255) & ~(size_t)255) : 0)) : nullptr;
  const size_t kv_elems = (size_t)pb.B * pb.Hkv * pb.Nk * pb.d;
  const uint8_t* table = distr ? perm : nullptr;
  const bf16* qx = distr ? qrep : (const bf16*)q;
  const int n_groups = distr ? pb.n_groups : pb.d;
  if (bwd_short(pb, distr)) {
#define DA_SHORT(NW, GR)                                                                                            \
  hipLaunchKernelGGL((bwd_short_kernel<NW, GR>), dim3((unsigned)(pb.B * pb.H)), dim3(NW * 64), 0, stream, (const bf16*)q, \
                     (const bf16*)k, (const bf16*)v, (const bf16*)o, (const bf16*)dout, lse, (bf16*)dq, (bf16*)dk,    \
                     (bf16*)dv, table, pb.N, pb.Nk, pb.Br, Tq, pb.d / n_groups, pb.causal, pb.scale)
    if (pb.Nk <= 128 && distr) DA_SHORT(4, true);
    else if (pb.Nk <= 128) DA_SHORT(4, false);
    else if (distr) DA_SHORT(8, true);
    else DA_SHORT(8, false);
#undef DA_SHORT
    return hipGetLastError();
  }
  const int dq_order = pb.causal && q_units <= kBalancedUnits ? kPaired : kHeadMajor;
  const int dkv_order = pb.causal && k_units * hsplit <= kBalancedUnits ? (pb.d == 64 ? kPaired : kLongestFirst) : kHeadMajor;
#define DA_BWD(DD)                                                                                                   \
  do {                                                                                                               \
    hipLaunchKernelGGL((bwd_dq_kernel<DD>), dim3((unsigned)q_units), dim3(kBwdThreads), 0, stream, (const bf16*)q,   \
                       (const bf16*)k, (const bf16*)v, (const bf16*)o, (const bf16*)dout, lse, qrep, lse2, delta,     \
                       (bf16*)dq, table, pb.H, pb.Hkv, pb.N, pb.Nk,                                                  \
                       pb.Br, Tq, Twq, n_groups, pb.causal, dq_order, pb.scale);                                               \
    hipLaunchKernelGGL((bwd_dkv_kernel<DD>), dim3((unsigned)(k_units * hsplit)), dim3(kBwdThreads), 0, stream, qx,   \
                       (const bf16*)k, (const bf16*)v, (const bf16*)dout, lse2, delta, (bf16*)dk, (bf16*)dv, part,    \
                       hsplit, pb.H, pb.Hkv, pb.N, pb.Nk, Twk, pb.causal, dkv_order, pb.scale);                                 \
    if (hsplit > 1)                                                                                                  \
      hipLaunchKernelGGL(bwd_reduce_kernel, dim3((unsigned)((2 * kv_elems / 4 + 255) / 256)), dim3(256), 0, stream,  \
                         part, (bf16*)dk, (bf16*)dv, kv_elems, hsplit);                                              \
  } while (0)
  if (pb.d == 64) DA_BWD(64);
  else DA_BWD(128);
#undef DA_BWD
  return hipGetLastError();
}

}  // namespace da
