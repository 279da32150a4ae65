// Attention forward (exact and DistrAttention) in float arithmetic for gfx950: the reference-precision
// path, for float tensors and (the mirrored form only) for bf16 tensors converted on load.
//
// Same steps as the bf16 kernel (Sec. 2.2.2 tiling; Sec. 3.2 sampling and fusion per Q block,
// Sec. 3.3; Eq. 2) on the float matrix instruction v_mfma_f32_32x32x2_f32 (float operands, float
// products and sums: the precision of the vector ALUs at twice their rate without packed forms).
// Bound: that instruction, 64 cycles for 4096 FLOP; where both operands are floats summed over groups of two or four channels
// (float_by_pieces in f32_tiles.h) the products are taken of three bf16 pieces each (6 products of 32 cycles for 8 of 64; what
// they leave out is 2^-24 of a product at most, and the distance from 64 bits is a fifth below that of the float instruction: H8 N2048
// 4.7e-7 -> 3.9e-7). There a tile is 36 products and 16 for the splitting, bound by issue and the clock (1.85 GHz under them, pipes busy
// 52 % of the time in which their unit has work). A workgroup with rows that pieces do not hold walks its keys twice: with all of
// them so (an infinity in V, a key of 2^70) mirrored H8 N2048 takes 126 us instead of 63, a training step 449-573 instead of 241.
// Both products are taken transposed, so that one lane owns one query row:
//   S^T[kv][q] = Kx Qx^T     A = keys from LDS, B = queries in registers
//   O^T[ch][q] = V^T P^T     A = V straight from global memory, B = P in registers: register i of
//                            a score accumulator holds the keys 8*(i/4) + i%4 (+ 4 in the upper
//                            half of the wave), which is the contraction index of step i.
//
// Split: a workgroup owns 32 query rows and its NW (4 or 8) waves deal the 32-key tiles out among
// themselves, each with a softmax state of its own; the states meet in LDS once at the end. No wave
// waits for another before that, and a problem of few rows still fills the chip: sharing tiles
// among waves of different rows instead would leave N = 256 with 8 working waves.
// Measured (B1 H8 N2048 d64 n_groups 32): by pieces 57 us, by floats 72 (92 TFLOP/s of the 157 the instruction can reach; float
// multiply-adds on the vector ALUs, a thread quad per row: 1430 us); mirrored 65 and 78; B1 H1 N256, grouping and all: 10.6 us (a kernel in front of it for the grouping: 12.4).
//
// Score product, by MODE:
//   kQueryFused  the wave writes its K tile into LDS in sorted channel order, a group's G channels
//                are then adjacent and are summed as they are read (Sec. 3.2 fusion); contraction
//                over n_groups. Built for groups of 2 and 4 channels.
//   kQueryFull   the same product as Q~ K^T, Q~ = Q with every channel replaced by its group's
//                sampled channel (a sum over groups of sums over members): contraction over d, for
//                every other group size; exact attention is groups of one channel.
//   kKeyFused,   the mirrored form of Sec. 3.1 (last sentence of the Eq. 2 paragraph, Fig. 4 right
//   kKeyFull     side): the grouping belongs to the K block (Bc rows, table [B][Hkv][Tk][d] from
//                the LSH stage run on K), one K column per group is sampled and the group's Q columns are
//                summed: every K block needs its own fused queries (the reloading Sec. 3.3 gives as
//                the reason for sampling Q instead), gathered from the Q rows in LDS. kKeyFull
//                replaces every key channel by its group's sampled one instead.
#include <cfloat>
#include <type_traits>

#include "f32_tiles.h"
#include "lsh_block.h"

namespace da {

namespace {

constexpr int kOwnRows = 256;   // of a Q block that a workgroup groups itself, d = 64 (with the tiles 93 KB of LDS, 128 KB for eight waves: one workgroup to a CU)

enum Mode { kQueryFull, kQueryFused, kKeyFull, kKeyFused };

// OWN: the workgroup groups the Q block that its rows lie in itself, into lds.perm, and writes its table where perm_w is given
// (rule: launch_waves).
template <typename E, int D, int G, int MODE, int NW, bool PIECES, bool OWN>
__global__ __launch_bounds__(NW * 64, (D == 64 && !(OWN && NW == 4) ? 2 : 1)) void attn_f32_kernel(
    const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v, E* __restrict__ o,
    const uint8_t* __restrict__ perm, int H, int Hkv, int N, int Nk, int Br, int Tq, int Tw, int n_groups,
    int causal, float scale, int Bc, float* __restrict__ lse, uint8_t* __restrict__ perm_w, int n_planes, int gray_mode, uint64_t seed) {
  constexpr bool kMirrored = MODE == kKeyFull || MODE == kKeyFused;
  constexpr bool kFused = MODE == kQueryFused || MODE == kKeyFused;
  constexpr int T = NW * 64;
  constexpr int KRED = kFused ? D / G : D;       // contraction length of the score product
  constexpr int HS = KRED / 2;                   // steps: each takes one slot from either half of the wave
  constexpr int NB = D / 32;                     // 32-channel blocks of the output; lane m owns channels NB*m ..
  constexpr int RS = D + 4;                      // LDS row length in floats: 16-byte aligned rows whose starts
                                                 // are 4 banks apart (16 lanes cover all 64 banks)
  constexpr int KU = kTile * D / 4 / 64;         // 4-channel pieces of a K tile per lane
  __shared__ __attribute__((aligned(16))) float q_lds[kTile * RS];
  __shared__ __attribute__((aligned(16))) float k_lds[NW][kTile * RS];   // K tile of each wave, at the end its output
  __shared__ float stat_lds[NW][2][kTile];
  __shared__ __attribute__((aligned(16))) uint8_t map_lds[kMirrored ? NW : 1][D];
  __shared__ uint32_t mark_lds[kTile + 1];   // PIECES: what is known of a row (kRowAgain ..); whether a key is beyond_pieces

  __shared__ typename std::conditional<OWN, LshLds<float, D, kOwnRows>, char>::type lsh_lds;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  // causal: the row tiles with the most keys first, over all heads
  const int n_bh = gridDim.x / Tw;
  const int t = causal ? Tw - 1 - (int)blockIdx.x / n_bh : (int)blockIdx.x / n_bh;
  const int bh = blockIdx.x % n_bh;
  const int b = bh / H, h = bh % H, hk = h / (H / Hkv);
  const int r0 = t * kTile;
  const int shift = Nk - N;   // causal: key n is visible to query i iff n <= i + shift

  const unsigned kv_bytes = (unsigned)Nk * D * sizeof(E);
  const __amdgpu_buffer_rsrc_t k_rsrc = head_rsrc(k + (size_t)(b * Hkv + hk) * Nk * D, kv_bytes);
  const __amdgpu_buffer_rsrc_t v_rsrc = head_rsrc(v + (size_t)(b * Hkv + hk) * Nk * D, kv_bytes);
  const __amdgpu_buffer_rsrc_t q_rsrc = head_rsrc(q + (size_t)bh * N * D, (unsigned)N * D * sizeof(E));

  const int n_end = causal ? min(Nk, r0 + kTile + shift) : Nk;
  const int n_tiles = (n_end + kTile - 1) / kTile;
  const int TB = kMirrored ? Bc / kTile : 1;     // tiles dealt out together: one K block of the mirrored form
  auto next_tile = [&](int tile) { return (TB > 1 && (tile + 1) % TB != 0 && tile + 1 < n_tiles) ? tile + 1 : (tile / TB + NW) * TB; };

  // K tile: piece u of this lane is row (u*64 + lane) / (D/4), channels 4*((u*64 + lane) % (D/4)) ..
  // (64 lanes cover whole rows); rows past the end read as zeros (range check of the descriptor).
  typename Quad<E>::raw kreg[KU];
  uint8_t map_reg[D / 64];
  auto load_k = [&](int tile) {
#pragma unroll
    for (int u = 0; u < KU; ++u) kreg[u] = Quad<E>::load(k_rsrc, (u * 64 + lane) * 4 * (int)sizeof(E), tile * (kTile * D * (int)sizeof(E)));
    if constexpr (kMirrored) {
      const size_t row = (size_t)(b * Hkv + hk) * ((Nk + Bc - 1) / Bc) + tile / TB;
#pragma unroll
      for (int u = 0; u < D / 64; ++u) map_reg[u] = perm[row * D + u * 64 + lane];
    }
  };
  // V of a tile is asked for behind the products of the tile before it, in front of the staging of its own K (a compute unit takes the
  // 24 KB of a wave's tile in at 64 bytes a cycle, half a microsecond for four waves, in which a wave cannot go on): d128 H4 N2000 89.2 ->
  // 85.1 us, groups of four H2 N1000 44.8 -> 41.2, d64 H8 N2048 59.0 -> 58.0. Slower with it: the mirrored form at d = 64 (62.8 -> 64.3), and eight waves
  // that begin with their first tiles (table given or exact, two waves to a SIMD: H8 N300 8.8 -> 9.4, exact 11.3 -> 11.8, H4 N500 13.4 -> 14.4).
  constexpr bool V_AHEAD = D == 128 || (!kMirrored && (OWN || NW == 4));
  constexpr int VR = NB / 2;   // raw pairs per row of V and lane
  typename Pair<E>::raw vreg[16][VR];
  auto load_v = [&](int tile) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int j = 0; j < VR; ++j)
        vreg[i][j] = Pair<E>::load(v_rsrc, (acc_row(i, hh) * D + lq * NB + 2 * j) * (int)sizeof(E), tile * (kTile * D * (int)sizeof(E)));
  };
  int tile = w * TB;
  if (tile < n_tiles) {
    load_k(tile);
    if (V_AHEAD && OWN) load_v(tile);
  }

  // Q rows of the workgroup into LDS; the Q block's permutation beside them.
  {
    constexpr int QU = kTile * D / 4 / T;
    typename Quad<E>::raw x[QU];
#pragma unroll
    for (int u = 0; u < QU; ++u) x[u] = Quad<E>::load(q_rsrc, (u * T + tid) * 4 * (int)sizeof(E), r0 * (D * (int)sizeof(E)));
#pragma unroll
    for (int u = 0; u < QU; ++u) *(f32x4*)&q_lds[(u * T + tid) / (D / 4) * RS + (u * T + tid) % (D / 4) * 4] = Quad<E>::values(x[u]);
    if (PIECES && tid <= kTile) mark_lds[tid] = 0;
  }
  if (V_AHEAD && !OWN && tile < n_tiles) load_v(tile);   // (in front of Q it would be waited for with it: d128 H8 N600 causal 33.6 -> 34.6 us)
  if constexpr (OWN) {
    const int t_block = r0 / Br;
    lsh_block<float, D, kOwnRows, T, true>((const float*)q + ((size_t)bh * N + (size_t)t_block * Br) * D, min(Br, N - t_block * Br), n_planes,
                                              gray_mode, seed, perm_w && r0 % Br == 0 ? perm_w + ((size_t)bh * Tq + t_block) * D : nullptr, nullptr, lsh_lds);
  }
  // the Q block's permutation
  auto table = [&]() {
    if constexpr (OWN) return (const uint8_t*)lsh_lds.perm;
    else return perm + ((size_t)bh * Tq + r0 / Br) * D;
  };
  int kdst[4];          // kQueryFused: where the lane's four channels go in a row sorted by group
  if constexpr (!kMirrored) {
    // map: position of a channel in sorted order (kQueryFused) / sampled channel of its group (kQueryFull)
    if (OWN || perm) {
      // D is a power of two: an out-of-range entry of a caller's table cannot index past a row
      const uint8_t* pr = table();
      const int group = D / n_groups;
      for (int i = tid; i < D; i += T)
        map_lds[0][pr[i] & (D - 1)] = kFused ? (uint8_t)i : (uint8_t)(pr[i / group * group] & (D - 1));
    } else {
      for (int i = tid; i < D; i += T) map_lds[0][i] = (uint8_t)i;
    }
  }
  __syncthreads();
  if constexpr (kFused && !kMirrored) {
#pragma unroll
    for (int e = 0; e < 4; ++e) kdst[e] = map_lds[0][(lane * 4 + e) % D] & (D - 1);
  }

  // One walk over the keys for the rows of the bit mask `rows`, products by pieces or on the float instruction. By pieces, the rows
  // to be taken again are returned; a second walk takes the scores by pieces that the first took by them (beyond_pieces), and with
  // k_again set it is for the rows, too, that see a key that is not held by pieces.
  bool k_again = false;
  auto pass = [&](auto pieces, uint32_t rows) -> uint32_t {
    constexpr bool BY_PIECES = decltype(pieces)::value;
    constexpr float raise_v = std::is_same<E, float>::value ? kRaise : 1.0f;   // (a bf16 value is its first piece)
    const Splitter splitter(lane);
    float qop[HS];
    if constexpr (MODE == kQueryFused) {
      // sampling: the group's first channel in sorted order
      const uint8_t* pr = table();
#pragma unroll
      for (int s = 0; s < HS; ++s) qop[s] = q_lds[lq * RS + (pr[(hh * HS + s) * G] & (D - 1))];
    } else if constexpr (MODE == kQueryFull) {
#pragma unroll
      for (int s = 0; s < HS; ++s) qop[s] = q_lds[lq * RS + (map_lds[0][hh * HS + s] & (D - 1))];
    } else if constexpr (MODE == kKeyFull) {
#pragma unroll
      for (int s = 0; s < HS; ++s) qop[s] = q_lds[lq * RS + hh * HS + s];
    }
    Pieces qpc[PIECES ? HS / 8 : 1];
    auto split_q = [&]() {
      if constexpr (PIECES) split_steps<HS, false>(splitter, qop, [&](int s, const Pieces& p) { qpc[s] = p; });
    };
    if constexpr (!kMirrored) split_q();
    uint32_t any_beyond = 0, q_beyond = 0;   // rows whose scores are not by pieces
    auto find_q_beyond = [&]() {
      float m = 0.0f;
      if constexpr (kMirrored) {
#pragma unroll
        for (int c = 0; c < D / 2; c += 4) m = largest(m, *(const f32x4*)&q_lds[lq * RS + hh * (D / 2) + c]);
      } else {
        m = largest(qop);
      }
      q_beyond = rows_of(beyond_pieces(m));
    };
    if constexpr (PIECES) find_q_beyond();
    float* kt = k_lds[w];
    int koff[kMirrored ? HS : 1];   // channel of the K row that contraction slot s takes (mirrored form)
    f32x16 oacc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) zero(oacc[mb]);
    // Reference and scores stay unscaled until their difference is taken: exact to the last bit of the difference
    // whatever their size (one fused multiply-add against a scaled reference keeps the rounding of the reference).
    float m_run = -FLT_MAX, l_run = 0.0f;   // l over this lane's half of the keys
    const float scale_log2e = scale * 1.4426950408889634f;
    const int q_abs = r0 + lq;
    const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;   // last key this row sees

    // The loop on an instruction line: by where the code in front put it H1 N256 in groups of two took 12.4 .. 12.7 us.
    if constexpr (kFused && D == 64) asm volatile(".p2align 6");
    while (tile < n_tiles) {
      // ---- stage the K tile (and, mirrored, the K block's grouping) -------------------------------
      wave_order();   // the reads of the previous tile come first
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        const f32x4 x = Quad<E>::values(kreg[u]);
        const int row = (u * 64 + lane) / (D / 4), c = (u * 64 + lane) % (D / 4) * 4;
        if constexpr (MODE == kQueryFused) {
#pragma unroll
          for (int e = 0; e < 4; ++e) kt[row * RS + kdst[e]] = x[e];
        } else {
          *(f32x4*)&kt[row * RS + c] = x;
        }
      }
      const bool new_block = kMirrored && tile % TB == 0;
      if constexpr (kMirrored) {
        if (new_block) {
          if constexpr (kFused) {
#pragma unroll
            for (int u = 0; u < D / 64; ++u) map_lds[w][u * 64 + lane] = map_reg[u] & (D - 1);
          } else {
            // a channel's group's first channel: lane i of the sorted order names its own
            const int group = D / n_groups;
            uint8_t* tmp = (uint8_t*)&stat_lds[w][0][0];   // (the softmax states use it after the loop only)
#pragma unroll
            for (int u = 0; u < D / 64; ++u) tmp[u * 64 + lane] = map_reg[u] & (D - 1);
            wave_order();
#pragma unroll
            for (int u = 0; u < D / 64; ++u) {
              const int i = u * 64 + lane;
              map_lds[w][tmp[i]] = tmp[i / group * group];
            }
          }
        }
      }
      wave_order();
      // (V of this tile and) K of the next one: in flight under the products
      if (!V_AHEAD) load_v(tile);
      // (unconditional, so that the waits for V can count the loads of K behind it: the last tile again when there is no next one)
      const int following = next_tile(tile);
      load_k(min(following, n_tiles - 1));

      if constexpr (kMirrored) {
        if (new_block) {
          // entries of this half of the wave: positions hh*D/2 .. of the sorted order (kKeyFused), the
          // sampled channels of its channels (kKeyFull)
#pragma unroll
          for (int c16 = 0; c16 < D / 2; c16 += 16) {
            const u32x4 e4 = *(const u32x4*)&map_lds[w][hh * (D / 2) + c16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int ch = (e4[e >> 2] >> (8 * (e & 3))) & (D - 1);
              if constexpr (MODE == kKeyFull) {
                koff[c16 + e] = ch;
              } else {
                const float x = q_lds[lq * RS + ch];   // fusion of Q, members in sorted order
                if ((c16 + e) % G == 0) {
                  koff[(c16 + e) / G] = ch;
                  qop[(c16 + e) / G] = x;
                } else {
                  qop[(c16 + e) / G] += x;
                }
              }
            }
          }
          if constexpr (MODE == kKeyFused) split_q();
        }
      }

      // ---- scores -----------------------------------------------------------------------------------
      PieceSum by_pieces;
      ChannelSum<HS> by_floats;
      float kop[PIECES ? HS : 1];
      auto put = [&](int s, float x) {   // float s of the lane's half row
        if constexpr (PIECES) kop[s] = x;
        else by_floats.step(s, x, qop[s]);
      };
      if constexpr (kMirrored) {
#pragma unroll
        for (int s = 0; s < HS; ++s) put(s, kt[lq * RS + koff[s]]);
      } else {
#pragma unroll
        for (int c = 0; c < D / 2; c += 4) {
          const f32x4 x = *(const f32x4*)&kt[lq * RS + hh * (D / 2) + c];
          if constexpr (MODE == kQueryFull) {
#pragma unroll
            for (int e = 0; e < 4; ++e) put(c + e, x[e]);
          } else if constexpr (G == 2) {
            put(c / 2, x[0] + x[1]);
            put(c / 2 + 1, x[2] + x[3]);
          } else {
            put(c / 4, ((x[0] + x[1]) + x[2]) + x[3]);
          }
        }
      }
      f32x16 sacc;
      if constexpr (PIECES) {
        if constexpr (BY_PIECES) any_beyond |= rows_of(beyond_pieces(largest(kop)));
        split_steps<HS>(splitter, kop, [&](int s, const Pieces& p) { by_pieces.step(p, qpc[s]); });
        sacc = by_pieces.sum();
      }
      if constexpr (!PIECES) {
        sacc = by_floats.sum();
      } else if constexpr (!BY_PIECES) {
        const uint32_t k_beyond = rows_of(beyond_pieces(largest(kop)));
        if (k_beyond != 0 && tile * kTile + __builtin_ctz(k_beyond) <= lim) atomicOr(&mark_lds[lq], kRowBeyond);
        if ((q_beyond | k_beyond) != 0) {
#pragma unroll
          for (int s = 0; s < HS; ++s) by_floats.step(s, kop[s], qop[s]);
          const f32x16 y = by_floats.sum();
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[i] = ((q_beyond >> lq | k_beyond >> acc_row(i, hh)) & 1) != 0 ? y[i] : sacc[i];
        }
      }
      const int n0 = tile * kTile;
      if (n0 + kTile > Nk || (causal && n0 + kTile - 1 > r0 + shift)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (n0 + acc_row(i, hh) > lim) sacc[i] = -INFINITY;
      }
      // ---- online softmax step (Sec. 2.2.2) -------------------------------------------------------
      float mt = sacc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mt = fmaxf(mt, sacc[i]);
      const float m_new = fmaxf(m_run, half_swap_max(mt));
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);
        l_run *= alpha;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[mb][i] *= alpha;
        m_run = m_new;
      }
      float ps[16], sum0 = 0.0f, sum1 = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        ps[i] = __builtin_amdgcn_exp2f((sacc[i] - m_run) * scale_log2e);
        ps[i + 1] = __builtin_amdgcn_exp2f((sacc[i + 1] - m_run) * scale_log2e);
        sum0 += ps[i];
        sum1 += ps[i + 1];
      }
      l_run += sum0 + sum1;
      // ---- O^T += V^T P^T -----------------------------------------------------------------------------
      if constexpr (BY_PIECES) {
        f32x16 x;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = ps[i] * kRaise;
        Pieces p0, p1, v0, v1;
        splitter(x, p0, p1);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = Pair<E>::value(vreg[i][mb >> 1], mb & 1) * raise_v;
          splitter(x, v0, v1);
          oacc[mb] = mfma(v0, p0, oacc[mb]);
          oacc[mb] = mfma(v1, p1, oacc[mb]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int mb = 0; mb < NB; ++mb)
            oacc[mb] = mfma(Pair<E>::value(vreg[i][mb >> 1], mb & 1), ps[i], oacc[mb]);
      }
      if (V_AHEAD) load_v(min(following, n_tiles - 1));
      tile = following;
    }

    // ---- the waves' states meet: rows of (reference, sum), then the outputs -------------------------
    const float l_tot = half_swap_sum(l_run);
    wave_order();
    if (hh == 0) {
      stat_lds[w][0][lq] = m_run;
      stat_lds[w][1][lq] = l_tot;
    }
    __syncthreads();
    float m_all = stat_lds[0][0][lq];
#pragma unroll
    for (int j = 1; j < NW; ++j) m_all = fmaxf(m_all, stat_lds[j][0][lq]);
    float l_all = 0.0f;
#pragma unroll
    for (int j = 0; j < NW; ++j) l_all += stat_lds[j][1][lq] * __builtin_amdgcn_exp2f((stat_lds[j][0][lq] - m_all) * scale_log2e);
    const float weight = __builtin_amdgcn_exp2f((m_run - m_all) * scale_log2e) / l_all;
    if constexpr (BY_PIECES) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mb][i] *= 1.0f / (kRaise * raise_v);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = acc_row(i, hh);
      if constexpr (NB == 2) {
        const float x[2] = {oacc[0][i] * weight, oacc[1][i] * weight};
        __builtin_memcpy(__builtin_assume_aligned(&kt[lq * RS + m * 2], 8), x, 8);
      } else {
        const f32x4 x = {oacc[0][i] * weight, oacc[1][i] * weight, oacc[2][i] * weight, oacc[NB - 1][i] * weight};
        *(f32x4*)&kt[lq * RS + m * 4] = x;
      }
    }
    // row statistics for a backward pass: ln(sum of exp(score)) = rounded reference (see scaled_plus) + ln(sum)
    auto wanted = [&](int row) { return (rows >> row & 1) != 0 || (PIECES && !BY_PIECES && (mark_lds[row] & kRowBeyond) != 0); };
    if (lse && w == 0 && hh == 0 && q_abs < N && wanted(lq))
      lse[(size_t)bh * N + q_abs] = __builtin_fmaf(__builtin_log2f(l_all), 0.6931471805599453f, m_all * scale);
    __syncthreads();
    for (int i = tid; i < kTile * D / 4; i += T) {
      const int row = i / (D / 4), c = i % (D / 4) * 4;
      if (r0 + row < N && wanted(row)) {
        f32x4 x = *(const f32x4*)&k_lds[0][row * RS + c];
#pragma unroll
        for (int j = 1; j < NW; ++j) x += *(const f32x4*)&k_lds[j][row * RS + c];
        if (BY_PIECES && !all_finite(x)) atomicOr(&mark_lds[row], kRowAgain);
        E* dst = o + ((size_t)bh * N + r0 + row) * D + c;
        if constexpr (std::is_same<E, float>::value) {
          *(f32x4*)dst = x;
        } else {
          const bf16x4 y = {(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
          *(bf16x4*)dst = y;
        }
      }
    }
    if constexpr (!BY_PIECES) return 0;
    if (any_beyond != 0) atomicOr(&mark_lds[kTile], 1u);
    __syncthreads();
    k_again = mark_lds[kTile] != 0;
    return rows_of((mark_lds[lq] & kRowAgain) != 0) | q_beyond;
  };
  if constexpr (PIECES) {
    const uint32_t again = pass(std::true_type(), ~0u);
    if (again == 0 && !k_again) return;
    tile = w * TB;
    if (tile < n_tiles) {
      load_k(tile);
      if (V_AHEAD) load_v(tile);
    }
    pass(std::false_type(), again);
  } else {
    pass(std::false_type(), ~0u);
  }
}

template <typename E, int D, int G, int MODE, int NW, bool PIECES, bool OWN>
hipError_t launch_own(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb,
                      int n_groups, hipStream_t stream) {
  const int Tq = (pb.N + pb.Br - 1) / pb.Br, Tw = (pb.N + kTile - 1) / kTile;
  hipLaunchKernelGGL((attn_f32_kernel<E, D, G, MODE, NW, PIECES, OWN>), dim3((unsigned)((long long)pb.B * pb.H * Tw)), dim3(NW * 64), 0, stream,
                     (const E*)q, (const E*)k, (const E*)v, (E*)o, perm, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq, Tw, n_groups,
                     pb.causal, pb.scale, pb.Bc, pb.lse, pb.perm_w, pb.n_planes, pb.gray_mode, pb.seed);
  return hipGetLastError();
}

template <typename E, int D, int G, int MODE, int NW, bool PIECES>
hipError_t launch_one(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb,
                      int n_groups, hipStream_t stream) {
  if constexpr (std::is_same<E, float>::value && D == 64 && (MODE == kQueryFull || MODE == kQueryFused)) {
    if (pb.group_in_kernel) return launch_own<E, D, G, MODE, NW, PIECES, true>(q, k, v, o, nullptr, pb, n_groups, stream);
  }
  return launch_own<E, D, G, MODE, NW, PIECES, false>(q, k, v, o, perm, pb, n_groups, stream);
}

// Eight waves per workgroup where the row tiles leave compute units idle and there are tiles for all of them (dealt out by K blocks
// in the mirrored form): two waves per SIMD, as two workgroups would be; with more row tiles than compute units two workgroups of
// four have fewer states to merge. At d = 128 a wave's registers fill its SIMD. us, 4 | 8 waves, exact, groups of two, mirrored:
//   H1 N2048 40.9 | 38.2, 44.3 | 38.1, 51.6 | 41.6; H8 N1024 causal 24.0 | 23.1, 27.5 | 25.3, 29.5 | 25.4
//   H4 N521 16.4 | 15.7, 20.6 | 19.2, 21.3 | 19.1; 8 key tiles (H1 N256) 8.9 | 9.2, 12.6 | 12.7; H8 N1500 57.5 | 60.0
template <typename E, int D, int G, int MODE>
hipError_t launch_waves(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb, int n_groups,
                        hipStream_t stream) {
  constexpr bool kFused = MODE == kQueryFused || MODE == kKeyFused;
  const int tiles = (pb.Nk + kTile - 1) / kTile, TB = MODE == kKeyFull || MODE == kKeyFused ? pb.Bc / kTile : 1;
  const bool wide = D == 64 && (long long)pb.B * pb.H * ((pb.N + kTile - 1) / kTile) <= kComputeUnits && tiles > 8 && (tiles + TB - 1) / TB > 4;
  if constexpr (kFused && (D == 64 || MODE == kKeyFused)) {
    if (float_by_pieces(pb)) {
      if constexpr (D == 64) {
        if (wide) return launch_one<E, D, G, MODE, 8, true>(q, k, v, o, perm, pb, n_groups, stream);
      }
      return launch_one<E, D, G, MODE, 4, true>(q, k, v, o, perm, pb, n_groups, stream);
    }
  } else if constexpr (D == 64) {
    if (wide) return launch_one<E, D, G, MODE, 8, false>(q, k, v, o, perm, pb, n_groups, stream);
  }
  return launch_one<E, D, G, MODE, 4, false>(q, k, v, o, perm, pb, n_groups, stream);
}

template <typename E, int D>
hipError_t launch_typed(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb,
                        int distr, hipStream_t stream) {
  if ((long long)pb.B * pb.H * ((pb.N + kTile - 1) / kTile) > 0x7fffffffLL) return hipErrorInvalidValue;
  const int G = distr ? D / pb.n_groups : 1;
  if (distr && pb.side == 1) {
    if (G == 2) return launch_waves<E, D, 2, kKeyFused>(q, k, v, o, perm, pb, pb.n_groups, stream);
    if (G == 4) return launch_waves<E, D, 4, kKeyFused>(q, k, v, o, perm, pb, pb.n_groups, stream);
    return launch_waves<E, D, 1, kKeyFull>(q, k, v, o, perm, pb, pb.n_groups, stream);
  }
  if constexpr (std::is_same<E, float>::value) {
    if (!distr) return launch_waves<E, D, 1, kQueryFull>(q, k, v, o, nullptr, pb, D, stream);
    if (G == 2) return launch_waves<E, D, 2, kQueryFused>(q, k, v, o, perm, pb, pb.n_groups, stream);
    if (G == 4) return launch_waves<E, D, 4, kQueryFused>(q, k, v, o, perm, pb, pb.n_groups, stream);
    return launch_waves<E, D, 1, kQueryFull>(q, k, v, o, perm, pb, pb.n_groups, stream);
  }
  return hipErrorInvalidValue;   // bf16 tensors take this path for the mirrored form only
}

}  // namespace

// Grouping by the float kernel itself instead of a kernel in front of it: at d = 64, where every workgroup has a compute unit to
// itself, so that its LDS and the grouping, repeated by the workgroups of a Q block, cost nothing but their time, which K and V of the first
// tiles travel in. us, LSH kernel | itself, groups of two: H1 N64 9.9 | 8.4, H1 N256 (4 projections) 12.4 | 10.6, H4 N200 causal 13.5 | 11.5,
// H8 N700 causal 18.4 | 16.0, H8 N1000 22.2 | 21.1, H2 N2000 30.6 | 29.2. At d = 128 (twice the channels for four waves, which
// the LSH kernel gives eight) it loses: H2 N100 16.4 | 21.9, H4 N2000 89 | 96. Blocks of 256 rows, 16 projections: H1 N256 17.2 | 16.1,
// H4 N300 17.6 | 17.3, H8 N1000 25.5 | 24.5, H2 N4000 60.6 | 59.2. More than 16 projections walk the block's rows once more, 32 of them: H1 N256 Br256
// 24.1 | 22.7, H8 N1000 32.4 | 32.1, Br64 H4 N300 14.9 | 14.3, but Br128 H8 N300 17.5 | 17.6, groups of eight H4 N500 Br256 29.6 | 30.2: no line of their own,
// as a call that groups itself needs no room for a table.
bool attn_f32_groups(const Problem& pb, int dtype) {
  return dtype == 1 && pb.side == 0 && pb.d == 64 && (long long)pb.B * pb.H * ((pb.N + kTile - 1) / kTile) <= kComputeUnits;
}

// dtype 0: bf16 tensors (converted on load, rounded on store), 1: float tensors; float arithmetic either way
hipError_t launch_attn_f32(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                           const Problem& pb, int dtype, int distr, hipStream_t stream) {
  if (pb.d == 64)
    return dtype == 0 ? launch_typed<bf16, 64>(q, k, v, o, perm, pb, distr, stream)
                      : launch_typed<float, 64>(q, k, v, o, perm, pb, distr, stream);
  if (pb.d == 128)
    return dtype == 0 ? launch_typed<bf16, 128>(q, k, v, o, perm, pb, distr, stream)
                      : launch_typed<float, 128>(q, k, v, o, perm, pb, distr, stream);
  return hipErrorInvalidValue;
}

}  // namespace da
