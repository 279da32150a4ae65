// bf16 attention forward (exact and DistrAttention) of short sequences at d = 64: image-sized batches.
//
// Bound: reading Q, K, V and writing O once. The general kernel gives every Q block a workgroup of its own, which
// at a few tiles of keys is mostly a chain of dependent steps (rows, grouping, sampling, the first keys), paid for
// by every block, with a barrier per tile behind it. Here one workgroup takes a whole head:
//   * K and V are asked for at once by direct global->LDS loads and stay in LDS (64 KB: two workgroups, four waves per
//     SIMD). DistrAttention first has Q in V's place and the projection table in K's, and groups all Q blocks:
//     projections shared by all waves, then one wave ranks a block, which takes no further barrier;
//   * wave w owns the rows 32*w .. and walks the keys 32 at a time without a barrier, the scores of the next
//     32 keys on the matrix pipe beside the exponentials of these; causal waves stop at their last key;
//   * V travels behind K: the barrier after Q~ waits for LDS alone, and the first scores for K alone (H12 N197 B64 28.7 -> 27.4 us, exact
//     23.7 -> 23.0, where __syncthreads waited for K before V was asked for);
//   * DistrAttention is taken as S^ = Q~ K^T (ScoreMode kReplicated).
// Layouts, operands, rounding of P and the lazy reference are the general kernel's (attn_bf16_impl.h).
// Measured, general | this: H12 N197 B64 41 | 27 us (exact 29 | 21), B8 14.3 | 13.1, B1 13.0 | 12.0; N128 B64 23 | 15;
// N64 B64 12.1 | 11.1, B4 9.3 | 7.6; H32 Hkv8 causal N256 B16 exact 20 | 14.
#include "attn_bf16_impl.h"

namespace da {

namespace {

template <int NW, bool GROUPED>
__global__ __launch_bounds__(NW * 64, 4) void attn_bf16_short_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, bf16* __restrict__ o,
    const uint8_t* __restrict__ perm, uint8_t* __restrict__ perm_w, int H, int Hkv, int N, int Nk, int Br, int Tq,
    int n_groups, int causal, float scale_log2e, int n_planes, int gray_mode, uint64_t lsh_seed, float* __restrict__ lse) {
  constexpr int D = 64, ROWB = D * 2, CH = D / 8, KS = D / 16, T = NW * 64, ROWS = NW * 32;
  constexpr int RPAD = ROWS + 8;         // bf16 pieces of R: 16 lanes read 16 rows of the table at once
  constexpr int BLOCKS = ROWS / 64;      // most Q blocks of a head
  __shared__ __attribute__((aligned(1024))) char k_lds[ROWS * ROWB];   // the projection table, K, rows of O
  __shared__ __attribute__((aligned(1024))) char v_lds[ROWS * ROWB];   // Q, V
  __shared__ uint32_t code_lds[GROUPED ? BLOCKS : 1][D];
  __shared__ __attribute__((aligned(16))) uint32_t key_lds[GROUPED ? BLOCKS : 1][D];
  __shared__ uint8_t perm_lds[GROUPED ? BLOCKS : 1][D];
  __shared__ __attribute__((aligned(8))) uint8_t from_lds[GROUPED ? BLOCKS : 1][D];
  static_assert(2 * 16 * RPAD * 2 <= ROWS * ROWB, "the projection table fits K's place");

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  int bh = (int)blockIdx.x;              // heads of a kv head share an XCD's L2
  if ((gridDim.x & 7) == 0) bh = (bh & 7) * (int)(gridDim.x >> 3) + (bh >> 3);
  const int bk = bh / H * Hkv + bh % H / (H / Hkv);
  const int shift = Nk - N;

  // ---- loads into LDS, 1 KB per wave and load. Positions of a row's 16-byte chunks: Q and K chunk ^ (row / 2) % 8; V as
  // in the general kernel (32-byte segments). Rows past the end read as zeros.
  auto load = [&](auto v_c, const bf16* src, int rows, char* dst) {
    typedef __attribute__((address_space(3))) void lds_void;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, (unsigned)rows * ROWB, 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int slot = (j * NW + wave) * 64 + lane, row = slot / CH, pc = slot % CH;
      const int chunk = decltype(v_c)::value ? (((pc >> 1) ^ v_swizzle<ROWB>(row)) << 1) | (pc & 1) : pc ^ ((row >> 1) & 7);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + (j * NW + wave) * 1024), 16, row * ROWB + chunk * 16, 0, 0, 0);
    }
  };
  const std::true_type as_v;
  const std::false_type as_k;
  const bf16* qh = q + (size_t)bh * N * D;
  const bf16* kh = k + (size_t)bk * Nk * D;
  const bf16* vh = v + (size_t)bk * Nk * D;
  auto landed = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  const int my_row = wave * 32 + lq;
  bf16x8 qop[KS];
  if constexpr (GROUPED) {
    const int group = D / n_groups;
    auto q_at = [&](int row, int chunk) -> const char* { return v_lds + row * ROWB + ((chunk ^ ((row >> 1) & 7)) << 4); };
    load(as_k, qh, N, v_lds);
    if (perm != nullptr) {
      load(as_k, kh, Nk, k_lds);
#pragma unroll 1
      for (int i = tid; i < Tq * D; i += T) perm_lds[i / D][i % D] = perm[(size_t)bh * Tq * D + i] & (D - 1);
      landed();
#pragma unroll 1
      for (int i = tid; i < Tq * D; i += T) {
        const uint8_t* pl = perm_lds[i / D];
        from_lds[i / D][pl[i % D]] = (uint8_t)(2 * pl[i % D / group * group]);
      }
    } else {
      // ---- LSH hash-and-group of the head's Q blocks: the general kernel's stage (same bound, same tables)
      bf16* rp1 = (bf16*)k_lds;
      bf16* rp2 = rp1 + 16 * RPAD;
      const int rr = min(Br, ROWS);      // rows of a block that can exist (a power of two)
      const int rr_log = 31 - __builtin_clz(rr);
#pragma unroll 1
      for (int i = tid; i < rr * 16; i += T) {
        const int r = i & (rr - 1), pl = i >> rr_log;
        const float rv = pl < n_planes ? hyperplane_entry(lsh_seed, (uint32_t)pl, (uint32_t)r) : 0.0f;
        const bf16 r1 = (bf16)rv;
        rp1[pl * RPAD + r] = r1;
        rp2[pl * RPAD + r] = (bf16)(rv - (float)r1);
      }
      landed();
      const int pl16 = lane & 15, kg = lane >> 4;
      const float doubt_rel = 3.1e-7f * rr, kTiny = 1e-30f;
#pragma unroll 1
      for (int task = wave; task < Tq * (D / 16); task += NW) {
        const int blk = task / (D / 16), ct = task % (D / 16), b0 = blk * Br;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, bnd = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int ks = 0; ks < rr / 32; ks += 2) {
          s16x8 a[2], b1[2], b2[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int row = 32 * (ks + j) + 8 * kg, chunk = 2 * ct + ((pl16 & 3) >> 1), inch = 8 * (pl16 & 1);
            const int row0 = b0 + row + (pl16 >> 2);
            a[j] = lds_read_tr_pair<s16x8>(q_at(row0, chunk) + inch, q_at(row0 + 4, chunk) + inch);
            b1[j] = *(const s16x8*)&rp1[pl16 * RPAD + row];
            b2[j] = *(const s16x8*)&rp2[pl16 * RPAD + row];
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j]), __builtin_bit_cast(bf16x8, b1[j]), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j]), __builtin_bit_cast(bf16x8, b2[j]), acc, 0, 0, 0);
            bnd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j] & (short)0x7fff),
                                                          __builtin_bit_cast(bf16x8, b1[j] & (short)0x7fff), bnd, 0, 0, 0);
          }
        }
        bool positive[4], doubt[4], any_doubt = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          positive[i] = acc[i] > 0.0f;
          doubt[i] = pl16 < n_planes && !(__builtin_fabsf(acc[i]) > doubt_rel * bnd[i] + kTiny);
          any_doubt |= doubt[i];
        }
        if (__builtin_amdgcn_ballot_w64(any_doubt) != 0)
          settle_doubts(doubt, positive, rr, rp1, rp2, RPAD, [&, block = (const char*)v_lds + b0 * ROWB](int row, int ch) {
            return *(const bf16*)(block + row * ROWB + (((2 * ct + (ch >> 3)) ^ ((row >> 1) & 7)) << 4) + (ch & 7) * 2);
          });
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint64_t signs = __builtin_amdgcn_ballot_w64(positive[i]);
          if (pl16 == 0)
            code_lds[blk][16 * ct + 4 * kg + i] = __builtin_bitreverse32((uint32_t)(signs >> (16 * kg)) & 0xffffu) >> (32 - n_planes);
        }
      }
      __syncthreads();
      if (wave < Tq) {
        // Lane = channel. Rank by counting = stable ascending sort (hashes have at most 16 bits: hash and channel make
        // one key). The wave's LDS accesses take effect in its order.
        const uint32_t mine = lsh_hash_of_code(code_lds[wave][lane], gray_mode) << 6 | lane;
        key_lds[wave][lane] = mine;
        __builtin_amdgcn_wave_barrier();
        int rank = 0;
#pragma unroll 4
        for (int c4 = 0; c4 < D; c4 += 4) {
          const u32x4 other = *(const u32x4*)&key_lds[wave][c4];
#pragma unroll
          for (int j = 0; j < 4; ++j) rank += other[j] < mine ? 1 : 0;
        }
        perm_lds[wave][rank] = (uint8_t)lane;
        __builtin_amdgcn_wave_barrier();
        const uint8_t c = perm_lds[wave][lane];
        if (perm_w != nullptr) perm_w[((size_t)bh * Tq + wave) * D + lane] = c;
        from_lds[wave][c] = (uint8_t)(2 * perm_lds[wave][lane / group * group]);
      }
    }
    __syncthreads();
    if (perm == nullptr) load(as_k, kh, Nk, k_lds);
    // Q~: the sampled channel of every channel's group
    // (from_lds holds byte offsets inside a row; chunk ^ x is offset ^ 16 x, for four of them at once)
    const uint8_t* from = from_lds[min(wave * 32 / Br, Tq - 1)];
    const uint32_t swz = ((my_row >> 1) & 7) * 0x10101010u;
    const char* row = v_lds + my_row * ROWB;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x2 f = *(const u32x2*)&from[16 * s + 8 * hh];
      f[0] = (f[0] & 0x7e7e7e7eu) ^ swz;
      f[1] = (f[1] & 0x7e7e7e7eu) ^ swz;
#pragma unroll
      for (int j = 0; j < 8; ++j) qop[s][j] = *(const bf16*)(row + ((f[j >> 2] >> (8 * (j & 3))) & 255));
    }
    lds_barrier();                       // Q has been read; K travels on
    load(as_v, vh, Nk, v_lds);
  } else {
#pragma unroll
    for (int s = 0; s < KS; ++s) qop[s] = *(const bf16x8*)(qh + (size_t)min(my_row, N - 1) * D + 16 * s + 8 * hh);
    load(as_k, kh, Nk, k_lds);
    load(as_v, vh, Nk, v_lds);
  }
  // K has landed (V, whose four loads are the last, is awaited behind the first scores)
  asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  lds_barrier();
  const int qw0 = wave * 32, q_abs = qw0 + lq;

  // ---- 32 keys at a time
  int ka_off[KS], va_off[2];
#pragma unroll
  for (int s = 0; s < KS; ++s) ka_off[s] = lq * ROWB + ((2 * s + hh) ^ ((lq >> 1) & 7)) * 16;
  {
    const int row_l = 4 * hh + ((lane & 15) >> 2);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
      va_off[mb] = row_l * ROWB + ((2 * mb + ((lane >> 4) & 1)) ^ v_swizzle<ROWB>(row_l)) * 32 + 8 * (lane & 3);
  }
  const int n_end = causal ? min(Nk, qw0 + 32 + shift) : Nk;
  const int n_blocks = qw0 < N ? (n_end + 31) / 32 : 0;              // (no rows: no keys either)
  const int lim = causal ? min(q_abs + shift, Nk - 1) : Nk - 1;      // last key this row sees
  const int n_free = causal ? min(qw0 + shift + 1, Nk) : Nk;         // keys every row of the wave sees
  f32x16 oacc[2];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[mb][i] = 0.0f;
  float nref = 0.0f, l_run = 0.0f;       // negated reference (exp2 domain); sum over this lane's half of the keys

  auto scores = [&](int b, f32x16& sc) {
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) sc = mfma_32x32x16(*(const bf16x8*)(k_lds + b * 32 * ROWB + ka_off[s]), qop[s], sc);
  };
  auto mask = [&](int b, f32x16& sc) {
    if (b * 32 + 32 > n_free) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (b * 32 + 8 * (i >> 2) + 4 * hh + (i & 3) > lim) sc[i] = -INFINITY;
    }
  };
  auto block_max = [&](const f32x16& sc) {   // relative to the reference
    float mx = sc[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
    return __builtin_fmaf(half_swap_max(mx), scale_log2e, nref);
  };
  auto exponentials = [&](const f32x16& sc, bf16x8 (&pop)[2]) {
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
    float rs0 = 0.0f, rs1 = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const bf16x2 pr = {(bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], scale_log2e, nref)),
                         (bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[i + 1], scale_log2e, nref))};
      pop[i >> 3][i & 7] = pr[0];
      pop[i >> 3][(i & 7) + 1] = pr[1];
      if (i & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs1, false);
      else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs0, false);
    }
    return rs0 + rs1;
  };
  auto body = [&](auto have_next, int b, f32x16& sc, f32x16& sn) {
    if (!decltype(have_next)::value && b + 1 < n_blocks) scores(b + 1, sn);
    bf16x8 va[2][2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const char* p0 = v_lds + (b * 32 + 16 * tt) * ROWB + va_off[mb];
        va[tt][mb] = lds_read_tr_pair<bf16x8>(p0, p0 + 8 * ROWB);
      }
    bf16x8 pop[2];
    float rs = exponentials(sc, pop);
    if (__builtin_amdgcn_ballot_w64(!(rs <= 16 * 256.0f)) != 0) {
      // a score more than kTau above its row's reference (16 keys per lane): the reference moves up
      const float mt = block_max(sc), delta = mt > kTau ? mt : 0.0f, alpha = __builtin_amdgcn_exp2f(-delta);
      nref -= delta;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mb][i] *= alpha;
      rs = exponentials(sc, pop);
    }
    l_run += rs;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) oacc[mb] = mfma_32x32x16(va[tt][mb], pop[tt], oacc[mb]);
    if (!decltype(have_next)::value && b + 1 < n_blocks) mask(b + 1, sn);
  };
  // The first reference is the maximum over 64 keys, as in the general kernel (over 32, P exceeds 1 more often and its
  // rounding grows: relative error 2.24e-3 instead of 2.21e-3 at H12 N197). Key 0 is visible to every row, but its score, and
  // those of the next keys, can be minus infinity: such rows take the first maximum that is finite.
  f32x16 s0, s1;
  scores(0, s0);
  mask(0, s0);
  float first = block_max(s0);
  if (n_blocks > 1) {
    scores(1, s1);
    mask(1, s1);
    first = fmaxf(first, block_max(s1));
  }
  for (int b = 2; b < n_blocks && __builtin_amdgcn_ballot_w64(first == -INFINITY) != 0; ++b) {
    f32x16 later;
    scores(b, later);
    mask(b, later);
    first = first == -INFINITY ? block_max(later) : first;
  }
  nref = first == -INFINITY ? 0.0f : -first;
  landed();
  if (n_blocks > 0) body(std::true_type(), 0, s0, s1);
  for (int b = 1; b < n_blocks; b += 2) {
    body(std::false_type(), b, s1, s0);
    if (b + 1 < n_blocks) body(std::false_type(), b + 1, s0, s1);
  }

  // ---- O by way of LDS, whole rows to memory
  __syncthreads();                       // K has been read
  const float l_tot = half_swap_sum(l_run), inv = 1.0f / l_tot;
  if (lse && q_abs < N && hh == 0) lse[(size_t)bh * N + q_abs] = 0.6931471805599453f * (__builtin_log2f(l_tot) - nref);
  char* out = k_lds + qw0 * ROWB;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      bf16x4 y;
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = (bf16)(oacc[mb][4 * i4 + j] * inv);
      *(bf16x4*)(out + lq * ROWB + (((4 * mb + i4) ^ (lq & 7)) << 4) + 8 * hh) = y;
    }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = u * 8 + lane / CH, chunk = lane % CH;
    const u32x4 x = *(const u32x4*)(out + row * ROWB + ((chunk ^ (row & 7)) << 4));
    if (qw0 + row < N) *(u32x4*)(o + ((size_t)bh * N + qw0 + row) * D + chunk * 8) = x;
  }
}

}  // namespace

// What the LDS holds. Exact, with fewer heads than compute units, the general kernel's Q blocks spread further
// (H12 N197 B1: 6.6 | 7.3 us).
bool attn_bf16_short(const Problem& pb, int distr) {
  return pb.d == 64 && pb.N <= 256 && pb.Nk <= 256 && !attn_bf16_few_rows(pb, distr) && (distr || (long long)pb.B * pb.H >= 256);
}

hipError_t launch_attn_bf16_short(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb,
                                  int distr, hipStream_t stream) {
  const long long units = (long long)pb.B * pb.H;
  if (units > 0x7fffffffLL || !attn_bf16_short(pb, distr)) return hipErrorInvalidValue;
  const int Tq = (pb.N + pb.Br - 1) / pb.Br;
  const float scale_log2e = pb.scale * 1.4426950408889634f;
#define DA_SHORT(NW, GR)                                                                                               \
  hipLaunchKernelGGL((attn_bf16_short_kernel<NW, GR>), dim3((unsigned)units), dim3(NW * 64), 0, stream, (const bf16*)q, \
                     (const bf16*)k, (const bf16*)v, (bf16*)o, perm, pb.perm_w, pb.H, pb.Hkv, pb.N, pb.Nk, pb.Br, Tq,   \
                     pb.n_groups, pb.causal, scale_log2e, pb.n_planes, pb.gray_mode, pb.seed, pb.lse)
  const int rows = pb.N > pb.Nk ? pb.N : pb.Nk;
  if (rows <= 64 && distr) DA_SHORT(2, true);
  else if (rows <= 64) DA_SHORT(2, false);
  else if (rows <= 128 && distr) DA_SHORT(4, true);
  else if (rows <= 128) DA_SHORT(4, false);
  else if (distr) DA_SHORT(8, true);
  else DA_SHORT(8, false);
#undef DA_SHORT
  return hipGetLastError();
}

}  // namespace da
