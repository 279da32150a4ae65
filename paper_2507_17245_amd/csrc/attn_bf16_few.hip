// bf16 attention forward (exact and DistrAttention) for few query rows against many keys: decoding.
//
// Bound: reading K and V once. The general kernel gives every (query head, Q block) a workgroup whose
// waves own 32 query rows each; with one row per head 31 of 32 of its matrix work is padding, the
// query heads of a kv head read the same keys one by one, and a head's keys are walked by one wave.
// Here:
//   * the rows of all query heads of a kv head are one run of rows of q; a workgroup takes 32 of them
//     (grouped heads share every tile) and a share of the keys;
//   * its four waves deal the key tiles of the share out among themselves. A wave loads its own tiles
//     (direct global->LDS loads, 8 KB of K and of V, one tile ahead) and has a softmax state of its
//     own: no barrier in the loop, 64 KB in flight per compute unit, which covers the memory latency
//     at the full rate. The states meet in LDS at the end, the shares in the combine kernel;
//   * DistrAttention is taken as S^ = Q~ K^T (ScoreMode kReplicated): no transposed copy of the
//     cache. The grouping of a head's N <= 64 rows (one Q block) is computed by the workgroup, in the
//     defining float order, while its first tiles travel (behind barriers that wait for LDS alone: with __syncthreads, which
//     waits for the tiles too, a decoding call took 14.2 us, 13.0 now); hash and channel rank as one key.
// Layouts, operands and the rounding of P are the general kernel's (attn_bf16_impl.h).
// Measured (B1 H32 Hkv8 N1 Nk16384 d64, 34 MB of keys and values): 10 us + 3 us for the combine kernel, 130 us +
// 7 us for the key pre-pass before; B16 H32 Hkv4 N1 Nk8192: 33 us, 4.1 TB/s (174 us). (The last share of a row tile to end as the one that
// adds them up, by stores and loads past the L2 and a counter: 16.2 us; the start of a kernel costs less.)
#include <cfloat>

#include "attn_bf16_impl.h"

namespace da {

namespace {

constexpr int kFewRows = 32, kFewWaves = 4, kFewThreads = kFewWaves * 64;
constexpr int kFewTileBytes = 8192;   // of K, and of V, per wave and buffer

template <int D, bool GROUPED>
__global__ __launch_bounds__(kFewThreads, 2) void attn_bf16_few_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, bf16* __restrict__ o,
    const uint8_t* __restrict__ perm, uint8_t* __restrict__ perm_w, int H, int Hkv, int N, int Nk, int n_groups,
    int causal, float scale_log2e, int n_planes, int gray_mode, uint64_t lsh_seed, float* __restrict__ lse, int RT,
    int n_split, float* __restrict__ part_o, f32x2* __restrict__ part_stat) {
  constexpr int ROWB = D * 2, CH = D / 8, KT = kFewTileBytes / ROWB;   // keys per tile: 64 (d = 64), 32 (d = 128)
  constexpr int MB = KT / 32, TT = KT / 16, KS = D / 16, NMB = D / 32;
  constexpr int CPT = kFewTileBytes / 1024;                            // direct loads per tile
  // One object per buffer: reads of one do not wait for loads in flight into the other.
  __shared__ __attribute__((aligned(1024))) char k_lds0[kFewWaves][kFewTileBytes];
  __shared__ __attribute__((aligned(1024))) char k_lds1[kFewWaves][kFewTileBytes];
  __shared__ __attribute__((aligned(1024))) char v_lds0[kFewWaves][kFewTileBytes];
  __shared__ __attribute__((aligned(1024))) char v_lds1[kFewWaves][kFewTileBytes];
  __shared__ __attribute__((aligned(16))) bf16 q_lds[kFewRows][D + 8];
  __shared__ f32x2 stat_lds[kFewWaves][kFewRows];
  // grouping, for every head that has a row here
  __shared__ uint8_t perm_lds[GROUPED ? kFewRows : 1][GROUPED ? D : 1];
  __shared__ uint8_t from_lds[GROUPED ? kFewRows : 1][GROUPED ? D : 1];
  __shared__ float R_lds[GROUPED ? 64 * 16 : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const int units = gridDim.x / n_split;
  const int unit = blockIdx.x % units, part = blockIdx.x / units;
  const int bk = unit / RT, rt = unit % RT;          // b * Hkv + hk, row tile of the kv head
  const int rep = H / Hkv, rows = rep * N;           // rows of the kv head
  const size_t row0 = (size_t)bk * rows;             // its first row of q and o
  const int m0 = rt * kFewRows;
  const int m = m0 + lq, m_ld = min(m, rows - 1);    // this lane's row (surplus rows: a valid one, never stored)
  const int head0 = m0 / N, n_heads = min(rows - 1, m0 + kFewRows - 1) / N - head0 + 1;   // heads with a row here
  const int shift = Nk - N;

  const int all_tiles = (Nk + KT - 1) / KT;
  const int t0 = (int)((long long)all_tiles * part / n_split), t1 = (int)((long long)all_tiles * (part + 1) / n_split);

  // Rows of Q for the operands; issued first: a wait for them must not wait for the tiles behind.
  constexpr int QU = kFewRows * CH / kFewThreads;
  bf16x8 qx[QU];
#pragma unroll
  for (int u = 0; u < QU; ++u) {
    const int i = u * kFewThreads + tid;
    qx[u] = *(const bf16x8*)(q + (row0 + min(m0 + i / CH, rows - 1)) * D + i % CH * 8);
  }

  const unsigned head_bytes = (unsigned)Nk * D * 2;
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(k + (size_t)bk * Nk * D), 0, head_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(v + (size_t)bk * Nk * D), 0, head_bytes, 0x00020000);
  int dma_k[CPT], dma_v[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int slot = j * 64 + lane, row = slot / CH, pc = slot % CH;
    dma_k[j] = row * ROWB + (pc ^ (D == 128 ? (row & 15) : ((row >> 1) & 7))) * 16;
    dma_v[j] = row * ROWB + ((((pc >> 1) ^ v_swizzle<ROWB>(row)) << 1) | (pc & 1)) * 16;
  }
  auto load_tile = [&](auto par_c, int tile) {
    typedef __attribute__((address_space(3))) void lds_void;
    char* kd = decltype(par_c)::value ? k_lds1[wave] : k_lds0[wave];
    char* vd = decltype(par_c)::value ? v_lds1[wave] : v_lds0[wave];
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (lds_void*)(kd + j * 1024), 16, dma_k[j], tile * kFewTileBytes, 0, 0);
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (lds_void*)(vd + j * 1024), 16, dma_v[j], tile * kFewTileBytes, 0, 0);
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
  int tile = t0 + wave;

  // ---- grouping (Sec. 3.2): one Q block per head, its N rows --------------------------------------
  if constexpr (GROUPED) {
    if (perm == nullptr) {
      for (int i = tid; i < N * 16; i += kFewThreads)
        R_lds[i] = (i & 15) < n_planes ? hyperplane_entry(lsh_seed, (uint32_t)(i & 15), (uint32_t)(i >> 4)) : 0.0f;
    } else {
      for (int i = tid; i < n_heads * D; i += kFewThreads)
        perm_lds[i / D][i % D] = perm[((size_t)bk * rep + head0) * D + i] & (D - 1);   // (see the general kernel)
    }
  }
#pragma unroll
  for (int u = 0; u < QU; ++u) {
    const int i = u * kFewThreads + tid;
    *(bf16x8*)&q_lds[i / CH][i % CH * 8] = qx[u];
  }
  if (tile < t1) load_tile(even, tile);
  // (barriers that leave the tiles in flight)
  if constexpr (GROUPED) {
    const int group = D / n_groups;
    uint32_t* keys = (uint32_t*)k_lds1;   // (receives its first tile after the barrier that ends this stage)
    static_assert(kFewRows * D * 4 <= kFewWaves * kFewTileBytes, "the keys of all heads fit");
    lds_barrier();
    if (perm == nullptr) {
      // signs of the float sums, one fused multiply-add per row, rows ascending, from +0
      for (int i = tid; i < n_heads * D; i += kFewThreads) {
        const int hd = head0 + i / D, c = i % D;
        float acc[16];
#pragma unroll
        for (int p = 0; p < 16; ++p) acc[p] = 0.0f;
        auto add_row = [&](float x, int r) {
#pragma unroll
          for (int p = 0; p < 16; ++p) acc[p] = __builtin_fmaf(x, R_lds[r * 16 + p], acc[p]);
        };
        const int mr = hd * N - m0;
        if (mr >= 0 && mr + N <= kFewRows) {
          for (int r = 0; r < N; ++r) add_row((float)q_lds[mr + r][c], r);
        } else {   // a head whose rows reach into other row tiles
          const bf16* col = q + (row0 + (size_t)hd * N) * D + c;
#pragma unroll 8
          for (int r = 0; r < N; ++r) add_row((float)col[(size_t)r * D], r);
        }
        uint32_t bits = 0;
#pragma unroll
        for (int p = 0; p < 16; ++p)
          if (p < n_planes && acc[p] > 0.0f) bits |= 1u << (n_planes - 1 - p);   // projection 0 = top bit
        keys[i] = lsh_hash_of_code(bits, gray_mode) << 7 | c;   // (at most 16 bits: hash and channel make one key)
      }
      lds_barrier();
      // rank by counting = stable ascending sort
      for (int i = tid; i < n_heads * D; i += kFewThreads) {
        const uint32_t* others = keys + i / D * D;
        const uint32_t mine = keys[i];
        int rank = 0;
#pragma unroll 8
        for (int o4 = 0; o4 < D; o4 += 4) {
          const u32x4 other = *(const u32x4*)&others[o4];
#pragma unroll
          for (int j = 0; j < 4; ++j) rank += other[j] < mine ? 1 : 0;
        }
        perm_lds[i / D][rank] = (uint8_t)(i % D);
      }
      lds_barrier();
      if (perm_w && part == 0)
        for (int i = tid; i < n_heads * D; i += kFewThreads) perm_w[((size_t)bk * rep + head0) * D + i] = perm_lds[i / D][i % D];
    }
    for (int i = tid; i < n_heads * D; i += kFewThreads) {
      const uint8_t* pl = perm_lds[i / D];
      from_lds[i / D][pl[i % D]] = pl[i % D / group * group];
    }
  }
  lds_barrier();
  bf16x8 qop[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if constexpr (GROUPED) {
      const uint8_t* fl = from_lds[m_ld / N - head0];
#pragma unroll
      for (int j = 0; j < 8; ++j) qop[s][j] = q_lds[lq][fl[16 * s + 8 * hh + j] & (D - 1)];
    } else {
      qop[s] = *(const bf16x8*)&q_lds[lq][16 * s + 8 * hh];
    }
  }

  // ---- the wave's key tiles -----------------------------------------------------------------------
  int ka_off[KS], va_off[NMB];
#pragma unroll
  for (int s = 0; s < KS; ++s) ka_off[s] = lq * ROWB + ((2 * s + hh) ^ (D == 128 ? (lq & 15) : ((lq >> 1) & 7))) * 16;
  {
    const int row_l = 4 * hh + ((lane & 15) >> 2);
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
      va_off[mb] = row_l * ROWB + ((2 * mb + ((lane >> 4) & 1)) ^ v_swizzle<ROWB>(row_l)) * 32 + 8 * (lane & 3);
  }
  f32x16 oacc[NMB];
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[mb][i] = 0.0f;
  // The reference is the largest score so far, unscaled like the scores until their difference is taken: exact
  // however large they are (a scaled reference is a rounded one; with scores of 1e10 P came out as 0 or infinity).
  float ref = -FLT_MAX, l_run = 0.0f;   // the sum is over this lane's half of the keys
  const int lim = causal ? m_ld % N + shift : Nk - 1;   // last key this row sees

  auto step = [&](auto par_c, int t) {
    constexpr int par = decltype(par_c)::value;
    const char* kb = par ? k_lds1[wave] : k_lds0[wave];
    const char* vb = par ? v_lds1[wave] : v_lds0[wave];
    // the next tile into the other buffer, whose reads are done; then this tile has to be there
    if (t + kFewWaves < t1) {
      load_tile(std::integral_constant<int, par ^ 1>(), t + kFewWaves);
      asm volatile("s_waitcnt vmcnt(%0)" ::"i"(2 * CPT) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    f32x16 sc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[mb][i] = 0.0f;
#pragma unroll
      for (int s = 0; s < KS; ++s) sc[mb] = mfma_32x32x16(*(const bf16x8*)(kb + ka_off[s] + mb * 32 * ROWB), qop[s], sc[mb]);
    }
    const int n0 = t * KT;
    if (n0 + KT > (causal ? shift + 1 : Nk)) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (n0 + 32 * mb + 8 * (i >> 2) + 4 * hh + (i & 3) > lim) sc[mb][i] = -INFINITY;
    }
    float mx = sc[0][0];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[mb][i]);
    const float ref_new = fmaxf(ref, half_swap_max(mx));
    if (__builtin_amdgcn_ballot_w64(ref_new > ref) != 0) {
      const float alpha = __builtin_amdgcn_exp2f((ref - ref_new) * scale_log2e);
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mb][i] *= alpha;
      ref = ref_new;
    }
    // P rounded to bf16 as the operands of P.V; the row sum is taken over the rounded values
    bf16x8 pop[TT];
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const bf16x2 pr = {(bf16)__builtin_amdgcn_exp2f((sc[mb][i] - ref) * scale_log2e),
                           (bf16)__builtin_amdgcn_exp2f((sc[mb][i + 1] - ref) * scale_log2e)};
        pop[mb * 2 + (i >> 3)][i & 7] = pr[0];
        pop[mb * 2 + (i >> 3)][(i & 7) + 1] = pr[1];
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l_run, false);
      }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        const char* p0 = vb + va_off[mb] + 16 * tt * ROWB;
        oacc[mb] = mfma_32x32x16(lds_read_tr_pair<bf16x8>(p0, p0 + 8 * ROWB), pop[tt], oacc[mb]);
      }
  };
  while (tile < t1) {
    step(even, tile);
    tile += kFewWaves;
    if (tile >= t1) break;
    step(odd, tile);
    // Where the loop ends the compiler waits for these products by its longest way out; on the shortest their sums would be
    // read two instructions early.
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");
    tile += kFewWaves;
  }

  // ---- the waves' states meet ------------------------------------------------------------------------
  const float l_tot = half_swap_sum(l_run);
  if (hh == 0) stat_lds[wave][lq] = f32x2{ref, l_tot};
  __syncthreads();   // also: nobody reads tiles any more
  float ref_all = stat_lds[0][lq][0], l_all = 0.0f;
#pragma unroll
  for (int j = 1; j < kFewWaves; ++j) ref_all = fmaxf(ref_all, stat_lds[j][lq][0]);
#pragma unroll
  for (int j = 0; j < kFewWaves; ++j) l_all += stat_lds[j][lq][1] * __builtin_amdgcn_exp2f((stat_lds[j][lq][0] - ref_all) * scale_log2e);
  const float weight = __builtin_amdgcn_exp2f((ref - ref_all) * scale_log2e) * (n_split > 1 ? 1.0f : 1.0f / l_all);
  // wave w's sums: 32 rows of D floats, the 16-byte pieces exchanged by the row (its own buffers: K at
  // d = 64, K and V at d = 128)
  float* half0 = (float*)k_lds0[wave];
  float* half1 = (float*)(D == 128 ? v_lds0[wave] : k_lds0[wave]);
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const int piece = 8 * mb + 2 * i4 + hh;   // channels 4*piece ..
      float* dst = mb < 2 ? half0 : half1;
      const f32x4 x = {oacc[mb][4 * i4] * weight, oacc[mb][4 * i4 + 1] * weight, oacc[mb][4 * i4 + 2] * weight, oacc[mb][4 * i4 + 3] * weight};
      *(f32x4*)&dst[lq * 64 + (((piece & 15) ^ (lq & 15)) << 2)] = x;
    }
  __syncthreads();
  auto finish = [&](const char (*sums)[kFewTileBytes], int c0) {   // 64 channels from c0 on
#pragma unroll
    for (int i = tid; i < kFewRows * 16; i += kFewThreads) {
      const int row = i / 16, piece = i % 16;
      if (m0 + row >= rows) continue;
      f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int j = 0; j < kFewWaves; ++j) x += *(const f32x4*)((const float*)sums[j] + row * 64 + ((piece ^ (row & 15)) << 2));
      const size_t at = (row0 + m0 + row) * D + c0 + piece * 4;
      if (n_split > 1) {
        *(f32x4*)(part_o + (size_t)part * (units / RT) * rows * D + at) = x;
      } else {
        const bf16x4 y = {(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
        *(bf16x4*)(o + at) = y;
      }
    }
  };
  finish(k_lds0, 0);
  if constexpr (D == 128) finish(v_lds0, 64);
  if (wave == 0 && hh == 0 && m < rows) {
    if (n_split > 1) part_stat[(size_t)part * (units / RT) * rows + row0 + m] = f32x2{ref_all * scale_log2e, l_all};
    else if (lse) lse[row0 + m] = 0.6931471805599453f * (ref_all * scale_log2e + __builtin_log2f(l_all));
  }
}

template <int D>
hipError_t launch_d(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb, int distr,
                    hipStream_t stream) {
  const int RT = (pb.H / pb.Hkv * pb.N + kFewRows - 1) / kFewRows;
  const dim3 grid((unsigned)((long long)pb.B * pb.Hkv * RT * pb.n_split)), block(kFewThreads);
  const float scale_log2e = pb.scale * 1.4426950408889634f;
#define DA_FEW(GR)                                                                                                         \
  hipLaunchKernelGGL((attn_bf16_few_kernel<D, GR>), grid, block, 0, stream, (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, \
                     perm, pb.perm_w, pb.H, pb.Hkv, pb.N, pb.Nk, pb.n_groups, pb.causal, scale_log2e, pb.n_planes, pb.gray_mode,  \
                     pb.seed, pb.lse, RT, pb.n_split, pb.part_o, (f32x2*)pb.part_stat)
  if (distr) DA_FEW(true);
  else DA_FEW(false);
#undef DA_FEW
  return hipGetLastError();
}

}  // namespace

// Where this kernel is the better one: H32 Hkv32 N32 Nk8192 d64 26 us against 28 with the general kernel (keys
// split there too), but N64 47 against 36 (two row tiles of one head read the keys twice); grouped heads
// win up to 128 rows (Hkv4 N16: 20 against 25; B8 Hkv4 N16 Nk2048 d128: 36 against 58). Below 256 keys there
// is no tile for every wave. Exact calls, whose workgroups of the general kernel start at once, need more than two tiles
// per wave (H16 N1 Nk512 d64 7.9 against 7.4, Nk1000 9.0 against 11.5; d128 Nk512 9.5 against 10.6) and, where no heads
// share their keys, no more workgroups than compute units (B16 H32 N1 Nk1000 d64 24.3 against 22.2).
bool attn_bf16_few_rows(const Problem& pb, int distr) {
  const int rep = pb.H / pb.Hkv;
  if (pb.N > 32 || (long long)rep * pb.N > 128 || pb.Nk < 256) return false;
  return distr || ((long long)pb.Nk * pb.d > 32768 && (rep > 1 || (long long)pb.B * pb.H <= 256));
}

// One workgroup per compute unit (the tiles in flight take its LDS), every wave at least one tile; undivided unless five
// tiles come off a wave's walk, which is what the combine kernel costs (H16 N1 d64, 1 | 16 and more shares: Nk1000 8.7 | 11.2 us,
// Nk1500 11.1 | 11.2, Nk2200 14.5 | 11.1; d128 Nk512 9.5 | 11.3, Nk1000 14.2 | 11.3).
int attn_bf16_few_splits(const Problem& pb) {
  const int RT = (pb.H / pb.Hkv * pb.N + kFewRows - 1) / kFewRows;
  const long long units = (long long)pb.B * pb.Hkv * RT;
  const int tile = kFewTileBytes / (pb.d * 2);
  const long long tiles = (pb.Nk + tile - 1) / tile;
  long long n = 256 / units;
  if (n > tiles / kFewWaves) n = tiles / kFewWaves;
  if (n < 2 || tiles - tiles / n < 20) n = 1;
  return (int)n;
}

hipError_t launch_attn_bf16_few(const void* q, const void* k, const void* v, void* o, const uint8_t* perm, const Problem& pb,
                                int distr, hipStream_t stream) {
  if ((long long)pb.B * pb.Hkv * ((pb.H / pb.Hkv * pb.N + kFewRows - 1) / kFewRows) * pb.n_split > 0x7fffffffLL) return hipErrorInvalidValue;
  return pb.d == 64 ? launch_d<64>(q, k, v, o, perm, pb, distr, stream) : launch_d<128>(q, k, v, o, perm, pb, distr, stream);
}

}  // namespace da
