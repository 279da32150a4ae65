// Entry of the bf16 attention kernels: which shapes are built, and the dispatch over the K/V tile
// size (one translation unit per tile size: attn_bf16_bc32/64/128.hip, kernel in attn_bf16_impl.h).
#include <algorithm>

#include "da_common.h"

namespace da {

hipError_t launch_attn_bf16_bc32(const void*, const void*, const void*, void*, const uint8_t*, const void*,
                                 const Problem&, int, hipStream_t);
hipError_t launch_attn_bf16_bc64(const void*, const void*, const void*, void*, const uint8_t*, const void*,
                                 const Problem&, int, hipStream_t);
hipError_t launch_attn_bf16_bc128(const void*, const void*, const void*, void*, const uint8_t*, const void*,
                                  const Problem&, int, hipStream_t);

bool attn_bf16_supported(const Problem& pb, int distr) {
  if (pb.d != 64 && pb.d != 128) return false;
  if (pb.Br != 64 && pb.Br != 128 && pb.Br != 256) return false;
  if (pb.Bc != 32 && pb.Bc != 64 && pb.Bc != 128) return false;
  if (distr) {
    // groups of up to 16 channels (G* in {1, 2, 4, 8, 16}, Sec. 3.2 and Table 4); K/V tiles other
    // than 64 rows are built for 16, 32 and 64 groups
    const int kr = pb.n_groups;
    if (kr > pb.d || pb.d % kr != 0 || pb.d / kr > 16) return false;
    if (kr == pb.d) return true;
    if (kr != 4 && kr != 8 && kr != 16 && kr != 32 && kr != 64) return false;
    if (pb.Bc != 64 && kr < 16) return false;
  }
  return true;
}

// Query rows that see a key, masked ones taken off.
static double visible_rows(const Problem& pb) {
  return (double)(pb.H / pb.Hkv) * pb.N * (pb.causal ? 1.0 - 0.5 * pb.N / pb.Nk : 1.0);
}

// The transposed copy's bytes and launch against a seventh of the whole product, 1570 visible rows per key.
bool attn_bf16_light(const Problem& pb) {
  return visible_rows(pb) < 1570.0 + 7.8e9 / ((double)pb.d * pb.B * pb.Hkv * pb.Nk);
}

// Q~ K^T (see ScoreMode in attn_bf16_impl.h) instead of Q_r K_f^T where the transposed copy of K costs more than the
// shorter contraction saves. The copy: its launch (4.5 us) and 0.35 us per million elements. The saving: `gain` us per
// 10^9 (visible pairs times channels), by the group size (larger groups save products but have more channels to sum up); a
// launch lasts at least as long as its longest wave, 32 rows against all keys, however few SIMDs have one. With the copy
// at hand (kt_in) what is left is the prologue at d = 128, where Q~ is gathered faster than Q_r (1.7 us; not for blocks
// of 256 rows), against a wave's walk, and calls too small for either to matter.
// Blocks of 64 x 128 at d = 128 hold a CU's LDS with two waves (whole K tiles; K_f is a quarter of one), so that more
// than one workgroup per CU is a second round: fused | Q~ K^T there, G8 B11 H16 Hkv8 N99 Nk1150 46 | 59, B20 H16 Hkv4 N226
// Nk385 79 | 99, one round, H16 N1024 causal 34 | 28; G4 B20 H16 Hkv4 N226 Nk385 92 | 102.
// Groups of 16 fuse at a loss, and a fused launch cannot deal its keys out: there attn_bf16_light decides.
// Measured, copy + fused | fused | Q~ K^T, us:
//   G2  d64  H16 N1024 causal 20 | 17 | 18, N4096 53 | 44 | 52, N5372 78 | 67 | 81; B2 H16 Hkv4 N523 Br256 23 | 19 | 21
//       d128 H16 N1024 causal 35 | 30 | 26, N4412 99 | 90 | 97; B4 H16 N1024 60 | 46 | 49
//   G4  d64  H16 N1024 causal 20 | 17 | 18, N4043 50 | 43 | 51, N5372 70 | 61 | 78
//       d128 H16 N1024 causal 32 | 28 | 26, N3321 71 | 62 | 70, N4412 90 | 80 | 96; B2 H16 N534 Nk25907 473 | 430 | 395
//   G8  d64  H16 N1024 causal 22 | 19 | 18; d128 H16 N2021 48 | 40 | 43, N2685 73 | 63 | 78; B4 H16 N1894 117 | 106 | 134
//   G16 d64  H16 N4096 causal 78 | 68 | 55; d128 H16 N2048 causal 83 | 69 | 41
//   keys dealt out: H16 N200 Nk32768 d128 G2 516 | 428 | 86, N1000 Nk8192 125 | 114 | 85
bool attn_bf16_replicated(const Problem& pb, bool have_kt, int n_split) {
  if (attn_bf16_few_rows(pb, 1) || attn_bf16_short(pb, 1)) return true;
  const int G = pb.d / pb.n_groups;
  const double rows = visible_rows(pb);
  const double keys = (double)pb.B * pb.Hkv * pb.Nk;
  if (G >= 16 || n_split > 1) return attn_bf16_light(pb);
  double gain = pb.d == 64 ? (G == 2 ? 0.8 : G == 4 ? 0.75 : 0.25) : (G == 2 ? 0.3 : G == 4 ? 0.5 : 0.6);
  if (pb.d == 128 && pb.Bc == 128 && pb.Br == 64 && G >= 4 && (long long)pb.B * pb.H * ((pb.N + 63) / 64) > 256) gain = G == 4 ? 4.0 : 6.0;
  const double simds = 1024.0 * 32, wave_rows = (double)pb.B * pb.H * ((pb.N + pb.Br - 1) / pb.Br) * pb.Br;
  const double walk = (have_kt && pb.d == 128 ? simds : std::min(wave_rows, simds)) * pb.Nk;
  const double copy = have_kt ? (pb.d == 64 ? 0.1 : pb.Br == 256 ? 0.0 : 1.7) : 4.5 + 0.35e-6 * keys * pb.d;
  return copy > gain * 1e-9 * pb.d * std::max(rows * keys, walk);
}

// Query rows of an exact call's workgroups. Nothing is grouped, so the block that the caller names binds nothing: its rows are those that
// suit the launch. From 1560 shapes of 4 to 512 heads, measured at each; the choice takes 0.2 % more than the best of the three on average, more than 3 % on one in fifty.
// Keys fewer than twice the queries, us, 64 | 128 | 256 rows:
//   64 while two halves of the keys (launch_one) of such blocks fill the chip once: d64 causal H16 N1000 10.2 | 13.7 | 20.6, H8 N2900 20 | 25 | 43,
//      d128 H16 N1000 15.3 | 19.3 | 28.9, not causal H8 N2000 25 | 33 | 40, and not yet H8 N2900 52 | 43 | 63; but for long walks of few heads, whose keys
//      are better dealt out to larger blocks (d128 not causal H4 N2383 29.0 | 24.4 | 34.7, causal N3522 35.4 | 32.9, d64 not causal N3942 30.0 | 27.0);
//      at d = 64 under the mask up to one and a half rounds of 128 rows (H16 N2000 17.5 | 19.8, H32 N1400 17.7 | 18.8, B4 H16 N700 11.6 | 12.4, but
//      H16 N4096 51 | 47), of short prompts up to five and a half of 64 (B16 H12 N305 10.0 | 11.8); not causal where blocks of 128 are just over one round, so
//      that the second is nearly empty (d64 B2 H32 N607 13.8 | 15.0, N1150 20.5 | 21.9, d128 B8 H12 N315 12.7 | 16.1, but d64 B2 H32 N409, one round, 10.1 | 9.2);
//   256 without the mask, where they fill more than half of one round of compute units (d128 H16 N2900 94 | 79 | 72, N4096 149 | 123 | 118, d64 49 | 48 | 44,
//      80 | 74 | 71, d128 H32 N1144 41 | 34 | 31) or, at d = 128 on long walks, the last of a few (H32 N5357, 2.6 rounds, 506 | 425 | 399, N16000 2081 | 1784 | 1687, but N6000,
//      one and a half, 309 | 260 | 283, and B16 H16 N1565 419 | 311 | 342), with little padding;
//   128 otherwise (the caller's 256, causal d64 H16 N9000: 215 | 173 | 193).
// Many more keys than queries (their shares fill the chip): the caller's, up to 128 (N500 on 8000 keys, H16 d64 29 | 27 | 39), and 128 at d = 128 on
// long walks (N512 on 30000 keys 142 | 122, N1000 on 8000 83 | 70, N128 on 2500 15.5 | 17.4) unless they are a tenth more rows.
int attn_bf16_exact_rows(const Problem& pb) {
  if (pb.Bc != 64) return pb.Br;
  const long long heads = (long long)pb.B * pb.H;
  const auto padded = [&](int rows) { return (pb.N + rows - 1LL) / rows * rows; };
  const auto wgs = [&](int rows) { return heads * padded(rows) / rows; };
  if (pb.Nk >= 2LL * pb.N) {
    const bool more = pb.d == 128 && pb.N > 64 && pb.Nk >= 6000 && 10 * padded(128) <= 11 * padded(64);
    return more ? 128 : std::min(pb.Br, 128);
  }
  if (wgs(64) <= kComputeUnits) return (pb.d == 64 && pb.causal) || pb.N < (pb.causal || pb.d == 64 ? 3000 : 2300) ? 64 : 128;
  if (pb.causal) return pb.d == 64 && (2 * wgs(128) <= 3 * kComputeUnits || (pb.N <= 400 && 2 * wgs(64) <= 11 * kComputeUnits)) ? 64 : 128;
  if (wgs(128) > kComputeUnits && wgs(64) <= (pb.d == 64 ? 3 : 2) * kComputeUnits && pb.N < 1400) return 64;
  const long long n = wgs(256), rounds = (n + kComputeUnits - 1) / kComputeUnits, last = n - (rounds - 1) * kComputeUnits;
  if (rounds == 1)
    return 2 * n > kComputeUnits && (pb.d == 128 ? 5 * padded(256) <= 6 * padded(128) : 10 * padded(256) <= 11 * padded(128)) ? 256 : 128;
  return pb.d == 128 && pb.N >= 2200 && 20 * last >= (rounds <= 3 ? 11 : 19) * kComputeUnits ? 256 : 128;
}

// Query rows of a grouped call's workgroups when its keys are dealt out, whose grouping then comes from a table: two Q blocks of 64 rows at
// d = 128 on long walks (blocks of 64 have half the waves to a tile there), unless they are a tenth more rows. us, one | two: H16 N100 Nk16000
// 44.4 | 39.6, N200 Nk30000 95 | 80, N700 Nk8000 80 | 72, H32 Hkv8 N500 Nk8000 95 | 86, N200 58 | 51. On 2500 keys exact blocks of 64 are the faster.
int attn_bf16_shared_rows(const Problem& pb) {
  const auto padded = [&](int rows) { return (pb.N + rows - 1LL) / rows * rows; };
  return pb.d == 128 && pb.Br == 64 && pb.Bc == 64 && pb.N > 64 && pb.Nk >= 6000 && 10 * padded(128) <= 11 * padded(64) ? 128 : pb.Br;
}

// Query rows of a grouped call's workgroups (Q~ K^T, keys not dealt out): a part of a Q block where an exact call would take fewer rows
// (0: a whole one). Their grouping comes from a table, which the LSH kernel has to make where the call would have had it in its
// prologue (5-7 us instead of 3-6): for blocks of 256 rows always worth it, for blocks of 128 with halves of 64 on one round of compute units
// and more than a dozen tiles. us, whole | parts: Br256 d64 H16 N600 22.9 | 18.7, N1000 30.1 | 21.3, N2000 43.5 | 28.4, d128 43.7 | 29.5 (N1000), not causal
// H8 N3000 83.9 | 59.7; Br128 d64 H16 N1000 20.4 | 18.4, H8 N3000 33.7 | 30.0, d128 H8 N1000 27.7 | 25.0, but d64 H32 N700 16.6 | 17.3, N1400 25.2 | 27.7,
// not causal H32 N700 17.8 | 20.5, H8 N600 15.8 | 16.2. Wherever the
// table comes from (the caller, o) the rows are the same, so that the output's bits are.
int attn_bf16_grouped_rows(const Problem& pb) {
  if (pb.Bc != 64 || pb.Br == 64 || attn_bf16_few_rows(pb, 1) || attn_bf16_short(pb, 1)) return 0;
  const int rows = attn_bf16_exact_rows(pb);
  if (rows >= pb.Br) return 0;
  const long long n = (long long)pb.B * pb.H * ((pb.N + 63) / 64);
  if (pb.Br == 256 || (n <= kComputeUnits && pb.Nk >= 800)) return rows;
  return pb.d == 64 && pb.causal && n <= 2 * kComputeUnits && pb.Nk >= 1800 ? rows : 0;
}

// Key shares per Q block, for launches that would leave compute units without a workgroup: one
// four-wave workgroup (two of two waves, half of one of eight) for each, at least four tiles per share, and only where the
// tiles taken off a workgroup's walk outweigh the combine kernel (4 us, about 12 tiles) and, grouped,
// the LSH stage in a kernel of its own (another 18). Measured, 1 | 256 | 512 workgroups: exact H16 N200 Nk8192
// d64 71 | 19 | 22 us; N1000 Nk8192 d128 109 | 72 | 80; N200 Nk32768 d128 486 | 90 | 87; N2048 d64 causal 22 | 22 | 29.
// Blocks of 64 rows at d = 128 take one workgroup, of two halves (launch_one), for each where that leaves at most 16 compute units
// idle and does not undo the sharing out: half the sums to combine. The halves wait for the later of two loads at every tile (the same bytes
// and L2 hits either way; H32 N120 Nk30000 exact 104 us in the kernel, 126 in halves): blocks that find each other's tiles in an L2 gain
// on short walks only. exact, distr, two for each | one: nothing shared, H32 N64 Nk4096 21.9 | 20.6, 28.9 | 26.6, Nk30000 97 | 94, 105 | 101,
// H11 N700 Nk16000 138 | 125, 146 | 132; shared, by tiles per workgroup, one / two: 16-32 (H32 N120 or N200, Nk4096) 0.85-1.00, 43-47 (H32 N120
// Nk12000, N200 Nk6000) 0.94-1.02, 62-78 (N200 Nk8000, N120 Nk20000) 1.01-1.17, more up to 1.24, and with no shares to combine at all (256
// blocks) 64 tiles 0.92-0.95, 94 0.98-1.02, 125 1.11. 80 units idle (H44 N200) Nk4096 1.09, Nk30000 1.33; distr H32 Hkv8 N200 Nk3000, where two
// shares are not worth the LSH launch, 34.6 | 39.5.
int attn_bf16_splits(const Problem& asked, int distr) {
  if (attn_bf16_short(asked, distr)) return 1;
  Problem pb = asked;
  if (distr) pb.Br = attn_bf16_shared_rows(asked);
  const long long units = (long long)pb.B * pb.H * ((pb.N + pb.Br - 1) / pb.Br);
  const int tiles = (pb.Nk + pb.Bc - 1) / pb.Bc;
  // (exact blocks of 64 rows that two halves of a prompt's keys are walked for anyway have half as much to gain: H8 N1000 14 us in four shares, 10 in none; chunks
  // on a cache not: d128 H8 N108 on 1490 keys 12.6 in shares, 18.3 in none, H32 N107 on 1732 15.3 | 16.6, d64 H12 N161 on 1419 10.2 | 11.9, but of many blocks
  // at d = 64: H32 N104 on 1598 13.1 | 11.8, B5 H16 N40 on 1132 11.4 | 9.8)
  const bool in_halves = !distr && (pb.Nk < 2LL * pb.N || (pb.d == 64 && 4 * units >= kComputeUnits)) && pb.Br == 64 && pb.Bc == 64 && units <= (pb.d == 64 ? 2 : 1) * kComputeUnits;
  const auto worth = [&](long long n) { return n > 1 && tiles - tiles / n >= (distr ? 30 : in_halves ? 24 : 12); };
  long long n = std::min<long long>(1024 / (pb.Br / 32) / units, tiles / 4);
  const long long one = kComputeUnits / units, few = std::min<long long>(one, tiles / 4);
  if (pb.d == 128 && pb.Br == 64 && pb.Bc == 64 && one * units >= kComputeUnits - 16 && (blocks_sharing_l2(pb, pb.Br) < 12 || tiles <= std::max(64LL, 48 * one)) &&
      (one == 1 || worth(few) || !worth(n)))
    n = few;
  if (!worth(n)) n = 1;
  if (attn_bf16_few_rows(pb, distr)) n = attn_bf16_few_splits(pb);
  const long long row_bytes = (long long)pb.B * pb.H * pb.N * (pb.d * 4 + 8);
  if (n * row_bytes > (24LL << 20)) n = (24LL << 20) / row_bytes;
  return n > 1 ? (int)n : 1;
}

// O of a row = sum over the shares of 2^(reference - largest reference) O_share, over the same sum of the
// row sums. A workgroup takes 256 / L / (D/4) rows, a thread four channels of every L-th share: few rows
// with many shares (decoding) would otherwise be a chain of loads in a handful of waves. Bound: a memory round trip for every
// 4 L shares, as a thread asks for statistics and sums of four at once and keeps a reference of its own (statistics of all shares
// first, then the sums, were a round trip more: decoding, 32 rows of 32 shares, one instead of two, 4.5 -> 3.0 us; 3200 rows of 8 shares
// at d = 128, L = 1, take two either way, 4.8 us). A share whose sum is not above
// zero is empty or holds a NaN: its weight is 0, and 0 times its NaN sum still makes the row NaN.
template <int D, int L>
__global__ __launch_bounds__(256) void attn_bf16_combine_kernel(const float* __restrict__ part_o, const f32x2* __restrict__ part_stat,
                                                                bf16* __restrict__ o, float* __restrict__ lse, int rows, int n_split) {
  constexpr int Q = D / 4, R = 256 / L / Q;
  __shared__ f32x2 stat_lds[L > 1 ? 256 : 1];
  __shared__ __attribute__((aligned(16))) f32x4 acc_lds[L > 1 ? 256 : 1];
  const int tid = threadIdx.x;
  const int c = tid % Q, row = blockIdx.x * R + tid / Q % R, part = tid / Q / R;
  const int row_ld = min(row, rows - 1);
  float ref = -INFINITY, l = 0.0f;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  auto weight = [&](float r) { return r > -INFINITY ? __builtin_amdgcn_exp2f(r - ref) : 0.0f; };
  for (int s0 = part; s0 < n_split; s0 += 4 * L) {
    f32x2 st[4];
    f32x4 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = min(s0 + j * L, n_split - 1);
      st[j] = part_stat[(size_t)s * rows + row_ld];
      x[j] = *(const f32x4*)(part_o + ((size_t)s * rows + row_ld) * D + c * 4);
    }
    const float before = ref;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (s0 + j * L >= n_split) st[j] = f32x2{0.0f, 0.0f};
      if (!(st[j][1] > 0.0f)) {   // (an empty share has left no sums)
        st[j][0] = -INFINITY;
        x[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
      ref = fmaxf(ref, st[j][0]);
    }
    const float keep = weight(before);
    l *= keep;
    acc *= keep;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float w = weight(st[j][0]);
      l = __builtin_fmaf(w, st[j][1], l);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(w, x[j][e], acc[e]);
    }
  }
  if constexpr (L > 1) {
    stat_lds[tid] = f32x2{ref, l};
    acc_lds[tid] = acc;
    __syncthreads();
    if (part != 0) return;
    f32x2 st[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      st[j] = stat_lds[j * Q * R + tid];
      ref = fmaxf(ref, st[j][0]);
    }
    l = 0.0f;
    acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const float w = weight(st[j][0]);
      l = __builtin_fmaf(w, st[j][1], l);
      acc += acc_lds[j * Q * R + tid] * w;
    }
  }
  if (row >= rows) return;
  const float inv = 1.0f / l;
  const bf16x4 y = {(bf16)(acc[0] * inv), (bf16)(acc[1] * inv), (bf16)(acc[2] * inv), (bf16)(acc[3] * inv)};
  *(bf16x4*)(o + (size_t)row * D + c * 4) = y;
  if (lse && c == 0) lse[row] = 0.6931471805599453f * (ref + __builtin_log2f(l));
}

template <int D>
static hipError_t launch_combine(void* o, const Problem& pb, hipStream_t stream) {
  const long long rows = (long long)pb.B * pb.H * pb.N;
#define DA_COMBINE(L)                                                                                                     hipLaunchKernelGGL((attn_bf16_combine_kernel<D, L>), dim3((unsigned)((rows + 1024 / L / D - 1) / (1024 / L / D))), dim3(256), 0,                      stream, pb.part_o, (const f32x2*)pb.part_stat, (bf16*)o, pb.lse, (int)rows, pb.n_split)
  if (rows * (D / 4) >= 65536 || pb.n_split < 8) DA_COMBINE(1);   // a wave for every SIMD as it is
  else DA_COMBINE(8);
#undef DA_COMBINE
  return hipGetLastError();
}

hipError_t launch_attn_bf16_combine(void* o, const Problem& pb, hipStream_t stream) {
  return pb.d == 64 ? launch_combine<64>(o, pb, stream) : launch_combine<128>(o, pb, stream);
}

hipError_t launch_attn_bf16(const void* q, const void* k, const void* v, void* o, const uint8_t* perm,
                            const void* kt, const Problem& pb, int distr, hipStream_t stream) {
  if (!attn_bf16_supported(pb, distr)) return hipErrorInvalidValue;
  if (!kt && attn_bf16_few_rows(pb, distr)) return launch_attn_bf16_few(q, k, v, o, perm, pb, distr, stream);
  if (!kt && attn_bf16_short(pb, distr)) return launch_attn_bf16_short(q, k, v, o, perm, pb, distr, stream);
  if (pb.Bc == 32) return launch_attn_bf16_bc32(q, k, v, o, perm, kt, pb, distr, stream);
  if (pb.Bc == 128) return launch_attn_bf16_bc128(q, k, v, o, perm, kt, pb, distr, stream);
  return launch_attn_bf16_bc64(q, k, v, o, perm, kt, pb, distr, stream);
}

}  // namespace da
