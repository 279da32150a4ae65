// Pieces shared by the float-arithmetic kernels (attn_f32.hip, attn_f32_bwd.hip), which work in tiles
// of 32 rows on v_mfma_f32_32x32x2_f32.
#pragma once
#include "da_common.h"

namespace da {

namespace {

constexpr int kTile = 32;   // rows per tile, on either side
// Register i of a 32 x 32 accumulator holds, in lane half hh, this row of its tile; as the contraction
// index of step i the same order makes an accumulator the operand of the next product.
__device__ inline int acc_row(int i, int hh) { return 8 * (i >> 2) + 4 * hh + (i & 3); }

__device__ inline void zero(f32x16& x) {
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = 0.0f;
}
__device__ inline f32x16 mfma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// A sum over STEPS contraction steps (all unrolled: `s` is known). ChannelSum takes it in two or four chains, for the
// rounding of short sums: in one chain, scores of up to 25 put the output of exact attention 1.6 times (d = 64) and
// twice (d = 128) as far from 64 bits as four partial sums per row do. Forward and backward sum alike, so that
// P = exp(S - lse) is taken of the S that lse was. The chains run one by one (the empty asm wants a chain's sum before
// the next one starts): several at once do not fit the registers (100 of them spilled).
struct OneChain {
  f32x16 total;
  __device__ void step(int s, float a, float b) {
    if (s == 0) zero(total);
    total = mfma(a, b, total);
  }
  __device__ f32x16 sum() const { return total; }
};
template <int STEPS>
struct ChannelSum {
  static constexpr int CHAIN = STEPS >= 32 ? STEPS / 4 : STEPS / 2;
  f32x16 total, chain;
  __device__ void step(int s, float a, float b) {
    if (s % CHAIN == 0) {
      if (s > 0) close(s == CHAIN);
      zero(chain);
    }
    chain = mfma(a, b, chain);
  }
  __device__ f32x16 sum() {
    close(false);
    return total;
  }

 private:
  __device__ void close(bool first) {
    if (first) total = chain;
    else total += chain;
    asm volatile("" : "+v"(total));
  }
};

// Eight floats as operands of v_mfma_f32_32x32x16_bf16: hi + mid + lo with eight significand bits each (rounded to
// nearest, so that mid and lo are at most 2^-8 and 2^-17 of the float), together the float itself unless it is below 2^-110
// (bf16 ends at 2^-133) or so near the largest that hi is infinite.
struct Pieces {
  bf16x8 hi, mid, lo;
};
typedef __attribute__((ext_vector_type(8))) float f32x8;
__device__ inline bf16x8 round8(f32x8 x) { return __builtin_convertvector(x, bf16x8); }
__device__ inline f32x8 rest8(f32x8 x, bf16x8 y) {
  const u32x4 b = __builtin_bit_cast(u32x4, y);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] -= __builtin_bit_cast(float, b[j] << 16);
    x[2 * j + 1] -= __builtin_bit_cast(float, b[j] & 0xffff0000u);
  }
  return x;
}
__device__ inline Pieces split(f32x8 x) {
  Pieces p;
  p.hi = round8(x);
  x = rest8(x, p.hi);
  p.mid = round8(x);
  p.lo = round8(rest8(x, p.mid));
  return p;
}
__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
// The same for sixteen floats a lane as two operands, the subtractions taken by the matrix instruction: the floats are
// an accumulator, and what is subtracted, the operand of steps t = 0 and 1, contributes -1 times its own place (at(8 t + j)). 24
// instead of 88 vector instructions, for 4 products.
struct Splitter {
  bf16x8 minus[2];
  __device__ explicit Splitter(int lane) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j) minus[t][j] = (bf16)((lane & 31) == acc_row(8 * t + j, lane >> 5) ? -1.0f : 0.0f);
  }
  __device__ void operator()(f32x16 x, Pieces& p0, Pieces& p1) const {
    p0.hi = round8(x.lo);
    p1.hi = round8(x.hi);
    x = mfma(minus[1], p1.hi, mfma(minus[0], p0.hi, x));
    p0.mid = round8(x.lo);
    p1.mid = round8(x.hi);
    x = mfma(minus[1], p1.mid, mfma(minus[0], p0.mid, x));
    p0.lo = round8(x.lo);
    p1.lo = round8(x.hi);
  }
};
// c += a b without what mid lo, lo mid and lo lo add (2^-24 of a b at most), the small products first.
__device__ inline f32x16 mfma_rest(const Pieces& a, const Pieces& b, f32x16 c) {
  c = mfma(a.lo, b.hi, c);
  c = mfma(a.hi, b.lo, c);
  c = mfma(a.mid, b.mid, c);
  c = mfma(a.mid, b.hi, c);
  return mfma(a.hi, b.mid, c);
}
__device__ inline f32x16 mfma(const Pieces& a, const Pieces& b, f32x16 c) { return mfma(a.hi, b.hi, mfma_rest(a, b, c)); }

// HS floats of a lane's half row as operands, split on the way: step(s, pieces)
template <int HS, bool BY_MFMA = true, typename STEP>
__device__ inline void split_steps(const Splitter& splitter, const float (&x)[HS], STEP step) {
  if constexpr (HS == 8 || !BY_MFMA) {
#pragma unroll
    for (int s = 0; s < HS; s += 8) {
      f32x8 y;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = x[s + e];
      step(s / 8, split(y));
    }
  } else {
#pragma unroll
    for (int s = 0; s < HS; s += 16) {
      f32x16 y;
#pragma unroll
      for (int e = 0; e < 16; ++e) y[e] = x[s + e];
      Pieces p0, p1;
      splitter(y, p0, p1);
      step(s / 8, p0);
      step(s / 8 + 1, p1);
    }
  }
}

// A sum over the channels, 16 a step, the products of the leading pieces and the others in a chain each.
struct PieceSum {
  f32x16 lead, rest;
  __device__ PieceSum() {
    zero(lead);
    zero(rest);
  }
  // b_first: the products in the order that step(b, a) takes them in
  template <bool b_first = false>
  __device__ void step(const Pieces& a, const Pieces& b) {
    if constexpr (b_first) {
      rest = mfma(a.hi, b.lo, rest);
      rest = mfma(a.lo, b.hi, rest);
      rest = mfma(a.mid, b.mid, rest);
      rest = mfma(a.hi, b.mid, rest);
      rest = mfma(a.mid, b.hi, rest);
    } else {
      rest = mfma_rest(a, b, rest);
    }
    lead = mfma(a.hi, b.hi, lead);
  }
  __device__ f32x16 sum() const {
    f32x16 total = lead + rest;
    asm volatile("" : "+v"(total));   // here: behind a branch the compiler does not wait long enough for the products on every path
    return total;
  }
};

// Products by pieces: groups of two and four channels at d = 64, and the mirrored form (which has no backward to agree with on the
// scores' last bits) at any d, from more than eight key tiles on. us of a call, float products | pieces, H1 d64 groups of two:
//   forward  N256 8.3 | 8.7, N320 10.0 | 9.1, N512 11.9 | 10.7, N1024 19.2 | 15.9; mirrored 8.7 | 9.2, 11.6 | 10.8, 12.8 | 11.9, 21.0 | 18.0
//   backward N128 18.3 | 20.0, N256 25.9 | 26.5, N320 34.7 | 31.8, N512 38.6 | 34.5, N1024 60.3 | 52.4
inline bool float_by_pieces(const Problem& pb) {
  const int G = pb.d / pb.n_groups;
  return (G == 2 || G == 4) && (pb.d == 64 || pb.side == 1) && pb.Nk > 8 * kTile && pb.scale <= 0x1p20f;
}

// A float times 2^24 is the sum of its pieces whatever its size, up to 2^103: its last bit, 2^-125 at least, is within bf16's range.
// Larger ones come out infinite or NaN and are taken again.
constexpr float kRaise = 0x1p24f;

// Which scores are taken by pieces, in every kernel alike (P = exp(S - lse) wants the S that lse was taken of): those whose operands,
// the sampled channels of a query row and the sums of a key row over the Q block's groups (the mirrored form: all channels of
// the query row, the sampled ones of the key row), are below 2^60. What pieces lose of the smallest floats is then 2^-60 of a
// score at most, and the scale is no larger than 2^20. The other scores are float products, pair by pair, in a second walk of
// the workgroups that have such rows.
constexpr float kPieceLimit = 0x1p60f;
__device__ inline float largest(float m, float x, float y) {   // (of magnitudes; NaN stays)
  return __builtin_elementwise_maximum(m, __builtin_elementwise_maximum(__builtin_fabsf(x), __builtin_fabsf(y)));
}
__device__ inline float largest(float m, float x) { return __builtin_elementwise_maximum(m, __builtin_fabsf(x)); }
__device__ inline float largest(float m, f32x4 x) { return largest(largest(m, x[0], x[1]), x[2], x[3]); }
template <int C>
__device__ inline float largest(const float (&x)[C]) {
  float m = 0.0f;
#pragma unroll
  for (int c = 0; c < C; c += 2) m = largest(m, x[c], x[c + 1]);
  return m;
}
__device__ inline bool beyond_pieces(float m) { return !(m < kPieceLimit); }
// rows of a bit mask, from what either half of the wave says of its 32 rows
__device__ inline uint32_t rows_of(bool any) {
  const uint64_t rows = __builtin_amdgcn_ballot_w64(any);
  return (uint32_t)rows | (uint32_t)(rows >> 32);
}

// Infinities and NaN (a product with them makes every sum of its row NaN) and what is too large are found in the results: a workgroup
// takes the rows of its 32 again that are not finite, all but the scores with float products.
constexpr uint32_t kRowAgain = 1, kRowBeyond = 2;   // kRowBeyond: with a score that is not by pieces (beyond_pieces)
__device__ inline bool all_finite(f32x4 x) { return largest(0.0f, x) < INFINITY; }

// Pieces of 32 rows of C floats in LDS; rows 16 bytes apart in the banks, a lane's operand is one read per piece.
template <int C>
struct PieceRows {
  static constexpr int RS = C + 8;
  bf16 x[3][kTile * RS];
  __device__ void store(int row, int c, const Pieces& p) {
    *(bf16x8*)&x[0][row * RS + c] = p.hi;
    *(bf16x8*)&x[1][row * RS + c] = p.mid;
    *(bf16x8*)&x[2][row * RS + c] = p.lo;
  }
  __device__ Pieces load(int row, int c) const {
    return {*(const bf16x8*)&x[0][row * RS + c], *(const bf16x8*)&x[1][row * RS + c], *(const bf16x8*)&x[2][row * RS + c]};
  }
};

// x * scale + y with the product rounded: a score that is its row's maximum, whose lse is the rounded maximum plus
// ln(sum), then gives exactly -ln(sum) in the backward pass, however large it is.
__device__ inline float scaled_plus(float x, float scale, float y) {
#pragma clang fp contract(off)
  return x * scale + y;
}

// Buffer descriptor over `bytes` of one head: loads past the end read as zeros.
__device__ inline __amdgpu_buffer_rsrc_t head_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}

// Four consecutive channels of a row, as loaded and as floats.
template <typename E>
struct Quad;
template <>
struct Quad<float> {
  typedef u32x4 raw;
  static __device__ raw load(__amdgpu_buffer_rsrc_t rsrc, int voff, int soff) {
    return __builtin_bit_cast(raw, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0));
  }
  static __device__ f32x4 values(raw x) { return __builtin_bit_cast(f32x4, x); }
};
template <>
struct Quad<bf16> {
  typedef u32x2 raw;
  static __device__ raw load(__amdgpu_buffer_rsrc_t rsrc, int voff, int soff) {
    return __builtin_bit_cast(raw, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, soff, 0));
  }
  static __device__ f32x4 values(raw x) {
    const u32x4 y = {x[0] << 16, x[0] & 0xffff0000u, x[1] << 16, x[1] & 0xffff0000u};
    return __builtin_bit_cast(f32x4, y);
  }
};
// Two consecutive channels.
template <typename E>
struct Pair;
template <>
struct Pair<float> {
  typedef u32x2 raw;
  static __device__ raw load(__amdgpu_buffer_rsrc_t rsrc, int voff, int soff) {
    return __builtin_bit_cast(raw, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, soff, 0));
  }
  static __device__ float value(raw x, int i) { return __builtin_bit_cast(f32x2, x)[i]; }
};
template <>
struct Pair<bf16> {
  typedef uint32_t raw;
  static __device__ raw load(__amdgpu_buffer_rsrc_t rsrc, int voff, int soff) {
    return __builtin_amdgcn_raw_buffer_load_b32(rsrc, voff, soff, 0);
  }
  static __device__ float value(raw x, int i) { return __builtin_bit_cast(float, i ? x & 0xffff0000u : x << 16); }
};

// LDS written by some lanes of a wave is read by others: nothing moves across (no instruction).
__device__ inline void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

}  // namespace da
