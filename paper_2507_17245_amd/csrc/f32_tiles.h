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
