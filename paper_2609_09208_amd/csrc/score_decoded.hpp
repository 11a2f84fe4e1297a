// Scores of a 64-key tile for the engines that multiply (Sec. III): PoT codes
// decoded to fp16 weights, and the INT8 and fp16 comparators. Same operand
// layout as the plane sums (score_planes.hpp): rows are keys, two keys (X in
// blocks 0-1, Y in blocks 2-3) to a row, columns 0-7 and 8-15 are the queries
// for X and for Y; a lane holds one half of one key per set and gets the
// scores of one head and 8 consecutive keys.
//
// Decoded weights (kScoreDs4a): element m is sigma (1 + j / 2^k) 2^(-8 - e),
// the fp16 number with sign bit sigma, exponent field 7 - e (the complement of
// the code's exponent bits) and the mantissa bits j on top of its mantissa; the zero code
// (e = 7, with j taken as 0) is exponent field 0: zero. Two elements take 4 VALU
// operations (6 with a mantissa; and about 19 per set that clear the mantissa bits
// of zero codes, whose planes may hold anything: 0.1 us of a call of one tile per
// wave, 6.87 -> 7.02 us at k = 1, B = 1, T = 1024). q^ 2^8 is an exact fp16 number,
// v_mfma_f32_16x16x32_f16 multiplies and sums, and 2^(k + F) makes the result the
// int32 score at head-room F: exact, since with unit 2^(F - 6) every partial sum is an integer
// below 64 * 127 * 1984 < 2^24. (One key per lane on v_dot4 / v_dot2 took 414
// VALU lane-operations per key at k = 0 and 817 at k = 4 and, like the other
// engines, a transpose through LDS.)
#pragma once

#include "pot_device.hpp"
#include "score_planes.hpp"

namespace potattn {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Code dword (K = 0) or transposed code dword (K > 0) w with mantissa nibbles
// j: the weights of nibbles n and n + 4, n = 0..3, as one fp16 pair each.
template <int K>
__device__ __forceinline__ half8 decode_weights(uint32_t w, uint32_t j) {
  const uint32_t nx = ~w;
  uint32_t v[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const uint32_t ex = n < 3 ? nx << (n < 3 ? 10 - 4 * n : 0) : nx >> 2;
    v[n] = ex & 0x1C001C00u;
    if constexpr (K > 0) {
      constexpr uint32_t kMant = ((1u << K) - 1) << (10 - K);
      const int sh = 10 - K - 4 * n;  // nibble n to the top of the mantissa
      v[n] |= (sh >= 0 ? j << (sh >= 0 ? sh : 0) : j >> (sh < 0 ? -sh : 0)) & (kMant * 0x10001u);
    }
    v[n] |= (w << (12 - 4 * n)) & 0x80008000u;
  }
  return __builtin_bit_cast(half8, make_uint4(v[0], v[1], v[2], v[3]));
}

// Bit 4i + c set where element 4i + c, nibble i of the transposed code dword
// c4[c], is the zero code: adding 1 to the exponent bits (sign cleared, so no
// carry between nibbles) sets bit 3 for exponent 7, and the dwords' bits merge in
// the order of the plane bits.
__device__ __forceinline__ uint32_t zero_codes(const uint32_t (&c4)[4]) {
  uint32_t y[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) y[c] = (c4[c] & 0x77777777u) + 0x11111111u;
  uint32_t z = y[3];
  constexpr uint32_t kSelectTable = 0xCA;  // a ? b : c, bit by bit
#pragma unroll
  for (int c = 2; c >= 0; --c)
    z = __builtin_amdgcn_bitop3_b32(0x11111111u << c, y[c] >> (3 - c), z, kSelectTable);
  return z;
}

// Place of element m of a half in the fp16 query operand: dword c, nibble nib,
// in the pair order of decode_weights (K < 0: natural order).
template <int K>
__device__ __forceinline__ int pair_order(int m) {
  if (K < 0) return m;
  const int at = plane_order<K < 0 ? 0 : K>(m);  // 8 c + nib
  return (at & ~7) + 2 * (at & 3) + ((at >> 2) & 1);
}

// Query operands: 32 fp16 numbers of the lane's half (fp16 keys, decoded
// weights), or 32 bytes (INT8 keys); zeros where the lane's block is not its
// column's.
struct HalfQuery {
  half8 h[4];
};
struct ByteQuery {
  i32x4 b[2];
};

__device__ __forceinline__ bool query_block_used(int lane, int G) {
  return ((lane >> 3) & 1) == (lane >> 5) && (lane & 7) < G;
}

template <int G>
__device__ __forceinline__ HalfQuery load_half_query(const _Float16 (*q)[kDim], int lane) {
  const int h = lane & 7;
  const bool used = query_block_used(lane, G);
  const uint4* p = reinterpret_cast<const uint4*>(&q[h < G ? h : 0][32 * ((lane >> 4) & 1)]);
  HalfQuery r;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint4 v = p[c];
    r.h[c] = __builtin_bit_cast(half8, used ? v : make_uint4(0u, 0u, 0u, 0u));
  }
  return r;
}

template <int G>
__device__ __forceinline__ ByteQuery load_byte_query(const int8_t (*q)[kDim]) {
  const int lane = lane_id(), h = lane & 7;
  const bool used = query_block_used(lane, G);
  const i32x4* p = reinterpret_cast<const i32x4*>(&q[h < G ? h : 0][32 * ((lane >> 4) & 1)]);
  ByteQuery r;
#pragma unroll
  for (int c = 0; c < 2; ++c) r.b[c] = used ? p[c] : i32x4{0, 0, 0, 0};
  return r;
}

// Decoded weights: the sum of q^ times the weights, times 2^(k + F) (to_int).
template <int K>
__device__ __forceinline__ f32x4 score_set_decoded(const uint32_t (&w)[4], const uint32_t* pl,
                                                   const HalfQuery& q, float to_int) {
  uint32_t c4[4];
  if constexpr (K == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) c4[c] = w[c];
  } else {
    transpose_codes(w, c4);
  }
  uint32_t pm[K > 0 ? K : 1];  // plane bits, 0 for zero codes
  if constexpr (K > 0) {
    const uint32_t z = zero_codes(c4);
#pragma unroll
    for (int b = 0; b < K; ++b) pm[b] = pl[b] & ~z;
  }
  f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t j = 0;
#pragma unroll
    for (int b = 0; b < K; ++b) {  // bit 4i + c of plane b to bit b of nibble i
      const uint32_t x = c >= b ? pm[b] >> (c >= b ? c - b : 0) : pm[b] << (c < b ? b - c : 0);
      j |= x & (0x11111111u << b);
    }
    d = __builtin_amdgcn_mfma_f32_16x16x32_f16(decode_weights<K>(c4[c], j), q.h[c], d, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // one operand at a time: registers
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) d[r] = __fmul_rn(d[r], to_int);
  return d;
}

// INT8 keys: v_mfma_i32_16x16x64_i8 over the lane's 32 bytes (exact).
__device__ __forceinline__ f32x4 score_set_int8(const uint4 (&k)[2], const ByteQuery& q) {
  i32x4 d = {0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < 2; ++c)
    d = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, k[c]), q.b[c], d, 0, 0, 0);
  return f32x4{(float)d[0], (float)d[1], (float)d[2], (float)d[3]};
}

// fp16 keys: v_mfma_f32_16x16x32_f16 over the lane's 32 elements.
__device__ __forceinline__ f32x4 score_set_fp16(const uint4 (&k)[4], const HalfQuery& q) {
  f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < 4; ++c)
    d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, k[c]), q.h[c], d, 0, 0, 0);
  return d;
}

}  // namespace potattn
