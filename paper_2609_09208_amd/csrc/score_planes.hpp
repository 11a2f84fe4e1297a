// Shift-accumulate scores of a 64-key tile on the matrix cores (Sec. II-B eq.
// sac, Sec. II-D eq. mant), regrouped by bit position.
//
// A code's magnitude in units of 2^-(6 + k) is (2^k + j) 2^(6 - e): bit b of
// the mantissa and the leading one (b = k) stand at position p = b + 6 - e.
// The key's sum is therefore
//     sum_m q^_m sigma_m (2^k + j_m) 2^(6 - e_m) = sum_p 2^p sum_m q^_m T_pm
// with T_pm in {-1, 0, +1}: the sign where bit p of the magnitude is set. The
// 7 + k ternary sums of q^ are formed by v_mfma_scale_f32_16x16x128_f8f6f4
// over fp4 operands whose only values are -1, -0, 0 and 1, so its multipliers
// see nothing else on the key side, and the shift by p is the power-of-two
// block scale of the fp4 operand, which the matrix core adds to the exponents.
// q^ in [-127, 127] goes in as 16 hi + lo, two bf6 (e3m2) operands of
// integers in [-8, 8]. The scales also carry 2^(F - 6), so the fp32 result is
// the int32 score at head-room F. It is exact: with unit 2^(F - 6) every
// partial sum is an integer of magnitude at most 64 * 128 * 1984 < 2^24
// (hi alone may reach 128; 1984 = 31 * 64 at k = 4).
//
// Operand layout. A (16 rows x 128) holds keys and B (128 x 16 columns) holds
// queries: lane l gives row / column l % 16 and the 32 elements of block
// l / 16. One key has 64 elements, two blocks, so a row carries two keys: X
// in blocks 0-1 and Y in blocks 2-3; columns 0-7 hold the queries of the 8
// heads in blocks 0-1 and zeros in blocks 2-3, columns 8-15 the same queries
// in blocks 2-3, so column h gets X's score for head h and column 8 + h gets
// Y's. Each lane's 32 elements are the 16 code bytes of one half of one key:
// one 16-byte load, and one dword of eight elements turns into one dword of
// the fp4 operand. Row i of set s (s = 0, 1) is key 8 (i / 4) + 4 s + i % 4
// of the tile (X) and that plus 32 (Y). The result then has lane l holding
// head l % 8 and keys 32 (l / 8 % 2) + 8 (l / 16) + 4 s + r in register r of
// set s: the 8 consecutive keys whose weights the lane forms for P.V. No
// transpose and no LDS.
//
// Cost per tile at k = 0: 136 VALU operations (2 per plane and code dword and
// 3 to set a dword up; v_bitop3_b32 on VGPRs, the fast issue class) and 28
// matrix instructions of 16 cycles.
#pragma once

#include "pot_device.hpp"

namespace potattn {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
typedef _Float16 half32 __attribute__((ext_vector_type(32)));

// Position within its half (32 elements) at which the operands hold element
// m. PoT-4: as the code dwords hold them. With mantissa planes the code
// nibbles are transposed to the order of the plane bits (transpose_codes).
template <int K>
__device__ __forceinline__ int plane_order(int m) {
  return K == 0 ? m : 8 * (m & 3) + (m >> 2);
}

// Code dwords w (nibble n of w[c]: element 8c + n) to c[s], nibble i: element
// 4i + s. A dword of plane bits (bit m: element m) then lines up with c[s]
// after one shift. A 4 x 4 byte transpose, then one nibble merge per dword.
__device__ __forceinline__ void transpose_codes(const uint32_t (&w)[4], uint32_t (&c)[4]) {
  const uint32_t a0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
  const uint32_t b0 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
  const uint32_t a1 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const uint32_t b1 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
#pragma unroll
  for (int sp = 0; sp < 2; ++sp) {
    const uint32_t sel = sp ? 0x07060302u : 0x05040100u;
    const uint32_t h0 = __builtin_amdgcn_perm(a1, a0, sel);  // bytes sp of w[0..3]
    const uint32_t h1 = __builtin_amdgcn_perm(b1, b0, sel);  // bytes 2 + sp
    c[2 * sp] = (h0 & 0x0F0F0F0Fu) | ((h1 << 4) & 0xF0F0F0F0u);
    c[2 * sp + 1] = ((h0 >> 4) & 0x0F0F0F0Fu) | (h1 & 0xF0F0F0F0u);
  }
}

// v_bitop3_b32 truth tables over (a, b, c) = (0xF0, 0xCC, 0xAA)
constexpr uint32_t minterm_table(int e) {
  return (((e & 1) ? 0xF0u : 0x0Fu) & ((e & 2) ? 0xCCu : 0x33u) & ((e & 4) ? 0xAAu : 0x55u)) & 0xFFu;
}
constexpr uint32_t kAndOrTable = 0xF8;  // a | (b & c)
constexpr uint32_t kMaskOrTable = 0xEA; // (a & b) | c

// One code dword of a half key: what its planes are made from. Bit 1 of each
// nibble is the working bit (fp4 1.0 is 0b0010).
struct CodeBits {
  uint32_t x0, x1, x2;  // exponent bits 0, 1, 2 moved to bit 1
  uint32_t sign;        // the sign bits in place (fp4's sign is bit 3 too)
};
__device__ __forceinline__ CodeBits code_bits(uint32_t w) {
  CodeBits b;
  b.x0 = w << 1;
  b.x1 = w;
  b.x2 = w >> 1;
  b.sign = w & 0x88888888u;
  return b;
}
// bit 1 of each nibble: exponent == E
template <int E>
__device__ __forceinline__ uint32_t exponent_is(const CodeBits& b) {
  constexpr uint32_t kTable = minterm_table(E);
  return __builtin_amdgcn_bitop3_b32(b.x0, b.x1, b.x2, kTable);
}

// The query operands of a lane (hi and lo parts, six dwords each) and the
// block scales: byte p % 4 of a[p / 4] is that of position p, byte 0 of b is
// that of lo and byte 1 that of hi.
struct PlaneQuery {
  i32x8 hi, lo;
  int a[3], b;
};

template <int P>
__device__ __forceinline__ void add_plane(const uint32_t (&t)[4], const PlaneQuery& q, f32x4& d) {
  const i32x8 av = {(int)t[0], (int)t[1], (int)t[2], (int)t[3], 0, 0, 0, 0};
  constexpr int kFp4 = 4, kBf6 = 3;
  d = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, q.hi, d, kFp4, kBf6, P % 4, q.a[P / 4],
                                                       1, q.b);
  d = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, q.lo, d, kFp4, kBf6, P % 4, q.a[P / 4],
                                                       0, q.b);
}

// Position P of one set, then the positions above it. eq[e][c] (exponent == e
// of code dword c) is formed at position 6 - e, the first that needs it, and
// lives for K + 1 positions. jb[b][c]: mantissa bit b of code dword c at bit 1.
template <int K, int P>
__device__ __forceinline__ void planes_from(const CodeBits (&cb)[4], uint32_t (&eq)[7][4],
                                            const uint32_t (*jb)[4], uint32_t m22,
                                            const PlaneQuery& q, f32x4& d) {
  uint32_t t[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if constexpr (P <= 6) eq[6 - P][c] = exponent_is<P <= 6 ? 6 - P : 0>(cb[c]);
    uint32_t m = 0;
    bool any = false;
    if constexpr (P >= K) {  // the leading one: e = K + 6 - P
      m = eq[P >= K ? K + 6 - P : 0][c];
      any = true;
    }
#pragma unroll
    for (int b = 0; b < K; ++b) {
      const int e = b + 6 - P;
      if (e < 0 || e > 6) continue;
      const uint32_t me = eq[e < 0 ? 0 : e > 6 ? 6 : e][c];
      m = any ? __builtin_amdgcn_bitop3_b32(m, me, jb[b][c], kAndOrTable) : (me & jb[b][c]);
      any = true;
    }
    t[c] = __builtin_amdgcn_bitop3_b32(m22, m, cb[c].sign, kMaskOrTable);
  }
  add_plane<P>(t, q, d);
  __builtin_amdgcn_sched_barrier(0);  // one plane's operand at a time: registers
  if constexpr (P < K + 6) planes_from<K, P + 1>(cb, eq, jb, m22, q, d);
}

// Scores (int32 values as fp32, at head-room F) of one set: w the lane's 16
// code bytes, pl its 32 mantissa bits of each plane. m22: 0x22222222 in a
// VGPR (an operand from an SGPR would put the op in the slower issue class).
template <int K>
__device__ __forceinline__ f32x4 score_set(const uint32_t (&w)[4], const uint32_t* pl,
                                           uint32_t m22, const PlaneQuery& q) {
  uint32_t c4[4];
  if constexpr (K == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) c4[c] = w[c];
  } else {
    transpose_codes(w, c4);
  }
  CodeBits cb[4];
  uint32_t eq[7][4], jb[K > 0 ? K : 1][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cb[c] = code_bits(c4[c]);
#pragma unroll
    for (int k = 0; k < K; ++k) jb[k][c] = c == 0 ? pl[k] << 1 : pl[k] >> (c - 1);
  }
  f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
  planes_from<K, 0>(cb, eq, jb, m22, q, d);
  return d;
}

// One element of q^ of one head as hi and lo (q^ = 16 hi + lo, hi in [-8, 8],
// lo in [-8, 7]) at its place in the operand order; the head's 64 elements
// make two blocks of 32.
template <int K>
__device__ __forceinline__ void store_query_element(int qi, int m, _Float16* hi_row,
                                                    _Float16* lo_row) {
  const int hi = (qi + 8) >> 4;
  const int at = (m & 32) + plane_order<K>(m & 31);
  hi_row[at] = (_Float16)hi;
  lo_row[at] = (_Float16)(qi - 16 * hi);
}

// The lane's query operands from the halves in LDS ([head][64] each) and the
// block scales for head-room F.
template <int G>
__device__ __forceinline__ PlaneQuery load_plane_query(const _Float16 (*hi)[kDim],
                                                       const _Float16 (*lo)[kDim], int frac_bits) {
  const int lane = lane_id(), col = lane & 15, blk = lane >> 4, h = col & 7;
  const bool used = (col >> 3) == (blk >> 1) && h < G;
  const int row = h < G ? h : 0;
  half32 vh, vl;
  const uint4* ph = reinterpret_cast<const uint4*>(&hi[row][32 * (blk & 1)]);
  const uint4* pl = reinterpret_cast<const uint4*>(&lo[row][32 * (blk & 1)]);
  struct Block {
    uint4 v[4];
  };
  Block bh, bl;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bh.v[i] = ph[i];
    bl.v[i] = pl[i];
  }
  vh = __builtin_bit_cast(half32, bh);
  vl = __builtin_bit_cast(half32, bl);
  const u32x6 h6 = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(vh, 1.0f);
  const u32x6 l6 = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(vl, 1.0f);
  PlaneQuery q;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    q.hi[i] = (i < 6 && used) ? (int)h6[i < 6 ? i : 0] : 0;
    q.lo[i] = (i < 6 && used) ? (int)l6[i < 6 ? i : 0] : 0;
  }
  // e8m0 exponents (bias 127): 2^(p + F - 6) for position p, 2^4 for hi
  const uint32_t base = (uint32_t)(127 + frac_bits - kExpMax) * 0x01010101u + 0x03020100u;
#pragma unroll
  for (int i = 0; i < 3; ++i) q.a[i] = (int)(base + (uint32_t)i * 0x04040404u);
  q.b = 127 | ((127 + 4) << 8);
  return q;
}

}  // namespace potattn
