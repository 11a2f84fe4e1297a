// Key encoders for gfx950: fp16 key rows -> PoT / PoT-Mk codes (Sec. II-A,
// II-D) and -> INT8 uniform codes (the multiply-accumulate comparator).
//
// The bulk PoT encoder works on 8 key rows per wavefront at a time: lane l
// takes row l / 8 of the group and elements 8g .. 8g + 7 of it (g = l % 8),
// so a row is one 16-byte load per lane over 8 lanes and its code word g (the
// 8 nibbles of those elements) is one 4-byte store; the row scale is a max over
// 8 values and three DPP lane exchanges. With the optional Walsh-Hadamard
// rotation it rotates them by fp64 butterflies or, over many rows, 16 at a time
// on the matrix cores, exactly (rows with elements above 4096 by the
// butterflies). Each ratio |x| / s is correctly rounded from one reciprocal per
// row (a Newton-corrected hardware reciprocal, then Markstein's correction of the
// quotient). PoT-4 then takes its code from the ratio's bits with integer
// operations (an add that carries into the exponent exactly above the cut point,
// a shift and a clamp) and its sign bits from the inputs' sign bits eight at a
// time by byte permutes; PoT-Mk (K > 0) squares the mantissa against the product
// of its two grid points. (The INT8 comparator's encoder takes the same shape; the
// fused per-token append in the decode kernel encodes one row per wavefront, one
// element per lane.)
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pot_device.hpp"
#include "pot_launch.hpp"

namespace potattn {

namespace {

// Largest fp32 strictly below sqrt(num / den^2) for num not a perfect square,
// with num / den^2 in [1, 4): the value is M * 2^-23 with M the integer part
// of sqrt(num * 2^46 / den^2) (exact integer square root).
float rd_sqrt_ratio(uint64_t num, uint64_t den) {
  // R * 2^46 = num * 2^46 / den^2; den is a power of two <= 16 so the
  // division is exact.
  unsigned __int128 v = ((unsigned __int128)num << 46) / ((unsigned __int128)den * den);
  uint64_t m = (uint64_t)std::sqrt((long double)v);
  while ((unsigned __int128)m * m > v) --m;
  while ((unsigned __int128)(m + 1) * (m + 1) <= v) ++m;
  return std::ldexp((float)m, -23);  // m < 2^25 so exact in fp32
}

EncodeTables make_encode_tables(int mant_bits) {
  EncodeTables t{};
  const uint64_t n = 1ull << mant_bits;
  for (uint64_t i = 0; i < n; ++i) t.cut[i] = rd_sqrt_ratio((n + i) * (n + i + 1), n);
  for (uint64_t i = n; i < 16; ++i) t.cut[i] = INFINITY;
  // 2^-(E+1/2) = sqrt(2) * 2^-7: RD of sqrt(2) scaled by an exact power of two.
  t.zero_cut = std::ldexp(rd_sqrt_ratio(2, 1), -(kExpMax + 1));
  t.mant_bits = mant_bits;
  return t;
}

}  // namespace

const EncodeTables& encode_tables(int mant_bits) {
  static const EncodeTables all[5] = {make_encode_tables(0), make_encode_tables(1),
                                      make_encode_tables(2), make_encode_tables(3),
                                      make_encode_tables(4)};
  return all[mant_bits];
}

// The row-per-wave kernels below step over rows with the grid's stride: a
// launch has at most kMaxGrid workgroups, since a dispatch is limited to
// 2^32 work-items per dimension (2^26 rows of one wave each).
constexpr int64_t kMaxGrid = 1 << 20;
// Workgroups of the bulk encoders: eight per CU, each wave looping over row
// groups, and up to 32 per CU while every wave still has eight groups (2 M rows:
// k = 0 66 -> 64 us, k = 4 90 -> 85; 131072 rows, one group per wave instead
// of two: 7.0 -> 7.4). Past that many rows the kernels that the memory stream bounds
// (PoT-4 and INT8, not rotated) go back to eight, whose waves pass over memory in
// a narrower window (8.39 M rows: k = 0 292 -> 269 us, INT8 357 -> 327; 4.19 M 133 ->
// 131, 162 -> 155); the others keep 32 (k = 1 321 against 336, rotated k = 4 453
// against 462).
constexpr int64_t kEncodeGrid = 256 * 8, kEncodeGridMax = 256 * 32;
inline uint32_t encode_grid(int64_t n_rows, bool stream_bound) {
  const int64_t groups = (n_rows + 7) / 8, wg = kBlock / 64;
  int64_t cap = std::max(kEncodeGrid, std::min(kEncodeGridMax, groups / (8 * wg)));
  if (stream_bound && groups > 8 * wg * kEncodeGridMax) cap = kEncodeGrid;
  return (uint32_t)std::min((groups + wg - 1) / wg, cap);
}

// Maximum over the 8 lanes of an aligned group (lane & ~7) of non-negative,
// non-NaN floats, compared as their bit patterns: swap neighbours, swap
// pairs, then the mirror image inside each half row (a maximum does not care
// which lane of the other quad it meets).
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xF, 0xF, true);
}
__device__ __forceinline__ float max_over_8_lanes(float v) {
  constexpr int kQuadSwap1 = 0xB1, kQuadSwap2 = 0x4E, kRowHalfMirror = 0x141;
  uint32_t b = __float_as_uint(v);
  b = max(b, dpp_u32<kQuadSwap1>(b));
  b = max(b, dpp_u32<kQuadSwap2>(b));
  return __uint_as_float(max(b, dpp_u32<kRowHalfMirror>(b)));
}

// Scales whose reciprocal takes the fast path: [2^-126, 2^126] (no NaN,
// sign, infinity or subnormal reciprocal), by one unsigned compare.
__device__ __forceinline__ bool recip_in_range(float s) {
  return __float_as_uint(s) - 0x00800000u <= 0x7E800000u - 0x00800000u;
}

// RN(1 / s) for s in [2^-126, 2^126]: v_rcp_f32 is within one ulp, and one
// Newton step with fused multiply-adds then rounds correctly for every start
// within an ulp, except for an all-ones mantissa, s = (2 - 2^-23) 2^k, where
// the step can land on a tie: there 1/s = 2^-(k+1) (1 + 2^-24 + 2^-48 ...)
// rounds to 2^-(k+1) (1 + 2^-23), whose bits are 0x7E800001 minus the
// exponent field of s. (Checked over every mantissa of one binade and every
// start within an ulp.)
__device__ __forceinline__ float recip_rn(float s) {
  const float r0 = __builtin_amdgcn_rcpf(s);
  const float r1 = __builtin_fmaf(__builtin_fmaf(-s, r0, 1.0f), r0, r0);
  const uint32_t sb = __float_as_uint(s);
  return ((sb & 0x007FFFFFu) == 0x007FFFFFu) ? __uint_as_float(0x7E800001u - (sb & 0x7F800000u))
                                               : r1;
}

inline uint32_t bounded_grid(int64_t blocks) {
  return (uint32_t)(blocks < kMaxGrid ? blocks : kMaxGrid);
}

// Clamp to [0, 1] with NaN mapped to 0: folds into the producing
// instruction's clamp bit (the DX10 clamp mode, on for compute kernels).
__device__ __forceinline__ float clamp01(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }

// Nibble masks of 8 signs: nibble i of the result is 0xF where bytes a (signs
// 0..3) and b (signs 4..7), each 0x00 or 0xFF, say sign i is set.
__device__ __forceinline__ uint32_t sign_nibbles(uint32_t a, uint32_t b) {
  const uint32_t even = __builtin_amdgcn_perm(b, a, 0x06040200u);  // signs 0 2 4 6
  const uint32_t odd = __builtin_amdgcn_perm(b, a, 0x07050301u);   // signs 1 3 5 7
  return (even & 0x0F0F0F0Fu) | (odd & 0xF0F0F0F0u);
}

// PoT-4 code word of 8 elements from their clamped ratios c_i = min(RN(|x_i|
// / s), 1) (0 for NaN) and sign masks. With c = (1 + M 2^-23) 2^(E-127) and
// the cut point RD(sqrt 2) = 1 + Mc 2^-23, the log-nearest exponent is
// e = 127 - (E + [M > Mc]) and the ratio is at or below the zero cut
// RD(sqrt 2) 2^-(E_max+1) exactly when E + [M > Mc] <= 127 - (E_max + 1).
// Adding 2^23 - 1 - Mc to the bits carries into the exponent exactly when
// M > Mc, so G = clamp((bits + 2^23 - 1 - Mc - (120 << 23)) >> 23, 0, 7)
// is 0 for zero and 7 - e otherwise (E_max = 6, c <= 1 saturates at e = 0).
// The word holds 7 - G per nibble, with the sign bit where G > 0.
__device__ __forceinline__ uint32_t pot4_word(const float (&c)[8], uint32_t sgn, uint32_t cst) {
  uint32_t w = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int t = (int)(__float_as_uint(c[i]) + cst) >> 23;
    const uint32_t gi = (uint32_t)min(max(t, 0), 7);
    w |= gi << (4 * i);
  }
  return (w ^ 0x77777777u) | (sgn & (w + 0x77777777u) & 0x88888888u);
}

// PoT-Mk code word and mantissa-plane bytes of 8 elements from their clamped
// half ratios v_i = min(RN(|x_i| / (2 s)), 1) (0 for NaN): ratios up to 2 on
// the unit interval, so that caller scales with |x| / s in [1, 2) still see
// their mantissa. With v = (1 + M 2^-23) 2^(E-127) and m = 1 + M 2^-23, the top
// K bits of M are j0, t = floor(m 2^k) = 2^k + j0, and m lies above the cut
// between grid points j0 and j0 + 1, RD(sqrt(t (t + 1)) / 2^k), exactly when
// (m 2^k)^2 > t (t + 1) (the root is irrational), which one fused multiply-add
// decides by its sign. E and j0 stand next to each other in v's bits, so adding
// that decision to the bits above them carries from the last grid point into
// the next binade by itself: u = (E - 119) 2^k + j0 + [above], clamped to 2^k
// .. 2^(k+3) - 1 (ratios past the top value and below the smallest magnitude)
// and 0 for a ratio at or below the zero cut, holds 7 - e above the mantissa.
// (Deciding exponent and mantissa apart took about 20 operations per element,
// this 14: 2 M rows k = 1 85 -> 81, k = 4 109 -> 96 us.) The u's are packed a byte
// each (bytes of a: elements 0..3, of b: 4..7), so exponents and mantissas come
// apart four at a time, and the mantissa nibbles (bit i of plane b: bit b of
// element i's j) become plane bytes by two exchanges of bits between bytes, all
// planes at once (a nibble each and a bit gather per plane: k = 1 80, k = 4 95 us;
// now 77 and 83).
// Returns the code word (signs as in pot4_word); byte b of planes is plane b's,
// bytes from K on hold no plane.
template <int K>
__device__ __forceinline__ uint32_t potmk_word(const float (&v)[8], uint32_t sgn,
                                               uint32_t zc_half, uint32_t& planes) {
  constexpr int n = 1 << K;
  uint32_t a = 0, b = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t vb = __float_as_uint(v[i]);
    const float mn = __uint_as_float((vb & 0x007FFFFFu) | ((127u + K) << 23));  // m 2^k
    const float t = truncf(mn);                  // 2^k + j0
    const float p = __builtin_fmaf(t, t, t);     // t (t + 1) <= 992, exact
    const int above = __builtin_fmaf(mn, mn, -p) > 0.0f ? 1 : 0;
    const int q = ((int)(vb - (119u << 23)) >> (23 - K)) + above;
    uint32_t u = (uint32_t)min(max(q, n), 8 * n - 1);
    u = vb > zc_half ? u : 0u;
    if (i < 4) a |= u << (8 * i);
    else b |= u << (8 * i - 32);
  }
  const uint32_t even = __builtin_amdgcn_perm(b, a, 0x06040200u);
  const uint32_t odd = __builtin_amdgcn_perm(b, a, 0x07050301u);
  const uint32_t w = ((even >> K) & 0x07070707u) | (((odd >> K) & 0x07070707u) << 4);
  // bit 8c + 4h + b of x: bit b of element 4h + c; exchange index bit 0 with 3, 1 with 4
  uint32_t x = (a & 0x0F0F0F0Fu) | ((b << 4) & 0xF0F0F0F0u);
  uint32_t t = (x ^ (x >> 7)) & 0x00AA00AAu;
  x ^= t ^ (t << 7);
  t = (x ^ (x >> 14)) & 0x0000CCCCu;
  planes = x ^ t ^ (t << 14);
  return (w ^ 0x77777777u) | (sgn & (w + 0x77777777u) & 0x88888888u);
}

// 8 elements 8g .. 8g + 7 (g = lane % 8) of a row from their fp16 words, with
// the optional rotation over the row's 8 lanes: butterflies over bits 0..2 of
// the element in registers, over bits 0..2 of g across lanes; fp16 inputs keep
// every fp64 sum exact.
template <bool HAD>
__device__ __forceinline__ void unpack_row(const uint32_t (&w4)[4], int lane, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __half2float(__ushort_as_half((unsigned short)(w4[i] & 0xFFFFu)));
    x[2 * i + 1] = __half2float(__ushort_as_half((unsigned short)(w4[i] >> 16)));
  }
  if constexpr (HAD) {
    const double sign1 = butterfly_sign<1>(lane), sign2 = butterfly_sign<2>(lane),
                 sign4 = butterfly_sign<4>(lane);
    double v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (double)x[i];
#pragma unroll
    for (int h = 1; h < 8; h <<= 1)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & h) == 0) {
          const double p = v[i], q = v[i + h];
          v[i] = p + q;
          v[i + h] = p - q;
        }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = butterfly<1>(v[i], sign1);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = butterfly<2>(v[i], sign2);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = butterfly<4>(v[i], sign4);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (float)(v[i] * 0.125);
  }
}

// The plane bytes of each lane of a quad (byte b: plane b; code words 4h .. 4h + 3 of a row)
// to one dword of plane j in lane j: a 4 x 4 byte transpose by two DPP moves
// and byte permutes, for one dword store per lane. (With a byte store per lane
// and plane 2 M rows at k = 4 took 117 us, so 108.)
__device__ __forceinline__ uint32_t quad_planes(uint32_t w, int lane) {
  w = __builtin_amdgcn_perm(lane_xor_u32<1>(w), w, lane & 1 ? 0x03070105u : 0x06020400u);
  return __builtin_amdgcn_perm(lane_xor_u32<2>(w), w, lane & 2 ? 0x03020706u : 0x05040100u);
}

// The bits-to-G offset of pot4_word (Mc from the fp32 cut point) and half the
// zero cut.
struct CutBits {
  uint32_t cst, zc_half;
};
__device__ __forceinline__ CutBits cut_bits(const EncodeTables& tab) {
  return {0x007FFFFFu - (__float_as_uint(tab.cut[0]) & 0x007FFFFFu) - (120u << 23),
          __float_as_uint(tab.zero_cut) - (1u << 23)};
}

// Sign nibbles of 8 fp32 numbers (selector 9 / 11: bit 31 of the low / high
// source, 12: zero byte).
__device__ __forceinline__ uint32_t float_signs(const float* x) {
  uint32_t xb[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) xb[i] = __float_as_uint(x[i]);
  return sign_nibbles(__builtin_amdgcn_perm(xb[1], xb[0], 0x0C0C0B09u) |
                          __builtin_amdgcn_perm(xb[3], xb[2], 0x0B090C0Cu),
                      __builtin_amdgcn_perm(xb[5], xb[4], 0x0C0C0B09u) |
                          __builtin_amdgcn_perm(xb[7], xb[6], 0x0B090C0Cu));
}

// A row's scale as its elements use it.
// The clamped ratio c = min(RN(|x| / ss), 1) per element (ss = s for PoT-4, 2 s
// for PoT-Mk), NaN -> 0 (zero code), comes from one correctly rounded reciprocal
// per row; other scales (zero, negative, NaN, infinite, or too small or too
// large for a normal reciprocal) divide instead. The quotient q = RN(|x| r) is
// clamped too: min(q, 1) is still within an ulp of a quotient below 1, any q >=
// 1 gives c >= 1, and an infinite or NaN q (infinite or NaN x) cannot poison
// the residual.
struct RowScale {
  float s, ss, r;
  bool fast;
};
template <int K>
__device__ __forceinline__ RowScale row_scale(float s) {
  const float ss = K == 0 ? s : 2.0f * s;
  return {s, ss, recip_rn(ss), recip_in_range(ss)};
}

// Code word and plane bytes (byte b: plane b) of 8 elements.
template <int K>
__device__ __forceinline__ uint32_t encode_word(const float* x, const RowScale& sc, uint32_t sgn,
                                                const CutBits& cut, uint32_t& planes) {
  float c[8];
  if (sc.fast) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float a = fabsf(x[i]);
      const float q = clamp01(a * sc.r);
      c[i] = clamp01(__builtin_fmaf(__builtin_fmaf(-q, sc.ss, a), sc.r, q));
    }
  } else {
    // (|x| / 2) / s rounds as |x| / (2 s) and stays finite-safe for huge s
#pragma unroll
    for (int i = 0; i < 8; ++i)
      c[i] = (sc.s > 0.0f) ? clamp01((K == 0 ? fabsf(x[i]) : fabsf(x[i]) * 0.5f) / sc.s) : 0.0f;
  }
  if constexpr (K == 0) return pot4_word(c, sgn, cut.cst);
  else return potmk_word<K>(c, sgn, cut.zc_half, planes);
}

// The arguments of one encode launch.
struct EncodeArgs {
  const __half* k;
  int64_t n_rows, out_stride;
  int scale_mode;
  float* key_scale;
  uint8_t* codes_se;
  uint8_t* codes_m;
};

// Rows row0 .. row0 + 7 (row0 uniform) by the calling wave.
template <int K, bool HAD>
__device__ __forceinline__ void encode_rows8(const EncodeArgs& a, int64_t row0,
                                             const CutBits& cut) {
  const int lane = lane_id(), g = lane & 7, rl = lane >> 3;
  // lane parts of the addresses; a group's bases are uniform
  const uint32_t in_off = (uint32_t)(rl * kDim * 2 + 16 * g);
  const int64_t out_row = (int64_t)rl * a.out_stride;
  const int64_t se_off = out_row * (kDim / 2) + 4 * g;
  const bool valid = row0 + rl < a.n_rows;  // uniform over the row's 8 lanes
  uint4 raw = make_uint4(0u, 0u, 0u, 0u);
  if (valid)
    raw = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.k) + row0 * kDim * 2 +
                                          in_off);
  const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
  float x[8];
  unpack_row<HAD>(w4, lane, x);
  const int64_t orow = (row0 * a.out_stride) + out_row;
  float s;
  if (a.scale_mode == 0) {
    // max |x| ignoring NaN (0 for a row of zeros and NaNs)
    s = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s = fmaxf(s, fabsf(x[i]));
    s = max_over_8_lanes(s);
  } else {
    s = valid ? a.key_scale[orow] : 0.0f;
  }
  // sign bits of the inputs: selectors 8..11 are bits 15, 31 of the low and of
  // the high source
  const uint32_t sgn =
      HAD ? float_signs(x)
          : sign_nibbles(__builtin_amdgcn_perm(w4[1], w4[0], 0x0B0A0908u),
                         __builtin_amdgcn_perm(w4[3], w4[2], 0x0B0A0908u));
  uint32_t planes = 0;
  const uint32_t word = encode_word<K>(x, row_scale<K>(s), sgn, cut, planes);
  uint32_t pq = 0;
  if constexpr (K > 0) pq = quad_planes(planes, lane);
  if (valid) {
    const int64_t urow = row0 * a.out_stride;  // uniform part of orow
    *reinterpret_cast<uint32_t*>(a.codes_se + urow * (kDim / 2) + se_off) = word;
    if constexpr (K > 0) {
      // lane j < K of a quad: plane j's bytes of the quad's four code words
      if ((g & 3) < K)
        *reinterpret_cast<uint32_t*>(a.codes_m + orow * 8 * K + 8 * (g & 3) + 4 * (g >> 2)) = pq;
    }
    if (a.scale_mode == 0 && g == 0) a.key_scale[orow] = s;
  }
}

template <int K, bool HAD>
__global__ __launch_bounds__(kBlock) void encode_pot_kernel(const EncodeArgs a,
                                                            const EncodeTables tab) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t groups = (uint32_t)((a.n_rows + 7) / 8);
  const uint32_t stride = gridDim.x * (kBlock / 64);
  const CutBits cut = cut_bits(tab);
  for (uint32_t grp = blockIdx.x * (kBlock / 64) + wave; grp < groups; grp += stride)
    // the group index as an opaque uniform value: addresses are rebuilt from
    // it each trip as scalar bases plus the fixed lane offsets
    encode_rows8<K, HAD>(a, (int64_t)__builtin_amdgcn_readfirstlane(grp) * 8, cut);
}

// Rotated keys: the 64 x 64 Hadamard matrix on the matrix cores, 16 rows per
// wave at a time, exactly. Every fp16 element x is split as hi + lo: lo is what
// rounding min(|x|, 16) to a multiple of 2^-5 leaves (below 2^-6, a multiple of
// 2^-24; 0 from 16 on) and hi = x - lo is a multiple of 2^-6; both are fp16
// numbers. v_mfma_f32_16x16x32_f16 with +-1 then sums 64 hi's (below 2^18 if
// |x| <= 4096: exact in fp32 with unit 2^-6) and 64 lo's (as lo 2^12, which is
// never subnormal: at most 2^12 with unit 2^-12), and fma(LO, 2^-12, HI) is the
// rotation's one rounding, as fp64 butterflies and a conversion round it. Rows
// with a larger, infinite or NaN element take the butterflies. A = H with rows
// in such an order that lane l gets elements 16 (l / 16) ..+15 of row l % 16: two
// code words. Butterflies cost about 250 VALU operations per 8 rows, this 45 per
// 16 and 16 matrix instructions. Butterflies -> here: 131072 rows k = 0 10.5 -> 9.6,
// k = 4 14.2 -> 13.5 (now 12.4); 2 M rows k = 0 102 -> 85, k = 4 150 -> 130 us
// (now 116). Up to kButterflyRows rows, where a wave has one group either way, the
// butterflies are the shorter chain (graph replays, k = 0 and 4: 1 row 2.2 and 2.5 us
// against 2.8 and 3.1 here, 4096 rows 2.5 and 2.8 against 3.0 and 3.4, 24576 rows 4.0
// and 4.6 against 4.2 and 5.0; 32768 rows 4.4 and 5.2 against 4.4 and 5.1).
typedef _Float16 half8e __attribute__((ext_vector_type(8)));
typedef _Float16 half2e __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2e __attribute__((ext_vector_type(2)));
typedef float f32x4e __attribute__((ext_vector_type(4)));
constexpr uint32_t kExactHalf = 0x6C00;  // 4096 in fp16
constexpr int64_t kButterflyRows = 24576;

// amdgpu_waves_per_eu(4): 98..104 VGPRs; at five waves the matrix spills.
template <int K>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
void encode_pot_had_kernel(const EncodeArgs a, const EncodeTables tab) {
  const int lane = lane_id(), col = lane & 15, blk = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t groups = (uint32_t)((a.n_rows + 15) / 16);
  const uint32_t stride = gridDim.x * (kBlock / 64);
  const CutBits cut = cut_bits(tab);
  // Row col of block nb of H is element m = 16 (col / 4) + 4 nb + col % 4, its
  // columns are k = 32 kb + 8 blk + j, and the sign is the parity of m & k: bits
  // 0..2 of j against col % 4 and nb's low bit, k's bits 3, 4 against nb's high
  // bit and bit 2 of col, bit 5 against bit 3 of col (h5, at kb = 1).
  constexpr uint32_t kSigns = 0x80008000u;
  const uint32_t h5 = (col & 8) ? kSigns : 0u;
  uint32_t h[4][4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const bool odd = (((nb >> 1) & blk) ^ ((col >> 2) & (blk >> 1))) & 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)  // j = 2q, 2q + 1
      h[nb][q] = 0x3C003C00u ^ (odd ? kSigns : 0u) ^ ((col & 1) ? 0x80000000u : 0u) ^
                 ((q & 1) && (col & 2) ? kSigns : 0u) ^ ((q & 2) && (nb & 1) ? kSigns : 0u);
  }
  for (uint32_t iv = blockIdx.x * (kBlock / 64) + wave; iv < groups; iv += stride) {
    const int64_t row0 = (int64_t)__builtin_amdgcn_readfirstlane(iv) * 16;
    const bool valid = row0 + col < a.n_rows;
    uint4 raw[2] = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u)};
    if (valid) {
      const char* src = reinterpret_cast<const char*>(a.k) + row0 * kDim * 2 + col * kDim * 2;
      raw[0] = *reinterpret_cast<const uint4*>(src + 16 * blk);
      raw[1] = *reinterpret_cast<const uint4*>(src + 64 + 16 * blk);
    }
    const uint32_t w8[8] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w,
                            raw[1].x, raw[1].y, raw[1].z, raw[1].w};
    u16x2e big = {0, 0};
#pragma unroll
    for (int i = 0; i < 8; ++i)
      big = __builtin_elementwise_max(big, __builtin_bit_cast(u16x2e, w8[i] & 0x7FFF7FFFu));
    if (__any(big[0] > kExactHalf || big[1] > kExactHalf)) {
      encode_rows8<K, true>(a, row0, cut);
      if (row0 + 8 < a.n_rows) encode_rows8<K, true>(a, row0 + 8, cut);
      continue;
    }
    uint32_t hw[8], lw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const half2e v = __builtin_bit_cast(half2e, w8[i]);
      const half2e c16 = {(_Float16)16.0f, (_Float16)16.0f},
                   c48 = {(_Float16)48.0f, (_Float16)48.0f},
                   c4k = {(_Float16)4096.0f, (_Float16)4096.0f};
      const half2e y = __builtin_elementwise_max(__builtin_elementwise_min(v, c16), -c16);
      const half2e lo = y - ((y + c48) - c48);
      hw[i] = __builtin_bit_cast(uint32_t, v - lo);
      lw[i] = __builtin_bit_cast(uint32_t, lo * c4k);
    }
    float x[16];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      f32x4e dh = {0.0f, 0.0f, 0.0f, 0.0f}, dl = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const half8e bh = __builtin_bit_cast(
            half8e, make_uint4(hw[4 * kb], hw[4 * kb + 1], hw[4 * kb + 2], hw[4 * kb + 3]));
        const half8e bl = __builtin_bit_cast(
            half8e, make_uint4(lw[4 * kb], lw[4 * kb + 1], lw[4 * kb + 2], lw[4 * kb + 3]));
        const uint32_t f = kb ? h5 : 0u;
        const half8e ha = __builtin_bit_cast(
            half8e, make_uint4(h[nb][0] ^ f, h[nb][1] ^ f, h[nb][2] ^ f, h[nb][3] ^ f));
        dh = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha, bh, dh, 0, 0, 0);
        dl = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha, bl, dl, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[4 * nb + r] = __fmul_rn(__builtin_fmaf(dl[r], 0x1p-12f, dh[r]), 0.125f);
    }
    const int64_t orow = (row0 + col) * a.out_stride;
    float s;
    if (a.scale_mode == 0) {
      s = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s = fmaxf(s, fabsf(x[i]));
      uint32_t b = __float_as_uint(s);  // not negative: compares as its bits
      const auto r16 = __builtin_amdgcn_permlane16_swap(b, b, false, false);
      b = max(r16[0], r16[1]);
      const auto r32 = __builtin_amdgcn_permlane32_swap(b, b, false, false);
      s = __uint_as_float(max(r32[0], r32[1]));
    } else {
      s = valid ? a.key_scale[orow] : 0.0f;
    }
    const RowScale sc = row_scale<K>(s);
    uint32_t p0 = 0, p1 = 0;
    uint2 word;
    word.x = encode_word<K>(x, sc, float_signs(x), cut, p0);
    asm volatile("" : "+v"(word.x));  // one word at a time: registers
    word.y = encode_word<K>(x + 8, sc, float_signs(x + 8), cut, p1);
    // 16 bits per plane and lane to 8 bytes of plane j in the lanes of block j:
    // plane bits against block bits, by the lane-half and the row exchange
    uint32_t t[2] = {0u, 0u};
    if constexpr (K > 0) {
      t[0] = __builtin_amdgcn_perm(p1, p0, 0x05010400u);
      t[1] = __builtin_amdgcn_perm(p1, p0, 0x07030602u);
      const auto r32 = __builtin_amdgcn_permlane32_swap(t[0], t[1], false, false);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const auto r16 = __builtin_amdgcn_permlane16_swap(r32[i], r32[i], false, false);
        t[i] = __builtin_amdgcn_perm(r16[1], r16[0], (blk & 1) ? 0x07060302u : 0x05040100u);
      }
    }
    if (valid) {
      *reinterpret_cast<uint2*>(a.codes_se + orow * (kDim / 2) + 8 * blk) = word;
      if constexpr (K > 0) {
        if (blk < K)
          *reinterpret_cast<uint2*>(a.codes_m + orow * 8 * K + 8 * blk) = make_uint2(t[0], t[1]);
      }
      if (a.scale_mode == 0 && blk == 0) a.key_scale[orow] = s;
    }
  }
}

// INT8 uniform codes, 8 rows per wave as the PoT encoder (one row per wave and
// element per lane took 20.7 us for 131072 rows and 333 us for 2 M; now 7.4
// and 76 us).
template <bool HAD>
__global__ __launch_bounds__(kBlock) void encode_int8_kernel(
    const __half* __restrict__ k, int64_t n_rows, int64_t out_stride,
    float* __restrict__ key_scale, int8_t* __restrict__ codes) {
  const int lane = lane_id(), g = lane & 7, rl = lane >> 3;
  const int64_t groups = (n_rows + 7) / 8, stride = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t grp = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); grp < groups;
       grp += stride) {  // uniform per wave
    const int64_t row = grp * 8 + rl;
    const bool valid = row < n_rows;  // uniform over the row's 8 lanes
    uint4 raw = make_uint4(0u, 0u, 0u, 0u);
    if (valid) raw = *reinterpret_cast<const uint4*>(k + row * kDim + 8 * g);
    const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
    float x[8];
    unpack_row<HAD>(w4, lane, x);
    // fmaxf throughout: NaN only if the whole row is
    float amax = fabsf(x[0]);
#pragma unroll
    for (int i = 1; i < 8; ++i) amax = fmaxf(amax, fabsf(x[i]));
    amax = fmaxf(amax, __uint_as_float(lane_xor_u32<1>(__float_as_uint(amax))));
    amax = fmaxf(amax, __uint_as_float(lane_xor_u32<2>(__float_as_uint(amax))));
    amax = fmaxf(amax, __uint_as_float(lane_xor_u32<4>(__float_as_uint(amax))));
    const bool zero = amax == 0.0f;
    const float inv = 127.0f / amax;  // correctly rounded divisions
    const float step = zero ? 0.0f : amax / 127.0f;
    uint32_t w[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i)
      w[i / 4] |= ((uint32_t)(zero ? 0 : quantize_int8(x[i], inv)) & 0xFFu) << (8 * (i & 3));
    if (valid) {
      const int64_t orow = row * out_stride;
      *reinterpret_cast<uint2*>(codes + orow * kDim + 8 * g) = make_uint2(w[0], w[1]);
      if (g == 0) key_scale[orow] = step;
    }
  }
}

// Value-cache store: token t of sequence s, dim d lives at
// ((s * t_cap + (t/8)*8) * 64 + d * 8 + t % 8) halves. One thread per
// (sequence, 8-token group, dim) gathers the group's 8 tokens of its dim and
// writes them as one 16-byte word (or only the tokens inside [t0, t0+n_tok)
// at the ends of the range). i indexes (sequence, group, dim).
__device__ __forceinline__ void store_value_group(const uint16_t* __restrict__ src, int64_t n_tok,
                                                  int64_t t_cap, int64_t t0, int64_t g_first,
                                                  int64_t n_groups, uint16_t* __restrict__ dst,
                                                  int64_t i) {
  const int d = (int)(i % kDim);
  const int64_t sg = i / kDim;
  const int64_t s = sg / n_groups, g = g_first + sg % n_groups;
  uint16_t* out = dst + (s * t_cap + g * 8) * kDim + d * 8;
  uint16_t vals[8];
  bool full = true;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int64_t t = g * 8 + k;
    const bool in = t >= t0 && t < t0 + n_tok;
    full = full && in;
    vals[k] = in ? src[(s * n_tok + (t - t0)) * kDim + d] : (uint16_t)0;
  }
  if (full) {
    uint4 w;
    w.x = vals[0] | ((uint32_t)vals[1] << 16);
    w.y = vals[2] | ((uint32_t)vals[3] << 16);
    w.z = vals[4] | ((uint32_t)vals[5] << 16);
    w.w = vals[6] | ((uint32_t)vals[7] << 16);
    *reinterpret_cast<uint4*>(out) = w;
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t t = g * 8 + k;
      if (t >= t0 && t < t0 + n_tok) out[k] = vals[k];
    }
  }
}

__global__ __launch_bounds__(256) void store_values_kernel(
    const uint16_t* __restrict__ src, int64_t n_seq, int64_t n_tok, int64_t t_cap, int64_t t0,
    int64_t g_first, int64_t n_groups, uint16_t* __restrict__ dst) {
  const int64_t n = n_seq * n_groups * kDim;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    store_value_group(src, n_tok, t_cap, t0, g_first, n_groups, dst, i);
}

hipError_t launch_store_values(const uint16_t* src, int64_t n_seq, int64_t n_tok, int64_t t_cap,
                               int64_t t0, uint16_t* dst, hipStream_t stream) {
  if (n_seq == 0 || n_tok == 0) return hipSuccess;
  const int64_t g_first = t0 / 8, g_last = (t0 + n_tok - 1) / 8;
  const int64_t n_groups = g_last - g_first + 1;
  const int64_t n = n_seq * n_groups * kDim;
  const int64_t grid = (n + 255) / 256;
  hipLaunchKernelGGL(store_values_kernel, dim3(bounded_grid(grid)), dim3(256), 0, stream, src,
                     n_seq, n_tok, t_cap, t0, g_first, n_groups, dst);
  return hipGetLastError();
}

// INT8 value store: token t of sequence s, dim d at byte
// (s * t_cap + (t / 8) * 8) * 64 + d * 8 + t % 8. One wave per 8-token group:
// lane l loads 16 bytes of token l / 8 (dims 8 (l % 8) ..+7), so a group is one
// contiguous KiB, finds the token's exponent with its 8 lanes and quantises.
// The 8 x 8 byte blocks of the eight lanes that share l % 8 are then
// transposed in registers, one exchange per bit of the token index
// (v_permlane32_swap, v_permlane16_swap, DPP): lane l gets dim 8 (l % 8) + l / 8
// of all eight tokens, one 8-byte store. One wave per token with byte stores
// of stride 8 was bound by those stores: 131072 tokens 21.8 us, now 5.6; 2 M
// tokens 359 us, now 77 (5.3 TB/s; graph replays). A group per wave: waves that loop over two
// to sixteen groups took 78 to 98 us. (The same transpose for fp16 values, with
// its 16-byte stores 128 bytes apart, was slower than the gathers above: 95
// to 117 us for 2 M tokens against 88.)
struct ValueRange {
  int64_t n_seq, n_tok, t_cap, t0, g_first, n_groups;
};

// Loads 16 bytes of this lane's token of group g (zeros outside the range).
__device__ __forceinline__ uint4 load_group(const uint16_t* __restrict__ src, const ValueRange& r,
                                            int64_t s, int64_t g, int lane) {
  const int64_t t = g * 8 + (lane >> 3) - r.t0;
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (t >= 0 && t < r.n_tok)
    v = *reinterpret_cast<const uint4*>(src + (s * r.n_tok + t) * kDim + 8 * (lane & 7));
  return v;
}
__device__ __forceinline__ bool group_is_full(const ValueRange& r, int64_t g) {
  return g * 8 >= r.t0 && g * 8 + 8 <= r.t0 + r.n_tok;
}
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// INT8 values with a power-of-two scale per token (Sec. II-E), as
// store_value_token_i8_wave defines them.
// Group i of the range, i counting over sequences and their groups: one per wave
// (with a workgroup's waves on one sequence, three of four had no group where a
// sequence has one).
__global__ __launch_bounds__(kBlock) void store_values_i8_kernel(const uint16_t* __restrict__ src,
                                                                 ValueRange r,
                                                                 uint8_t* __restrict__ v_u8,
                                                                 int8_t* __restrict__ v_exp) {
  const int lane = lane_id();
  const uint32_t sel16 = (lane >> 4) & 1 ? 0x07060302u : 0x05040100u;
  const uint32_t sel8 = (lane >> 3) & 1 ? 0x03070105u : 0x06020400u;
  const uint32_t n = (uint32_t)(r.n_seq * r.n_groups), per_seq = (uint32_t)r.n_groups;
  const uint32_t stride = gridDim.x * (kBlock / 64);
  for (uint32_t i = blockIdx.x * (kBlock / 64) +
                    __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       i < n; i += stride) {
    const uint32_t seq = i / per_seq;
    const int64_t s = seq, g8 = r.g_first + (i - seq * per_seq);
    const uint4 v = load_group(src, r, s, g8, lane);
    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
    float x[8];
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __half2float(__ushort_as_half((unsigned short)(w4[i] & 0xFFFFu)));
      x[2 * i + 1] = __half2float(__ushort_as_half((unsigned short)(w4[i] >> 16)));
      amax = fmaxf(amax, fmaxf(fabsf(x[2 * i]), fabsf(x[2 * i + 1])));
    }
    amax = max_over_8_lanes(amax);
    const int g = value_exponent(amax);
    uint32_t b[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i / 4] |= (uint32_t)value_byte(x[i], g) << (8 * (i & 3));
    // token bits 2, 1, 0 against dim bits 2 (dword), 1 (half) and 0 (byte)
    swap32(b[0], b[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint32_t lo = b[i], hi = b[i];
      swap16(lo, hi);  // lo: the even row's value, hi: the odd row's
      b[i] = __builtin_amdgcn_perm(hi, lo, sel16);
      b[i] = __builtin_amdgcn_perm(lane_xor_u32<8>(b[i]), b[i], sel8);
    }
    const int64_t row = s * r.t_cap + g8 * 8;
    const int d = 8 * (lane & 7) + (lane >> 3);
    uint8_t* out = v_u8 + row * kDim + d * 8;
    if (group_is_full(r, g8)) {
      *reinterpret_cast<uint2*>(out) = make_uint2(b[0], b[1]);
      if ((lane & 7) == 0) v_exp[row + (lane >> 3)] = (int8_t)g;
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t t = g8 * 8 + k;
        if (t >= r.t0 && t < r.t0 + r.n_tok) out[k] = (uint8_t)(b[k / 4] >> (8 * (k & 3)));
      }
      const int64_t t = g8 * 8 + (lane >> 3);
      if ((lane & 7) == 0 && t >= r.t0 && t < r.t0 + r.n_tok) v_exp[row + (lane >> 3)] = (int8_t)g;
    }
  }
}

static ValueRange value_range(int64_t n_seq, int64_t n_tok, int64_t t_cap, int64_t t0) {
  return {n_seq, n_tok, t_cap, t0, t0 / 8, (t0 + n_tok - 1) / 8 - t0 / 8 + 1};
}
// The same, one wave per token: for calls of one token per sequence, whose groups
// would have one lane in eight at work (65536 sequences 11.4 us against 18.3, 4096 2.6
// against 3.3; two tokens 21.4 against 18.3), and for small calls (up to kTokenWaves
// tokens: 256 sequences of 2 to 8 tokens 2.2 against 2.45; 16 tokens 2.6 and 2.5).
constexpr int64_t kTokenWaves = 2048;
__global__ __launch_bounds__(kBlock) void store_tokens_i8_kernel(const uint16_t* __restrict__ src,
                                                                 ValueRange r,
                                                                 uint8_t* __restrict__ v_u8,
                                                                 int8_t* __restrict__ v_exp) {
  const uint32_t n = (uint32_t)(r.n_seq * r.n_tok), n_tok = (uint32_t)r.n_tok;
  const uint32_t stride = gridDim.x * (kBlock / 64);
  for (uint32_t i = blockIdx.x * (kBlock / 64) +
                    __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       i < n; i += stride) {
    const uint32_t s = i / n_tok;
    store_value_token_i8_wave(src + (int64_t)i * kDim, v_u8 + s * r.t_cap * kDim,
                              v_exp + s * r.t_cap, r.t0 + (i - s * n_tok));
  }
}

hipError_t launch_store_values_i8(const uint16_t* src, int64_t n_seq, int64_t n_tok,
                                  int64_t t_cap, int64_t t0, uint8_t* v_u8, int8_t* v_exp,
                                  hipStream_t stream) {
  if (n_seq == 0 || n_tok == 0) return hipSuccess;
  const ValueRange r = value_range(n_seq, n_tok, t_cap, t0);
  const bool tokens = n_tok == 1 || n_seq * n_tok <= kTokenWaves;
  const int64_t waves = tokens ? n_seq * n_tok : n_seq * r.n_groups;
  const dim3 grid(bounded_grid((waves + kBlock / 64 - 1) / (kBlock / 64)));
  if (tokens)
    hipLaunchKernelGGL(store_tokens_i8_kernel, grid, dim3(kBlock), 0, stream, src, r, v_u8, v_exp);
  else
    hipLaunchKernelGGL(store_values_i8_kernel, grid, dim3(kBlock), 0, stream, src, r, v_u8, v_exp);
  return hipGetLastError();
}

__global__ void fill_zero_kernel(uint32_t* __restrict__ p, size_t n_words, uint8_t* tail,
                                 size_t tail_bytes) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words || i < tail_bytes;
       i += (size_t)gridDim.x * blockDim.x) {
    if (i < n_words) p[i] = 0u;
    if (i < tail_bytes) tail[i] = 0;
  }
}

hipError_t launch_encode_pot(const uint16_t* k, int64_t n_rows, int64_t out_stride,
                             int scale_mode, int hadamard, float* key_scale,
                             uint8_t* codes_se, uint8_t* codes_m, const EncodeTables& tab,
                             hipStream_t stream) {
  if (n_rows == 0) return hipSuccess;
  const EncodeArgs a{reinterpret_cast<const __half*>(k), n_rows, out_stride, scale_mode, key_scale,
                     codes_se, codes_m};
  auto go = [&](auto k_tag) {
    constexpr int KK = decltype(k_tag)::value;
    if (hadamard && n_rows > kButterflyRows)
      hipLaunchKernelGGL((encode_pot_had_kernel<KK>), dim3(encode_grid((n_rows + 1) / 2, false)),
                         dim3(kBlock), 0, stream, a, tab);
    else if (hadamard)
      hipLaunchKernelGGL((encode_pot_kernel<KK, true>), dim3(encode_grid(n_rows, false)),
                         dim3(kBlock), 0, stream, a, tab);
    else
      hipLaunchKernelGGL((encode_pot_kernel<KK, false>), dim3(encode_grid(n_rows, KK == 0)),
                         dim3(kBlock), 0, stream, a, tab);
  };
  switch (tab.mant_bits) {
    case 0: go(std::integral_constant<int, 0>{}); break;
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_encode_int8(const uint16_t* k, int64_t n_rows, int64_t out_stride,
                              int hadamard, float* key_scale, int8_t* codes,
                              hipStream_t stream) {
  if (n_rows == 0) return hipSuccess;
  const __half* kh = reinterpret_cast<const __half*>(k);
  const dim3 grid(encode_grid(n_rows, !hadamard));
  if (hadamard)
    hipLaunchKernelGGL((encode_int8_kernel<true>), grid, dim3(kBlock), 0, stream, kh, n_rows,
                       out_stride, key_scale, codes);
  else
    hipLaunchKernelGGL((encode_int8_kernel<false>), grid, dim3(kBlock), 0, stream, kh, n_rows,
                       out_stride, key_scale, codes);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  if (bytes == 0) return hipSuccess;
  const size_t n_words = bytes / 4;
  const size_t tail = bytes - n_words * 4;
  const size_t n = n_words > tail ? n_words : tail;
  const size_t grid = (n + 255) / 256;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(bounded_grid((int64_t)grid)), dim3(256), 0, stream,
                     reinterpret_cast<uint32_t*>(ptr), n_words,
                     reinterpret_cast<uint8_t*>(ptr) + n_words * 4, tail);
  return hipGetLastError();
}

}  // namespace potattn
