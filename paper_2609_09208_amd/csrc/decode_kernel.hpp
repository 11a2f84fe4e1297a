// Split-K decode attention for gfx950 over a PoT / INT8 / fp16 key cache.
//
// Grid (n_splits, Hkv, B), 256 threads = 4 wave64, or in the CU-wide variant
// one workgroup of pool_waves(...) waves per CU. A workgroup owns one key
// range of one (batch, kv-head) sequence and all G query heads sharing that
// kv head (GQA), so every code and value byte is read from HBM once and used
// G times. Inside the workgroup each wave streams its own 64-key tiles
// (tile j of the range goes to wave j % 4; in the CU-wide variant the waves
// may claim tiles from a counter in LDS), with the next tile's keys requested
// before a tile is scored and its values once this tile's are used; waves only
// meet at the end to merge their partial sums.
//
// Per 64-key tile and wave:
//  1. Scores (Sec. II-B eq. sac). Shift-accumulate: exact integer sums on the
//     matrix cores, one ternary operand per bit position, scaled by powers of
//     two (score_planes.hpp). A lane ends up with the scores of one head and
//     8 consecutive keys, the operand order of step 4. (Packed 16-bit shifts
//     and v_dot2 sums on the VALU, one key per lane, took 741 / 1119 / 2261
//     VALU lane-operations per key at k = 0 / 1 / 4 and were bound by their
//     issue: B = 64, T = 32768, PoT-4 222 us per call, now 202; B = 8, T =
//     32768, PoT-M4 80 us, now 41; B = 16, T = 16384, PoT-4 with INT8 values
//     39 us, now 28.) The decoded-code engines (a multiply path) and the
//     comparators take the same operand layout with fp16 or INT8 matrix
//     instructions (score_decoded.hpp); the decoded codes' int32 sums equal
//     the shift-accumulate ones.
//  2. x = fl32(fl32(float(acc) * s) * c), c = fl32(fl32(Delta * log2 e) *
//     2^-(F+k+3)) in this order.
//  3. Integer running maximum M = max(M, ceil(max x)) per head (eq. logsm);
//     when it rises the accumulators are rescaled by the exact power of two
//     2^(M_old - M_new).
//  4. A.V on the matrix cores: P (16 rows = 8 heads x {fp16 high part, fp16
//     low part} of p = 2^(x - M + 12)) times V (fp16) with
//     v_mfma_f32_16x16x32_f16, fp32 accumulation; the sums l of p are one
//     more column of it, values of 1 (the same parts, rounded and dropped
//     alike: constant values come back constant), or, with INT8 values whose
//     weights are scaled, per lane in fp32. The value cache is stored token-interleaved
//     ([t/8][d][t%8]) so a lane's 16-byte load is exactly its B fragment.
// With one split the workgroup writes O directly; otherwise it writes its
// (M_s, l_s, o_s), and the last workgroup of a unit, or for many splits a small
// combine kernel, merges the splits with exact 2^(M_s - M) weights.
// (Kernel templates; the instantiations live in decode_pot*.hip,
// decode_dot.hip and decode_cmp.hip, one translation unit per score mode and
// value format.)
#pragma once

#include <hip/hip_fp16.h>

#include <climits>
#include <type_traits>

#include "pot_device.hpp"
#include "pot_launch.hpp"
#include "score_decoded.hpp"
#include "score_planes.hpp"

namespace potattn {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kWaves = kBlock / 64;  // waves per workgroup of the default variant
// Waves per workgroup of the CU-wide variant (0: none). A SIMD issues the
// oldest of its ready waves first, so of the four equal workgroups that
// share a CU the first dispatched finishes in about a third of the time of
// the last, and the CU runs its last stretch with one wave per SIMD. In the
// CU-wide variant one workgroup holds all of a CU's waves (as many per SIMD
// as the kernel's registers allow: pool_waves) and its waves take tiles from
// a counter in LDS, so they all finish within about one tile of each other.
// Every engine but the fp16 comparator has it.
template <int MODE, int K, int VF>
constexpr int kPoolWaves = pool_waves(MODE, K, VF);
constexpr int kWTile = 64;    // keys per wave tile
constexpr float kPScale = 12.0f;  // p is formed as 2^(x - M + 12) (fp16-normal range)
constexpr int kDppRowRor8 = 0x128;  // DPP row_ror:8: lane l reads lane l ^ 8 within its row of 16

// max(a, b) for scores (never NaN) as v_max_f32 without operand canonicalisation
__device__ __forceinline__ float max_f32(float a, float b) {
  return __builtin_amdgcn_fmed3f(a, b, __builtin_inff());
}

// Waits until this wave's vector stores are acknowledged: by the L2, where every
// later load of the workgroup finds them, or, for agent-scope stores, from beyond
// it. For other XCDs (merge_splits) only the latter counts.
__device__ __forceinline__ void wait_stores_in_l2() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- streaming loads -----------------------------------------------------------
// The cache is read once per call, so its loads carry the non-temporal hint.
// It pays for the value fragments of every engine and for the 32-byte PoT
// code rows; the comparators' 64- and 128-byte key rows are read by several
// 16-byte loads per lane that revisit the same lines, and stay plain.
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

// Raw buffer resources over the cache rows of one tile (gfx9 descriptor word
// 3 = 0x00020000: untyped records, byte-granular range). Each load's resource
// starts at the tile's first row and ends at the key range's last row, and
// the whole offset is in the vector operand: the hardware compares only that
// offset (not the scalar one) with the record count, so a lane whose key is
// at or past the end reads zeros and touches no memory. The tile loops need
// no clamped addresses, and every offset is 32-bit.
typedef __amdgpu_buffer_rsrc_t BufRsrc;
constexpr int kBufWord3 = 0x00020000;
constexpr int kAuxNt = 2;  // cache policy of the loads: non-temporal
__device__ __forceinline__ BufRsrc buf_rsrc(const void* base, int64_t n_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n_bytes,
                                           kBufWord3);
}

// The streams of one (batch, kv head) sequence that a workgroup reads, as
// byte pointers to the sequence's row 0 and the rows that exist: keys
// (codes, mantissa planes, scales) below t_end, value groups (fp16 or
// bytes, INT8 exponents) below v_end (the end of the range's last 8-key
// group).
struct Streams {
  const uint8_t* codes;
  const uint8_t* planes;
  const uint8_t* scales;
  const uint8_t* values;
  const uint8_t* exps;
  int t_end, v_end;
};

// Resource over rows t0 .. lim - 1 of row_bytes bytes each (t0 < lim, both
// wave-uniform, lim * row_bytes < 2^31).
__device__ __forceinline__ BufRsrc tile_rsrc(const uint8_t* base, int t0, int lim, int row_bytes) {
  return buf_rsrc(base + (uint32_t)(t0 * row_bytes), (int64_t)((lim - t0) * row_bytes));
}

// ---- per-tile register payloads -----------------------------------------------
// One half of one key per lane and set (score_planes.hpp).
template <int MODE, int K>
struct KeyRegs {                   // PoT codes
  uint4 c[2];                      // 16 code bytes of set 0 and set 1
  uint32_t pl[2][K > 0 ? K : 1];   // mantissa bits as loaded
};
template <int K>
struct KeyRegs<kScoreInt8, K> {
  uint4 k[2][2];
};
template <int K>
struct KeyRegs<kScoreFp16, K> {
  uint4 k[2][4];
};

template <bool V8>
struct ValRegs {
  uint4 f[2][4];  // [K-block of 32 keys][16-dim block], 8 fp16 values each
};
template <>
struct ValRegs<true> {
  uint2 f[2][4];  // the same fragments as 8 value bytes (v^ + 128)
  uint2 g;        // exponents g of the 8 keys whose weights this lane forms
};

// Loads are unconditional (reads past a buffer resource's end return zeros) so
// that the compiler can count outstanding loads statically and keep the
// prefetch of the next tile in flight while the current one is processed; keys
// past the range are masked when the tile is consumed.
// A lane's offset, opaque in each tile: the constant distances of a tile's loads
// then fold into the instructions' immediate offsets, where the compiler would
// otherwise keep every sum in a register of its own across the loop.
__device__ __forceinline__ int tile_offset(int off, int t0) {
  asm("" : "+v"(off) : "s"(t0));
  return off;
}
__device__ __forceinline__ uint4 load_b128(BufRsrc rs, int off, bool aux_nt) {
  const u32x4v v = aux_nt ? __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, kAuxNt)
                          : __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Keys of a 64-key tile (score_planes.hpp): in set s lane l loads half
// l / 16 % 2 of key 32 (l / 32) + 8 (l % 16 / 4) + 4 s + l % 4. The mantissa
// planes of the key's row are loaded as pairs of planes, the two
// halves of each: the even block's lane takes planes 0 (0 and 1 at k = 4), the
// odd block's the next ones, and plane_bits exchanges the halves; a last odd
// plane is one dword. Keys at or past the range's end read zeros.
template <int MODE, int K>
__device__ __forceinline__ void load_keys(const Streams& st, int t0, int lane,
                                          KeyRegs<MODE, K>& r) {
  const int i = lane & 15, blk = lane >> 4, half = blk & 1;
  const int key = 32 * (blk >> 1) + 8 * (i >> 2) + (i & 3);
  if constexpr (MODE == kScoreInt8 || MODE == kScoreFp16) {
    constexpr int kRow = MODE == kScoreInt8 ? kDim : 2 * kDim, kLoads = kRow / 32;
    const BufRsrc rk = tile_rsrc(st.codes, t0, st.t_end, kRow);
    const int off = tile_offset(key * kRow + 16 * kLoads * half, t0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < kLoads; ++c)
        r.k[s][c] = load_b128(rk, off + 4 * s * kRow + 16 * c, false);
    return;
  } else {
  const BufRsrc rc = tile_rsrc(st.codes, t0, st.t_end, kDim / 2);
  const int off = tile_offset(key * 32 + 16 * half, t0);
#pragma unroll
  for (int s = 0; s < 2; ++s) r.c[s] = load_b128(rc, off + 128 * s, true);
  if constexpr (K > 0) {
    const BufRsrc rp = tile_rsrc(st.planes, t0, st.t_end, 8 * K);
    const int pair = tile_offset(key * 8 * K + (K == 4 ? 16 : 8) * half, t0);
    const int last = tile_offset(key * 8 * K + 8 * (K - 1) + 4 * half, t0);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if constexpr (K == 4) {
        const uint4 v = load_b128(rp, pair + 32 * K * s, true);
        r.pl[s][0] = v.x;
        r.pl[s][1] = v.y;
        r.pl[s][2] = v.z;
        r.pl[s][3] = v.w;
      } else {
        if constexpr (K >= 2) {
          const u32x2v v = __builtin_amdgcn_raw_buffer_load_b64(rp, pair + 32 * K * s, 0, kAuxNt);
          r.pl[s][0] = v.x;
          r.pl[s][1] = v.y;
        }
        if constexpr (K & 1)
          r.pl[s][K - 1] = __builtin_amdgcn_raw_buffer_load_b32(rp, last + 32 * K * s, 0, kAuxNt);
      }
    }
  }
  }
}

// Scales of the 8 keys whose scores the lane gets (keys 32 part + 8 grp ..+7),
// up to the end of the last 8-key group (rows that exist).
__device__ __forceinline__ void load_scales(const Streams& st, int t0, int lane,
                                            uint4 (&s)[2]) {
  const BufRsrc rs = tile_rsrc(st.scales, t0, st.v_end, 4);
  const int off = tile_offset((32 * ((lane >> 3) & 1) + 8 * (lane >> 4)) * 4, t0);
  s[0] = load_b128(rs, off, true);
  s[1] = load_b128(rs, off + 16, true);
}

// The lane's half of every mantissa plane of set s, from the pairs as loaded:
// v_permlane16_swap exchanges the odd blocks of its first operand with the
// even blocks of its second.
template <int MODE, int K>
__device__ __forceinline__ void plane_bits(const KeyRegs<MODE, K>& r, int s, uint32_t* pl) {
  if constexpr (K == 4) {
    const auto a = __builtin_amdgcn_permlane16_swap(r.pl[s][0], r.pl[s][1], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(r.pl[s][2], r.pl[s][3], false, false);
    pl[0] = a[0];
    pl[2] = a[1];
    pl[1] = b[0];
    pl[3] = b[1];
  } else {
    if constexpr (K >= 2) {
      const auto a = __builtin_amdgcn_permlane16_swap(r.pl[s][0], r.pl[s][1], false, false);
      pl[0] = a[0];
      pl[1] = a[1];
    }
    if constexpr (K & 1) pl[K - 1] = r.pl[s][K - 1];
  }
}

// B fragments of one 64-key tile: lane l takes keys t0 + 32*kb + 8*(l/16) ..+7
// of dim 16*nb + l%16, one 16-byte (fp16) or 8-byte (INT8) load each from the
// token-interleaved cache, through the tile's value resource: groups past
// the range's last group read zeros (their weights are 0). With INT8 values
// the lane also loads the exponents of the 8 keys t0 + 32*part + 8*grp ..+7
// whose weights it forms in stage 2.
// Blocks kFirst .. kEnd - 1 of the two K-blocks; the exponents come with block 0.
template <bool V8, int kFirst = 0, int kEnd = 2>
__device__ __forceinline__ void load_values_buf(const Streams& st, int t0, int lane,
                                                ValRegs<V8>& v) {
  constexpr int kGroupBytes = V8 ? 8 * kDim : 16 * kDim;  // one 8-token group
  const BufRsrc rv = tile_rsrc(st.values, t0, st.v_end, kGroupBytes / 8);
  const int voff = tile_offset((lane >> 4) * kGroupBytes + (lane & 15) * (V8 ? 8 : 16), t0);
#pragma unroll
  for (int kb = kFirst; kb < kEnd; ++kb) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int off = voff + kb * 4 * kGroupBytes + nb * 16 * (V8 ? 8 : 16);
      if constexpr (V8) {
        const u32x2v w = __builtin_amdgcn_raw_buffer_load_b64(rv, off, 0, kAuxNt);
        v.f[kb][nb] = make_uint2(w.x, w.y);
      } else {
        const u32x4v w = __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, kAuxNt);
        v.f[kb][nb] = make_uint4(w.x, w.y, w.z, w.w);
      }
    }
  }
  if constexpr (V8 && kFirst == 0) {
    const int part = (lane & 15) >> 3, grp = lane >> 4;
    const BufRsrc re = tile_rsrc(st.exps, t0, st.v_end, 1);
    const u32x2v g =
        __builtin_amdgcn_raw_buffer_load_b64(re, tile_offset(32 * part + 8 * grp, t0), 0, 0);
    v.g = make_uint2(g.x, g.y);
  }
}

// fp16 B fragment of 8 INT8 values held as v^ + 128: bytes u become the fp16
// numbers 1024 + u = 1152 + v^ (bit pattern 0x6400 | u, exact), two per
// v_perm_b32, and a packed fp16 addition takes the 1152 off again (exact).
// (Taking it off the fp32 sums instead costs 32 operations less per tile and
// most of their precision: 1.9e-5 against 64 bits where this has 4e-7.)
__device__ __forceinline__ half8 int8_value_fragment(uint2 w) {
  constexpr uint32_t kHi = 0x64646464u;
  half8 v = __builtin_bit_cast(
      half8, make_uint4(__builtin_amdgcn_perm(kHi, w.x, 0x04010400u),
                        __builtin_amdgcn_perm(kHi, w.x, 0x04030402u),
                        __builtin_amdgcn_perm(kHi, w.y, 0x04010400u),
                        __builtin_amdgcn_perm(kHi, w.y, 0x04030402u)));
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] -= (_Float16)1152.0f;
  return v;
}

// Zero the value fragments of tokens at or past t_end (tail tile only), so
// that whatever the cache holds there cannot reach the sums (p is 0 there).
__device__ __forceinline__ void mask_values(int t0, int t_end, int lane, ValRegs<false>& v) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int g8 = t0 + 32 * kb + 8 * (lane >> 4);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      uint32_t w4[4] = {v.f[kb][nb].x, v.f[kb][nb].y, v.f[kb][nb].z, v.f[kb][nb].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t lo = (g8 + 2 * i < t_end) ? 0x0000FFFFu : 0u;
        const uint32_t hi = (g8 + 2 * i + 1 < t_end) ? 0xFFFF0000u : 0u;
        w4[i] &= lo | hi;
      }
      v.f[kb][nb] = make_uint4(w4[0], w4[1], w4[2], w4[3]);
    }
  }
}

// ---- shared memory of the decode kernel -------------------------------------
template <int NW>
struct alignas(16) MergeSmem {
  alignas(16) float wo[NW][8][kDim];  // per-wave P.V
  float wl[NW][8];   // sums of the weights per head
  int wm[NW][8];
  int gm[NW];        // INT8 values: per-wave minimum exponent
  int next;          // CU-wide variant: the next unclaimed tile of the range
  int last;          // this workgroup merges its unit's splits
};
template <int MODE, int NW>
struct DecodeSmem : MergeSmem<NW> {
  alignas(16) _Float16 qh[8][kDim];  // decoded weights: q^ 2^8; fp16 keys: q
  float qc[8];                       // score factor per head
};
template <int NW>
struct DecodeSmem<kScorePot, NW> : MergeSmem<NW> {
  alignas(16) _Float16 qh[8][kDim];  // q^ = 16 hi + lo per head, in operand order
  alignas(16) _Float16 ql[8][kDim];
  float qc[8];
};
template <int NW>
struct DecodeSmem<kScoreInt8, NW> : MergeSmem<NW> {
  alignas(16) int8_t qb[8][kDim];  // q^
  float qc[8];
};

// The new token of one (batch, kv head) sequence appended at row T - 1
// (Sec. II-F, a cache that holds only codes): wave 0 encodes the key with the
// row absmax scale, wave 1 stores the values (fp16, or INT8 with their
// exponent). Only the workgroup whose key range holds row T - 1 calls it.
// Returns the exponent of INT8 values in wave 1, INT_MAX elsewhere.
template <int K>
__device__ __forceinline__ int append_token(const DecodeArgs& a, int64_t seq, int wave) {
  const int64_t row = seq * a.t_cap + (a.T - 1);
  if (wave == 0)
    encode_key_row_wave<K>(reinterpret_cast<const __half*>(a.app_k) + seq * kDim, a.hadamard, 0,
                        a.app_key_scale + row, a.app_codes_se + row * (kDim / 2),
                        a.app_codes_m + row * 8 * K, a.app_tab);
  else if (wave == 1 && a.app_v8 != nullptr)
    return store_value_token_i8_wave(a.app_v + seq * kDim, a.app_v8 + seq * a.t_cap * kDim,
                                     a.app_v_exp + seq * a.t_cap, a.T - 1);
  else if (wave == 1)
    store_value_token_wave(a.app_v + seq * kDim, a.app_v_cache + seq * a.t_cap * kDim, a.T - 1);
  return INT_MAX;
}

// Minimum over the wave.
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, (int)lane_xor_u32<1>((uint32_t)v));
  v = min(v, (int)lane_xor_u32<2>((uint32_t)v));
  v = min(v, (int)lane_xor_u32<4>((uint32_t)v));
  v = min(v, (int)lane_xor_u32<8>((uint32_t)v));
  const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = min((int)r16[0], (int)r16[1]);
  const auto r32 = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return min((int)r32[0], (int)r32[1]);
}

// The query elements of the heads this wave prepares (heads p, p + NW of
// p = prep_head(wave)), one per lane; loaded first thing so that their latency
// overlaps the rest of the prologue. Waves 0 and 1, which append the new
// token, come last.
template <int NW>
__device__ __forceinline__ int prep_head(int wave) {
  return wave >= 2 ? wave - 2 : wave + NW - 2;
}
template <int G, int NW>
struct QueryIn {
  static constexpr int kHeadsPerWave = (G + NW - 1) / NW;
  float v[kHeadsPerWave];
};
template <int G, int NW>
__device__ __forceinline__ QueryIn<G, NW> load_queries(const DecodeArgs& a, int kvh, int b) {
  const int lane = lane_id();
  const int head = prep_head<NW>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  QueryIn<G, NW> qin;
#pragma unroll
  for (int i = 0; i < QueryIn<G, NW>::kHeadsPerWave; ++i) {
    const int h = head + NW * i;
    qin.v[i] = h < G ? a.q[((int64_t)b * a.Hq + a.q_head(kvh * G + h)) * kDim + lane] : 0.0f;
  }
  return qin;
}

// Rotates (optionally) and quantises the G query vectors of one (batch, kv
// head) and writes the operands and per-head score factors into LDS. Called by
// all NW waves of the workgroup, each for the heads whose elements qin holds. taps: also write the q^ and Delta debug taps.
template <int MODE, int G, int K, int NW>
__device__ __forceinline__ void prepare_queries(const DecodeArgs& a, int kvh, int b,
                                                DecodeSmem<MODE, NW>& sm, bool taps,
                                                const QueryIn<G, NW>& qin) {
  const int lane = lane_id();
  const int head = prep_head<NW>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  constexpr int kHeadsPerWave = QueryIn<G, NW>::kHeadsPerWave;
#pragma unroll
  for (int i = 0; i < kHeadsPerWave; ++i) {
    const int h = head + NW * i;
    if (h >= G) break;
    const int64_t bq = (int64_t)b * a.Hq + a.q_head(kvh * G + h);
    float qv = qin.v[i];
    if constexpr (MODE == kScoreFp16) {
      sm.qh[h][lane] = (_Float16)qv;
      if (lane == 0) sm.qc[h] = __fmul_rn(log2e_f32(), 0.125f);
    } else {
      if (a.hadamard) qv = (float)(wave_fwht64((double)qv) * 0.125);
      float step;
      const int qi = wave_quantize_int8(qv, &step);
      if constexpr (MODE == kScorePot)
        store_query_element<K>(qi, lane, sm.qh[h], sm.ql[h]);
      else if constexpr (MODE == kScoreDs4a)
        sm.qh[h][(lane & 32) + pair_order<K>(lane & 31)] = (_Float16)(qi * 256);
      else
        sm.qb[h][lane] = (int8_t)qi;
      if (lane == 0) {
        const int bits = MODE == kScoreInt8 ? 3 : a.frac_bits + K + 3;
        sm.qc[h] =
            __fmul_rn(__fmul_rn(step, log2e_f32()), __builtin_amdgcn_ldexpf(1.0f, -bits));
      }
      if (taps) {
        if (a.dbg_qhat) a.dbg_qhat[bq * kDim + lane] = (int8_t)qi;
        if (a.dbg_delta && lane == 0) a.dbg_delta[bq] = step;
      }
    }
  }
}

// ---- merge of the key splits by the last workgroup of a unit ------------------
// A unit is one (batch, kv head) sequence. Its workgroups write their partials
// (M_s, l_s, o_s) and count themselves on the unit's ticket word in the
// workspace; the one that counts last merges, which saves the merge kernel's
// launch. Everything that passes between workgroups goes by agent-scope
// accesses (relaxed atomics: written through and read from beyond the XCD's
// own L2), and a wave waits until its stores have arrived before the barrier in
// front of the count. No fence: an agent-scope release or acquire fence writes
// back or invalidates the whole L2 of the XCD, per workgroup (that took B = 64
// from 258 to 541 us). This rests on the hardware and not on the memory model,
// which orders relaxed accesses to different words by fences only: an agent-scope
// store that s_waitcnt vmcnt(0) has seen acknowledged is at the point that
// agent-scope accesses of every XCD go to. Nothing ever waits for another
// workgroup.
//
// The workspace may hold anything before a call. The ticket word is the
// call's tag (52 bits, never 0) and the count (12 bits); every workgroup first
// puts {tag, 0} there unless the tag is there already (one compare-and-swap
// against what it read: it can only fail because another workgroup of the call
// put the tag there), and the last one clears the word, so that a replay of a
// captured call, which has the same tag, starts over.
constexpr int kTicketCountBits = 12;
constexpr int kTicketStride = 32;  // 64-bit words between tickets: a 256-byte line pair each

template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int wave_max_i32(int v) { return ~wave_min(~v); }
// Sum over the wave.
__device__ __forceinline__ float wave_sum(float v) {
  v += __uint_as_float(lane_xor_u32<1>(__float_as_uint(v)));
  v += __uint_as_float(lane_xor_u32<2>(__float_as_uint(v)));
  v += __uint_as_float(lane_xor_u32<4>(__float_as_uint(v)));
  v += __uint_as_float(lane_xor_u32<8>(__float_as_uint(v)));
  const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
  v = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
  const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
  return __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
}

// One head's merge by one wave: lane s holds split s's M_s and l_s, and every
// lane its dimension of all splits' sums, N >= Sn of them requested together
// (loads in a loop or behind branches wait for each other: 0.6 us a turn).
// Splits past the last read the last one and get factor 0.
template <int N, bool DEBUG>
__device__ __forceinline__ void merge_head(const DecodeArgs& a, int64_t bq, int lane) {
  const int Sn = a.n_splits, s_l = min(lane, Sn - 1);
  const int m_l = load_agent(a.part_m + bq * Sn + s_l);
  const float l_l = load_agent(a.part_l + bq * Sn + s_l);
  const float* po = a.part_o + bq * Sn * kDim + lane;
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = load_agent(po + min(i, Sn - 1) * kDim);
  const int M = wave_max_i32(m_l);
  const float f_l = lane < Sn && m_l != INT_MIN ? __builtin_amdgcn_ldexpf(1.0f, m_l - M) : 0.0f;
  const float l = wave_sum(f_l * l_l);
  float o = 0.0f;
#pragma unroll
  for (int i = 0; i < N; ++i)
    o = fmaf(__uint_as_float(
                 (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(f_l), i)),
             v[i], o);
  a.out[bq * kDim + lane] = o / l;
  if constexpr (DEBUG) {
    if (lane == 0 && a.dbg_m_final) a.dbg_m_final[bq] = M;
  }
}

template <int G, bool DEBUG, int NW, typename Smem>
__device__ __forceinline__ void merge_splits(const DecodeArgs& a, int64_t seq, int kvh, int b,
                                             Smem& sm) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Sn = a.n_splits;
  unsigned long long* ticket = a.tickets + seq * kTicketStride;
  wait_stores_in_l2();  // this wave's partials (and ticket) have arrived
  __syncthreads();
  if (tid == 0) {
    const unsigned long long old =
        __hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sm.last = (int)(old & ((1u << kTicketCountBits) - 1)) == Sn - 1;
  }
  __syncthreads();
  if (!sm.last) return;
  if (tid == 0) store_agent(ticket, 0ull);
  for (int h = wave; h < G; h += NW) {
    const int64_t bq = (int64_t)b * a.Hq + a.q_head(kvh * G + h);
    if (Sn <= 4) merge_head<4, DEBUG>(a, bq, lane);
    else if (Sn <= 8) merge_head<8, DEBUG>(a, bq, lane);
    else if (Sn <= 16) merge_head<16, DEBUG>(a, bq, lane);
    else merge_head<kMaxMergedSplits, DEBUG>(a, bq, lane);
  }
}

// VF: value format, 0 fp16 values, 1 INT8 values, 2 INT8 values with the
// power-of-two weights of eq. logsm.
// Value blocks (of two, 16 registers each; INT8 values 8) loaded before the
// scores; the others are loaded after them, since held meanwhile they would not
// fit the kernel's registers without spills. CU-wide kernels: 128 registers at
// four waves per SIMD (shift-accumulate at k = 3, 4: 168 at three); a wave has
// about 4 us per tile there and can wait for a load. The four-wave kernels keep
// the same budget, so that as many of their waves share a SIMD: without it they
// took 130 to 176 registers, three waves (two at k = 4). B * Hkv = 1024 in graph
// replays, T = 64 and 1024, us: PoT-4 10.2 -> 6.9 and 35.0 -> 32.1, PoT-M1 10.8 ->
// 7.6, PoT-M4 44.3 -> 40.4 at T = 1024, decoded M1 10.9 -> 7.1 and 36.0 -> 31.8, M1
// with INT8 values 11.5 -> 7.6 and 33.5 -> 30.9, INT8 keys 9.1 -> 6.3 and 36.3 ->
// 34.0; one tile per wave waits for the late values (PoT-M1, 260 units, T = 64 5.8
// -> 6.1).
template <int MODE, int K, int VF, bool POOL>
constexpr int kEarlyValueBlocks =
    POOL ? (MODE == kScorePot ? (K == 2 ? 0 : 1) : MODE == kScoreDs4a ? (K >= 1 ? 0 : 1) : 2)
    : K == 0            ? 2
    : VF != 0           ? (K == 2 ? 0 : 2)
    : MODE == kScorePot ? (K == 3 ? 2 : K == 2 ? 0 : 1)
                        : 0;

// Waves per SIMD that the registers have to allow.
template <int MODE, int K, int VF>
constexpr int kSimdWaves = kPoolWaves<MODE, K, VF> > 0 ? kPoolWaves<MODE, K, VF> / 4 : 1;

// NW: waves per workgroup, kWaves or kPoolWaves<MODE, K, VF> (the CU-wide
// variant, whose waves take their tiles from the counter sm.next).
template <int MODE, int G, int K, bool DEBUG, int VF, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(
    kSimdWaves<MODE, K, VF>))) void decode_kernel(const DecodeArgs a) {
  constexpr bool kPool = NW > kWaves;
  constexpr int kBlk = 64 * NW;
  __shared__ DecodeSmem<MODE, NW> sm;
  constexpr bool V8 = VF != 0;
  constexpr bool kPow2 = VF == 2;

  const int tid = threadIdx.x, lane = tid & 63;
  // the wave index is uniform in a wave; saying so keeps the tile loop's
  // control flow scalar (no per-lane loop exit masks)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int64_t seq = (int64_t)b * a.Hkv + kvh;
  const int64_t row0 = seq * a.t_cap;
  const int8_t* eseq = V8 ? a.v_exp + row0 : nullptr;
  // ---- per-wave streaming over 64-key tiles ------------------------------------
  const int t_begin = split * a.split_len;
  const int t_end = min(a.T, t_begin + a.split_len);
  const int n_tiles = (t_end - t_begin + kWTile - 1) / kWTile;
  const int row = lane & 15, grp = lane >> 4, hrow = row & 7, part = row >> 3;
  const bool hvalid = hrow < G;

  // the ticket of this unit (merge_splits): read now, set below
  const bool tickets = kPool && a.ticket != 0 && wave == NW - 1;  // uniform per wave
  unsigned long long* ticket = a.tickets + seq * kTicketStride;
  unsigned long long seen = 0;
  if (tickets) seen = load_agent(ticket);
  const QueryIn<G, NW> qin = load_queries<G, NW>(a, kvh, b);
  // The sequence's new token (fused append) belongs to the workgroup whose
  // range holds row T - 1.
  const bool appends = (MODE == kScorePot || MODE == kScoreDs4a) && a.app_k != nullptr &&
                       split == a.n_splits - 1;  // uniform per workgroup
  int gref = 0;
  float lsum = 0.0f;  // INT8 values: this lane's sum of the unscaled weights

  // acc[4], fp16 values: the sums of the weights, as one more column of P.V
  constexpr int kAcc = V8 ? 4 : 5;
  float4v acc[kAcc];
#pragma unroll
  for (int nb = 0; nb < kAcc; ++nb) acc[nb] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
  int m_run = INT_MIN;
  // -1 kept opaque so that p - hi stays one fma_mix reading hi as fp16
  float neg_one = -1.0f;
  asm("" : "+v"(neg_one));
  // the working bit of the score planes, kept in a VGPR (a VALU op that reads
  // an SGPR issues at the slower rate)
  uint32_t m22 = 0x22222222u;
  if constexpr (MODE == kScorePot) asm("" : "+v"(m22));

  KeyRegs<MODE, K> kr[2];
  const int g_last = (t_end - 1) & ~7;  // first token of the range's last 8-token group
  Streams st{};
  st.t_end = t_end;
  st.v_end = g_last + 8;
  if constexpr (MODE == kScorePot || MODE == kScoreDs4a) {
    st.codes = a.codes_se + row0 * (kDim / 2);
    st.scales = reinterpret_cast<const uint8_t*>(a.key_scale + row0);
    if constexpr (K > 0) st.planes = a.codes_m + row0 * 8 * K;
  } else if constexpr (MODE == kScoreInt8) {
    st.codes = reinterpret_cast<const uint8_t*>(a.codes_i8 + row0 * kDim);
    st.scales = reinterpret_cast<const uint8_t*>(a.key_scale + row0);
  } else {
    st.codes = reinterpret_cast<const uint8_t*>(a.k_f16 + row0 * kDim);
  }
  if constexpr (V8) {
    st.values = a.v8 + row0 * kDim;
    st.exps = reinterpret_cast<const uint8_t*>(a.v_exp + row0);
  } else {
    st.values = reinterpret_cast<const uint8_t*>(a.v + row0 * kDim);
  }
  auto load_keys_tile = [&](int jt, KeyRegs<MODE, K>& kk) {
    load_keys<MODE, K>(st, t_begin + kWTile * jt, lane, kk);
  };
  // Tiles: wave w starts with tiles w and w + NW; after that it takes every
  // NW-th tile or, with claim_tiles, claims the next unclaimed tile (from 2 NW
  // on) one tile ahead of its use.
  int j = wave;
  int jn = wave + NW;  // CU-wide variant: this wave's next tile
  int jc = 0;          // CU-wide variant: the tile after that
  const int j_last = n_tiles - 1;
  // Besides its keys a tile needs its scales and values: requested once the
  // previous tile's values are used, so that they arrive during the scores. (A
  // second set of value registers, one tile further ahead, made the engines
  // with short scores slower: PoT-4 decoded to weights 211 us against 200 at
  // B = 64, T = 32768, 34.5 against 33.3 at B = 16, T = 16384.)
  constexpr int kEarlyV = kEarlyValueBlocks<MODE, K, VF, kPool>;
  ValRegs<V8> vr;
  uint4 ksc[2];
  auto load_tile_scales = [&](int jt) {
    if constexpr (MODE != kScoreFp16) load_scales(st, t_begin + kWTile * jt, lane, ksc);
  };
  auto load_tile_values = [&](int jt) {
    load_values_buf<V8, 0, kEarlyV>(st, t_begin + kWTile * jt, lane, vr);
  };
  // A wave's first keys and scales are requested at once, unless the tile holds
  // the row that is being appended: then after the barrier below. The first
  // values follow after the barrier in any case: they are not needed before the
  // scores, and on a full chip the requests of all waves' values would hold up
  // the queries that the barrier waits for.
  const bool late_first = appends && j == j_last;
  if (j < n_tiles && !late_first) {
    load_keys_tile(j, kr[0]);
    load_tile_scales(j);
  }
  if constexpr (kPool) {
    if (tid == 0) sm.next = 2 * NW;
  }

  // With INT8 values, the reference exponent g_ref = min g over this
  // workgroup's keys (Sec. II-E eq. av): weights are formed as p 2^(g_ref -
  // g_j) <= p, so they stay in fp16 range for any g, and the sums are scaled
  // by 2^-g_ref at the end (fp32). The appended token's g comes from its store.
  int gmin = INT_MAX;
  const int g_end = V8 && appends ? t_end - 1 : t_end;
  uint2 g8 = make_uint2(0u, 0u);  // the first 8 exponents of this thread
  if constexpr (V8) {
    if (t_begin + 8 * tid < g_end) g8 = *reinterpret_cast<const uint2*>(eseq + t_begin + 8 * tid);
  }
  // The append and the query preparation while the first tiles load; one
  // barrier publishes all of it.
  if constexpr (MODE == kScorePot || MODE == kScoreDs4a) {
    if (appends) gmin = append_token<K>(a, seq, wave);
  }
  prepare_queries<MODE, G, K, NW>(a, kvh, b, sm, DEBUG && split == 0, qin);
  if constexpr (V8) {
    for (int t = t_begin + 8 * tid; t < g_end; t += 8 * kBlk) {
      const uint2 w = t < t_begin + 8 * kBlk ? g8 : *reinterpret_cast<const uint2*>(eseq + t);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int gi = (int)(int8_t)(((i < 4) ? w.x : w.y) >> (8 * (i & 3)));
        gmin = (t + i < g_end) ? min(gmin, gi) : gmin;
      }
    }
    gmin = wave_min(gmin);
    if (lane == 0) sm.gm[wave] = gmin;
  }
  if (tickets && lane == 0 && (seen >> kTicketCountBits) != a.ticket)
    __hip_atomic_compare_exchange_strong(ticket, &seen, a.ticket << kTicketCountBits,
                                         __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
  if (appends && wave < 2) wait_stores_in_l2();
  __syncthreads();
  if (j < n_tiles) {
    if (late_first) {
      load_keys_tile(j, kr[0]);
      load_tile_scales(j);
    }
    load_tile_values(j);
  }
  if constexpr (V8) {
    gref = sm.gm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) gref = min(gref, sm.gm[w]);
  }
  const float c_lane = hvalid ? sm.qc[hrow] : 0.0f;  // the score factor of this lane's head
  std::conditional_t<MODE == kScorePot, PlaneQuery,
                     std::conditional_t<MODE == kScoreInt8, ByteQuery, HalfQuery>>
      qop;
  if constexpr (MODE == kScorePot) qop = load_plane_query<G>(sm.qh, sm.ql, a.frac_bits);
  else if constexpr (MODE == kScoreInt8) qop = load_byte_query<G>(sm.qb);
  else qop = load_half_query<G>(sm.qh, lane);
  // decoded weights with a mantissa: the 16 registers of the operand are read
  // again from LDS in each tile, so that the values can have them meanwhile
  constexpr bool kReloadQ = MODE == kScoreDs4a && K > 0;
  // decoded weights: their sums to the int32 score at head-room F
  const float to_int = MODE == kScoreDs4a ? __builtin_amdgcn_ldexpf(1.0f, a.frac_bits + K) : 1.0f;

  // Stage 1 of a tile: request this wave's next keys, score (the loads land
  // meanwhile) and find the tile's integer maximum per head (in m_new).
  float xv[8];
  int m_new = m_run;
  bool first = true;
  auto stage1 = [&](const KeyRegs<MODE, K>& ks, KeyRegs<MODE, K>& knext, int jt) {
    const int t0 = t_begin + kWTile * jt;
    // the next tile's keys (past the range: the last tile again, unused)
    const int jl = min(kPool ? jn : jt + NW, j_last);
    load_keys_tile(jl, knext);
    if constexpr (kPool) {
      // claim the tile after jn now; it is needed one tile from now
      jc = jn + NW;
      if (a.claim_tiles) {  // uniform
        int c = 0;
        if (lane == 0) c = __hip_atomic_fetch_add(&sm.next, 1, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        jc = __builtin_amdgcn_readfirstlane(c);
      }
    }
    // ---- 1. scores: keys t0 + 32 part + 8 grp ..+7 of head hrow ----
    {
      if constexpr (kReloadQ) qop = load_half_query<G>(sm.qh, tile_offset(lane, t0));
      f32x4 d[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if constexpr (MODE == kScorePot || MODE == kScoreDs4a) {
          const uint32_t w[4] = {ks.c[i].x, ks.c[i].y, ks.c[i].z, ks.c[i].w};
          uint32_t pl[K > 0 ? K : 1];
          if constexpr (K > 0) plane_bits<MODE, K>(ks, i, pl);
          if constexpr (MODE == kScorePot) d[i] = score_set<K>(w, pl, m22, qop);
          else d[i] = score_set_decoded<K>(w, pl, qop, to_int);
          if constexpr (kReloadQ) asm volatile("" : "+v"(d[i]));
        } else if constexpr (MODE == kScoreInt8) {
          d[i] = score_set_int8(ks.k[i], qop);
        } else {
          d[i] = score_set_fp16(ks.k[i], qop);
        }
      }
      // keeps the matrix instructions above here (and so their operands' live
      // ranges short): the compiler would sink them to their first use
      asm volatile("" : "+v"(d[0]), "+v"(d[1]));
      if constexpr (kEarlyV < 2) load_values_buf<V8, kEarlyV, 2>(st, t0, lane, vr);
      // ---- 2. scores to the log2 domain ----
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t sc[4] = {ksc[i].x, ksc[i].y, ksc[i].z, ksc[i].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float x = d[i][r];
          if constexpr (MODE != kScoreFp16) x = __fmul_rn(x, __uint_as_float(sc[r]));
          x = __fmul_rn(x, c_lane);
          xv[4 * i + r] = hvalid ? x : -INFINITY;
          if constexpr (DEBUG) {
            const int key = t0 + 32 * part + 8 * grp + 4 * i + r;
            if (a.dbg_scores && hvalid && key < t_end)
              a.dbg_scores[((int64_t)b * a.Hq + a.q_head(kvh * G + hrow)) * a.T + key] =
                  (int32_t)d[i][r];
          }
        }
      }
    }
    const bool tail = t0 + kWTile > t_end;  // wave-uniform
    if (tail) {
      const int k0 = t0 + 32 * part + 8 * grp;
#pragma unroll
      for (int i = 0; i < 8; ++i) xv[i] = (k0 + i < t_end) ? xv[i] : -INFINITY;
      // weights past the range are 0; fp16 value bytes there could be inf or
      // NaN and are cleared, INT8 value bytes are always finite numbers
      if constexpr (!V8) mask_values(t0, t_end, lane, vr);
    }

    // ---- 3. integer running maximum per head ----
    float mx = xv[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = max_f32(mx, xv[i]);
    mx = max_f32(mx, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
                                                   __builtin_bit_cast(int, mx), kDppRowRor8, 0xF,
                                                   0xF, true)));  // the other part
    // ceil is monotonic, so M = max over lanes of ceil(x): the reduction over
    // the four rows of 16 lanes runs on int32 (swap odd with even rows, then
    // the two halves; v_permlane*_swap, no LDS)
    // a lane whose keys are all past the range holds -inf (no int32 ceiling)
    int mt = (hvalid && mx > -INFINITY) ? (int)ceilf(mx) : INT_MIN;
    {
      const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)mt, (uint32_t)mt, false, false);
      mt = max((int)r16[0], (int)r16[1]);
      const auto r32 = __builtin_amdgcn_permlane32_swap((uint32_t)mt, (uint32_t)mt, false, false);
      mt = max((int)r32[0], (int)r32[1]);
    }
    m_new = max(m_run, mt);
  };

  // acc <- diag(2^(M_old - M_new)) acc on the matrix cores: D = sum_j A_j B_j
  // with B_j = acc[.][j] (16x16x4 f32 layout: lane l holds row 4 (l / 16) + j
  // of column l % 16) and A_j[i][k] = f_i for i = 4k + j, else 0. Each
  // element gets one exact power-of-two product. It runs outside the hot
  // loop below, so the accumulators stay in the matrix-core registers there.
  auto rescale = [&]() {
    if (first) {  // nothing is summed yet
      m_run = m_new;
      return;
    }
    const float f = (m_run == INT_MIN) ? 0.0f : __builtin_amdgcn_ldexpf(1.0f, m_run - m_new);
    const int arow = lane & 15, acol = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < kAcc; ++nb) {
      float4v d = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(arow == 4 * acol + jj ? f : 0.0f, acc[nb][jj], d,
                                                 0, 0, 0);
      acc[nb] = d;
    }
    if constexpr (V8) lsum *= f;
    m_run = m_new;
  };

  // Stage 2 of a tile: weights from the scores and P.V on the matrix cores.
  auto stage2 = [&]() {
    // ---- 4. weights (fp16 high / low parts) and P.V on the matrix cores ----
    // Each lane splits its 8 weights into hi = rtz(p) and lo = rn(p - hi)
    // and hands lo to its partner lane (row ^ 8). Block kb = 0 then takes
    // rows 0-7 = hi, 8-15 = lo of the part-0 weights; block kb = 1 takes rows
    // 0-7 = lo, 8-15 = hi of the part-1 weights. Rows h and h + 8 are summed
    // at the end, so both blocks see hi + lo of every weight.
    const float bias = hvalid ? kPScale - (float)m_run : 0.0f;
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float p0, p1;
      if constexpr (kPow2) {
        // A~ = 2^-k with k = M - ceil(x - 1/2) (M - x rounded half up):
        // p = 2^(ceil(x - 1/2) - M + 12), exact; keys masked to -inf get 0.
        // ceil(x - 1/2) is ceil(x), less one when ceil(x) - x >= 1/2: that
        // difference is exact in fp32 where it decides (x - 1/2 itself is
        // not: -0.5 + 2^-25 would round to -1)
        auto pw = [&](float x) -> float {
          const float c = ceilf(x);
          const float r = (c - x >= 0.5f) ? c - 1.0f : c;
          return x > -INFINITY
                     ? __builtin_amdgcn_ldexpf(1.0f, (int)r - m_run + (int)kPScale)
                     : 0.0f;
        };
        p0 = pw(xv[2 * i]);
        p1 = pw(xv[2 * i + 1]);
      } else {
        p0 = __builtin_amdgcn_exp2f(xv[2 * i] + bias);
        p1 = __builtin_amdgcn_exp2f(xv[2 * i + 1] + bias);
      }
      if constexpr (V8) {
        // the softmax sum takes p; A.V takes p 2^(g_ref - g) (exact scaling)
        lsum += p0;
        lsum += p1;
        const uint32_t gw = (i < 2) ? vr.g.x : vr.g.y;
        p0 = __builtin_amdgcn_ldexpf(p0, gref - (int)(int8_t)(gw >> (16 * (i & 1))));
        p1 = __builtin_amdgcn_ldexpf(p1, gref - (int)(int8_t)(gw >> (16 * (i & 1) + 8)));
      }
      const half2v hi = __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(p0, p1));
      hw[i] = __builtin_bit_cast(uint32_t, hi);
      const half2v lo = {(_Float16)__builtin_fmaf(neg_one, (float)hi.x, p0),
                         (_Float16)__builtin_fmaf(neg_one, (float)hi.y, p1)};
      lw[i] = __builtin_bit_cast(uint32_t, lo);
    }
    uint32_t a0w[4], a1w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t rl =
          (uint32_t)__builtin_amdgcn_mov_dpp((int)lw[i], kDppRowRor8, 0xF, 0xF, true);
      a0w[i] = part ? rl : hw[i];
      a1w[i] = part ? hw[i] : rl;
    }
    const half8 af0 = __builtin_bit_cast(half8, make_uint4(a0w[0], a0w[1], a0w[2], a0w[3]));
    const half8 af1 = __builtin_bit_cast(half8, make_uint4(a1w[0], a1w[1], a1w[2], a1w[3]));
    auto bfrag = [&](int kb, int nb) -> half8 {
      if constexpr (V8) return int8_value_fragment(vr.f[kb][nb]);
      else return __builtin_bit_cast(half8, vr.f[kb][nb]);
    };
    auto weight_sums = [&]() {
      if constexpr (!V8) {
        half8 ones;
#pragma unroll
        for (int i = 0; i < 8; ++i) ones[i] = (_Float16)1.0f;
        acc[4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af0, ones, acc[4], 0, 0, 0);
        acc[4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af1, ones, acc[4], 0, 0, 0);
      }
    };
    // they do not wait for the values: before them, where the registers allow (PoT-4, 4
    // to 64 units, T <= 1024: 1.0% of a call over sums per lane, 1.6% after the values)
    constexpr bool kSumsLast = MODE == kScorePot && K == 2;
    if constexpr (!kSumsLast) weight_sums();
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af0, bfrag(0, nb), acc[nb], 0, 0, 0);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af1, bfrag(1, nb), acc[nb], 0, 0, 0);
    if constexpr (kSumsLast) weight_sums();
  };

  // The hot loop runs the tiles that do not raise any head's maximum; a tile
  // that does leaves it, is rescaled and finished in the outer loop (a few
  // times per wave). The prefetched registers move forward after each tile so
  // that every tile uses the same registers.
  auto advance = [&]() {
    kr[0] = kr[1];
    // also after a tile that raised nothing: scores at -2^31, whose ceiling is INT_MIN
    // itself, have had their weights summed, and a later maximum takes them out
    first = false;
    if constexpr (kPool) {
      j = jn;
      jn = jc;
    } else {
      j += NW;
    }
    if (j < n_tiles) {
      load_tile_scales(j);
      load_tile_values(j);
    }
  };
#pragma nounroll
  while (j < n_tiles) {
#pragma nounroll
    for (;;) {
      stage1(kr[0], kr[1], j);
      if (__any(m_new != m_run)) break;
      stage2();
      advance();
      if (j >= n_tiles) break;
    }
    if (j >= n_tiles) break;
    rescale();
    stage2();
    advance();
  }

  // ---- merge the waves ------------------------------------------------------
  // Only the sums of waves that had a tile are merged, in whole groups of four (a
  // wave of such a group without tiles has zero sums and factor 0). Rows h and h + 8 of
  // the products (weights' high and low parts) sit in the two halves of the
  // wave and are added on the way to LDS.
  const int n_act = kPool ? min(NW, (n_tiles + 3) & ~3) : NW;
  if (wave < n_act) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t v = __float_as_uint(acc[nb][r]);
        const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        const float sum = __uint_as_float(h[0]) + __uint_as_float(h[1]);
        if (lane < 32) sm.wo[wave][4 * grp + r][16 * nb + row] = sum;
      }
  }
  if (lane < 8) sm.wm[wave][lane] = m_run;
  if constexpr (V8) {
    // sum of the weights over the 8 lanes that formed a head's
    lsum += dpp_move<kDppRowRor8>(lsum);
    const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(lsum), __float_as_uint(lsum),
                                                      false, false);
    lsum = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(lsum), __float_as_uint(lsum),
                                                      false, false);
    lsum = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
    if (lane < 8) sm.wl[wave][lane] = lsum;
  } else {
    // rows 4 grp + r, the same in every column: column r hands over row r
    const float sum = row == 0 ? acc[4][0] : row == 1 ? acc[4][1] : row == 2 ? acc[4][2] : acc[4][3];
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum),
                                                    false, false);
    if (lane < 32 && row < 4)
      sm.wl[wave][4 * grp + row] = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  }
  __syncthreads();

  const int Sn = a.n_splits;
  for (int idx = tid; idx < G * kDim; idx += kBlk) {
    const int h = __builtin_amdgcn_readfirstlane(idx / kDim), d = idx % kDim;
    const int64_t bq = (int64_t)b * a.Hq + a.q_head(kvh * G + h);
    // lane w holds wave w's maximum, factor and sum of the head
    static_assert(NW <= 64, "a lane per wave");
    const int m_w = lane < NW ? sm.wm[lane < NW ? lane : 0][h] : INT_MIN;
    const float l_w = lane < NW ? sm.wl[lane < NW ? lane : 0][h] : 0.0f;
    const int M = wave_max_i32(m_w);
    const float f_w = m_w == INT_MIN ? 0.0f : __builtin_amdgcn_ldexpf(1.0f, m_w - M);
    const float l = wave_sum(f_w * l_w);
    float o = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; w += 4) {
      if (w >= n_act) break;  // uniform
#pragma unroll
      for (int i = w; i < w + 4; ++i)
        o = fmaf(__uint_as_float(
                     (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(f_w), i)),
                 sm.wo[i][h][d], o);
    }
    if constexpr (V8) o = __builtin_amdgcn_ldexpf(o, -gref);
    if (Sn == 1) {
      a.out[bq * kDim + d] = o / l;
      if constexpr (DEBUG) {
        if (d == 0 && a.dbg_m_final) a.dbg_m_final[bq] = M;
        if (d == 0 && a.dbg_m_split) a.dbg_m_split[bq] = M;
      }
    } else {
      const int64_t ps = bq * Sn + split;
      if (kPool && a.ticket != 0) {  // uniform
        store_agent(&a.part_o[ps * kDim + d], o);
        if (d == 0) {
          store_agent(&a.part_l[ps], l);
          store_agent(&a.part_m[ps], M);
        }
      } else {
        a.part_o[ps * kDim + d] = o;
        if (d == 0) {
          a.part_l[ps] = l;
          a.part_m[ps] = M;
        }
      }
      if (d == 0) {
        if constexpr (DEBUG) {
          if (a.dbg_m_split) a.dbg_m_split[ps] = M;
        }
      }
    }
  }
  if constexpr (kPool)
    if (Sn > 1 && a.ticket != 0) merge_splits<G, DEBUG, NW>(a, seq, kvh, b, sm);
}

// Merges the key splits of one (batch, query head): M = max_s M_s and
// O = sum_s 2^(M_s - M) o_s / sum_s 2^(M_s - M) l_s with exact power-of-two
// weights (Sec. II-E). Grid B * Hq, 4 waves; wave w takes splits w, w + 4,
// ... with one lane per output dimension, and the four waves meet in LDS.
// Up to 64 splits, every load of a wave is issued before the first wait (one
// memory latency for the whole merge); more splits go through a loop.
constexpr int kCombineWaves = 4;
constexpr int kCombineBatch = 16;  // splits per wave in the single-batch path
template <bool DEBUG>
__global__ __launch_bounds__(64 * kCombineWaves) void combine_kernel(const DecodeArgs a) {
  __shared__ float so[kCombineWaves][kDim];
  __shared__ float sl[kCombineWaves];
  __shared__ int smax[kCombineWaves];
  const int64_t bq = blockIdx.x;
  const int tid = threadIdx.x, d = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Sn = a.n_splits;
  const int32_t* __restrict__ pm = a.part_m + bq * Sn;
  const float* __restrict__ pl = a.part_l + bq * Sn;
  const float* __restrict__ po = a.part_o + bq * Sn * kDim;
  float L = 0.0f, O = 0.0f;
  int M;
  if (Sn <= kCombineWaves * kCombineBatch) {  // uniform
    // lane i (< 16) holds M_s and l_s of split s = w + 4 i; every lane holds
    // o_s[d] of all of them. Splits past the last read the last one
    // (unconditional loads, so all are in flight together) and are dropped.
    const int li = min(d, kCombineBatch - 1);
    const int s_l = w + kCombineWaves * li;
    const bool valid = d < kCombineBatch && s_l < Sn;
    const int m_l = pm[min(s_l, Sn - 1)];
    const float l_l = pl[min(s_l, Sn - 1)];
    float ov[kCombineBatch];
#pragma unroll
    for (int i = 0; i < kCombineBatch; ++i)
      ov[i] = po[min(w + kCombineWaves * i, Sn - 1) * kDim + d];
    int mw = valid ? m_l : INT_MIN;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mw = max(mw, __shfl_xor(mw, o, 64));
    if (d == 0) smax[w] = mw;
    __syncthreads();
    M = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
    const float f_l = valid ? __builtin_amdgcn_ldexpf(1.0f, m_l - M) : 0.0f;
    float fl = f_l * l_l;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) fl += __shfl_xor(fl, o, 64);
    L = fl;
#pragma unroll
    for (int i = 0; i < kCombineBatch; ++i) {
      const float f = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f_l), i));
      O = fmaf(f, ov[i], O);
    }
  } else {
    M = INT_MIN;
    for (int s = tid; s < Sn; s += 64 * kCombineWaves) M = max(M, pm[s]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) M = max(M, __shfl_xor(M, o, 64));
    if (d == 0) smax[w] = M;
    __syncthreads();
    M = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
#pragma unroll 8
    for (int s = w; s < Sn; s += kCombineWaves) {
      const float f = __builtin_amdgcn_ldexpf(1.0f, pm[s] - M);
      L = fmaf(f, pl[s], L);
      O = fmaf(f, po[s * kDim + d], O);
    }
  }
  so[w][d] = O;
  if (d == 0) sl[w] = L;
  __syncthreads();
  if (w == 0) {
    O = so[0][d];
    L = sl[0];
#pragma unroll
    for (int i = 1; i < kCombineWaves; ++i) {
      O += so[i][d];
      L += sl[i];
    }
    a.out[bq * kDim + d] = O / L;
    if constexpr (DEBUG) {
      if (d == 0 && a.dbg_m_final) a.dbg_m_final[bq] = M;
    }
  }
}

template <int MODE, int G, int K, bool DEBUG, int VF>
static hipError_t launch_t(const DecodeArgs& a, hipStream_t stream, hipEvent_t ev_begin,
                           hipEvent_t ev_end) {
  if constexpr (VF != 0 && MODE != kScorePot && MODE != kScoreDs4a) {
    return hipErrorInvalidValue;
  } else {
  constexpr int PW = kPoolWaves<MODE, K, VF>;
  hipError_t e = hipSuccess;
  if (ev_begin != nullptr && (e = hipEventRecord(ev_begin, stream)) != hipSuccess) return e;
  const dim3 grid((uint32_t)a.n_splits, (uint32_t)a.Hkv, (uint32_t)a.B);
  if constexpr (PW > 0) {
    if (a.wg_waves == PW)
      hipLaunchKernelGGL((decode_kernel<MODE, G, K, DEBUG, VF, PW>), grid, dim3(64 * PW), 0,
                         stream, a);
    else
      hipLaunchKernelGGL((decode_kernel<MODE, G, K, DEBUG, VF, kWaves>), grid, dim3(kBlock), 0,
                         stream, a);
  } else {
    hipLaunchKernelGGL((decode_kernel<MODE, G, K, DEBUG, VF, kWaves>), grid, dim3(kBlock), 0,
                       stream, a);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev_end != nullptr && (e = hipEventRecord(ev_end, stream)) != hipSuccess) return e;
  if (a.n_splits == 1 || a.ticket != 0) return hipSuccess;
  hipLaunchKernelGGL((combine_kernel<DEBUG>), dim3((uint32_t)(a.B * a.Hq)),
                     dim3(64 * kCombineWaves), 0, stream, a);
  return hipGetLastError();
  }
}

template <int MODE, int G, bool DEBUG, int VF>
static hipError_t launch_k(int mant_bits, const DecodeArgs& a, hipStream_t stream, hipEvent_t e0,
                           hipEvent_t e1) {
  if constexpr (!(MODE == kScorePot || (MODE == kScoreDs4a && VF == 0))) {
    return launch_t<MODE, G, 0, DEBUG, VF>(a, stream, e0, e1);
  } else {
    switch (mant_bits) {
      case 0: return launch_t<MODE, G, 0, DEBUG, VF>(a, stream, e0, e1);
      case 1: return launch_t<MODE, G, 1, DEBUG, VF>(a, stream, e0, e1);
      case 2: return launch_t<MODE, G, 2, DEBUG, VF>(a, stream, e0, e1);
      case 3: return launch_t<MODE, G, 3, DEBUG, VF>(a, stream, e0, e1);
      case 4: return launch_t<MODE, G, 4, DEBUG, VF>(a, stream, e0, e1);
      default: return hipErrorInvalidValue;
    }
  }
}

template <int MODE, bool DEBUG, int VF>
static hipError_t launch_g(int G, int mant_bits, const DecodeArgs& a, hipStream_t stream,
                           hipEvent_t e0, hipEvent_t e1) {
  switch (G) {
    case 1: return launch_k<MODE, 1, DEBUG, VF>(mant_bits, a, stream, e0, e1);
    case 2: return launch_k<MODE, 2, DEBUG, VF>(mant_bits, a, stream, e0, e1);
    case 4: return launch_k<MODE, 4, DEBUG, VF>(mant_bits, a, stream, e0, e1);
    case 8: return launch_k<MODE, 8, DEBUG, VF>(mant_bits, a, stream, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

// One score mode and value format: every head-group size and mantissa width
// the mode supports (the instantiations live in one translation unit per
// mode / format, declared in pot_launch.hpp).
template <int MODE, int VF>
hipError_t launch_mode_vf(int G, int mant_bits, bool debug, const DecodeArgs& a,
                          hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  if constexpr (MODE == kScoreFp16)
    return launch_g<MODE, false, VF>(G, mant_bits, a, stream, e0, e1);
  else
    return debug ? launch_g<MODE, true, VF>(G, mant_bits, a, stream, e0, e1)
                 : launch_g<MODE, false, VF>(G, mant_bits, a, stream, e0, e1);
}

}  // namespace potattn
