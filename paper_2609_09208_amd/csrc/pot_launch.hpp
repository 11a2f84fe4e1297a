// Host-side launch interface between the C ABI layer (api.cpp) and the
// kernel translation units. Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pot_attn.h"

namespace potattn {

constexpr int kMaxHqArg = 128;  // query heads addressable through kernel args (a byte each)

// Encoder tables passed by value as kernel arguments (no device globals).
struct EncodeTables {
  // Cut points between consecutive mantissa grid values inside one binade,
  // scaled to [1, 2): cut[i] = RD_fp32(sqrt((n+i)(n+i+1)) / n), n = 2^k,
  // i = 0..n-1 (the last one separates the binade top from the next binade).
  float cut[16];
  // RD_fp32(2^-(E + 1/2)): ratios at or below it become the exact zero.
  float zero_cut;
  int32_t mant_bits;
};

// EncodeTables for mantissa width k (0..4), from exact integer square roots.
const EncodeTables& encode_tables(int mant_bits);

hipError_t launch_encode_pot(const uint16_t* k, int64_t n_rows, int64_t out_stride,
                             int scale_mode, int hadamard, float* key_scale,
                             uint8_t* codes_se, uint8_t* codes_m,
                             const EncodeTables& tab, hipStream_t stream);

hipError_t launch_encode_int8(const uint16_t* k, int64_t n_rows, int64_t out_stride,
                              int hadamard, float* key_scale, int8_t* codes,
                              hipStream_t stream);

hipError_t launch_store_values(const uint16_t* src, int64_t n_seq, int64_t n_tok, int64_t t_cap,
                               int64_t t0, uint16_t* dst, hipStream_t stream);

// INT8 values with a power-of-two per-token scale: v_u8 holds v^ + 128
// token-interleaved like the fp16 cache, v_exp one g per cache row.
hipError_t launch_store_values_i8(const uint16_t* src, int64_t n_seq, int64_t n_tok,
                                  int64_t t_cap, int64_t t0, uint8_t* v_u8, int8_t* v_exp,
                                  hipStream_t stream);

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream);

// Records a printf-style detail for pot_last_error() on the calling thread and
// returns st (api.cpp).
pot_status report_error(pot_status st, const char* fmt, ...);

// kScoreDs4a: PoT codes decoded to fp16 weights that are multiplied (a
// multiply path, kept beside the shift path for measurement)
enum ScoreMode : int { kScorePot = 0, kScoreInt8 = 1, kScoreFp16 = 2, kScoreDs4a = 3 };

// Splits that the last workgroup of a unit merges (CU-wide workgroups); more go
// to the combine kernel, whose workgroups share the reading: one CU gets about
// 32 KB per us of partials that other XCDs wrote. PoT-4 graph replays, us, in
// the kernel and with the combine kernel: 4 units, T = 1024 (4 splits) 6.8 and
// 7.6, T = 4096 (16) 7.3 and 7.7, T = 8192 (32) 7.8 and 7.9, T = 16384 (64) 9.0 and
// 8.4, T = 32768 (64) 10.1 and 9.7; 16 units, T = 4096 (16) 7.8 and 8.4. A launch of the
// combine kernel also costs the host 3 us. Four-wave workgroups, with two heads to
// a wave, took 9.1 and 8.2 at 4 splits of fp16 keys and keep the combine kernel.
constexpr int kMaxMergedSplits = 32;

// Everything one decode launch needs. Passed by value as the kernel argument.
struct DecodeArgs {
  const float* q;
  const uint8_t* codes_se;   // PoT
  const uint8_t* codes_m;    // PoT-Mk planes
  const int8_t* codes_i8;    // INT8 keys
  const uint16_t* k_f16;     // fp16 keys
  const float* key_scale;
  const uint16_t* v;         // fp16 value cache, or
  const uint8_t* v8;         // INT8 value cache (v^ + 128) with
  const int8_t* v_exp;       // one exponent g per row: value v^ 2^-g
  float* out;
  // workspace
  int32_t* part_m;           // [B*Hq*S]
  float* part_l;             // [B*Hq*S]
  float* part_o;             // [B*Hq*S*64]
  unsigned long long* tickets;  // one word per (batch, kv head), merge_splits
  unsigned long long ticket;    // this call's tag; 0: a combine kernel merges the splits
  // debug taps (nullable)
  int8_t* dbg_qhat;
  float* dbg_delta;
  int32_t* dbg_scores;
  int32_t* dbg_m_final;
  int32_t* dbg_m_split;
  // fused append (PoT only; app_k NULL: none): the new token of every
  // (batch, kv head) sequence is encoded into cache row T - 1 and its values
  // stored there by the decode workgroup whose key range holds that row, in its
  // prologue. Waves whose first tile does not hold the row request that tile's
  // keys before; the wave whose first tile holds it, and every later load, comes
  // after the prologue's barrier
  const uint16_t* app_k;     // fp16 [B*Hkv][64]
  const uint16_t* app_v;     // fp16 [B*Hkv][64]
  uint8_t* app_codes_se;     // the cache arrays, written at row T - 1 only
  uint8_t* app_codes_m;
  float* app_key_scale;
  uint16_t* app_v_cache;     // fp16 value cache, or
  uint8_t* app_v8;           // INT8 value cache and
  int8_t* app_v_exp;         // its exponents
  EncodeTables app_tab;
  int64_t t_cap;
  int32_t B, Hq, Hkv, T;
  int32_t n_splits, split_len;
  int32_t frac_bits, hadamard;
  int32_t claim_tiles;         // CU-wide workgroups: tiles from a counter, else in fixed order
  int32_t wg_waves;            // waves per decode workgroup: 4, or pool_waves(...)
  uint32_t q_of_kv[kMaxHqArg / 4];  // [Hkv][G] query heads served by each kv head, a byte each

  // Query head g of a group in [Hkv][G] order (kvh * G + g).
  __host__ __device__ int q_head(int i) const { return (q_of_kv[i >> 2] >> (8 * (i & 3))) & 0xFF; }
};

// Waves per workgroup of a decode kernel's CU-wide variant, 0 if it has
// none: four SIMDs times the waves per SIMD that the kernel's registers
// allow (512 per lane and SIMD): the shift-accumulate kernels 4 at k <= 2
// and 3 at k = 3, 4 (fp16 or INT8 values); the decoded-code engines 4, or 3
// for PoT-4 bytes over fp16 values or with power-of-two weights; the INT8
// comparator 3. The fp16 comparator has none: with 12 waves it was no faster on
// long ranges (graph replays, us: 256 units T = 32768 322 against 323 on four
// waves, 64 units 86.2 and 85.8, 4 units 13.2 and 12.3).
constexpr int pool_waves(int mode, int mant_bits, int vf) {
  return mode == kScorePot    ? (mant_bits <= 2 ? 16 : 12)
         : mode == kScoreDs4a ? ((mant_bits > 0 || vf == 1) ? 16 : 12)
         : mode == kScoreInt8 ? 12
                              : 0;
}

// Longest key range of one decode call: the decode kernel reads each
// sequence's cache rows through buffer resources with 32-bit byte ranges
// (fp16 values: 128 bytes per key, rounded up to whole 8-key groups).
constexpr int kMaxKeys = (1 << 24) - 8;

// 32-bit words per decode workgroup at the head of the workspace (256 bytes at
// the least). The tickets of the split merge take a little of that room. The
// sizes that callers compute and allocate by are part of the interface, so the
// rest of it stays.
constexpr int query_words(int G) { return (33 * G + 63) / 64 * 64; }

// vf: value format. 0: fp16 value cache (a.v); 1: INT8 value cache (a.v8,
// a.v_exp); 2: INT8 values with the power-of-two weights of eq. logsm.
// Formats 1 and 2 exist for the score modes kScorePot and kScoreDs4a only.
// ev_begin / ev_end (may be null) are recorded on the stream right before and
// right after the decode kernel.
hipError_t launch_decode(int mode, int G, int mant_bits, bool debug, int vf,
                         const DecodeArgs& a, hipStream_t stream, hipEvent_t ev_begin = nullptr,
                         hipEvent_t ev_end = nullptr);

// The launch of one score mode and value format; each
// mode's kernels are instantiated in a translation unit of their own.
template <int MODE, int VF>
hipError_t launch_mode_vf(int G, int mant_bits, bool debug, const DecodeArgs& a,
                          hipStream_t stream, hipEvent_t e0, hipEvent_t e1);

}  // namespace potattn
