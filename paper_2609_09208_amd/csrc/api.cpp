// C ABI of libpotattn (declared in include/pot_attn.h).
//
// Every check runs on the host before any HIP call; a rejected call touches
// neither the device nor the stream. Launches are asynchronous on the
// caller's stream and allocate nothing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "pot_attn.h"
#include "pot_device.hpp"
#include "pot_launch.hpp"

using namespace potattn;

namespace {

thread_local std::string g_last_error;

pot_status fail(pot_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

}  // namespace

pot_status potattn::report_error(pot_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

namespace {

pot_status ok() {
  g_last_error.clear();
  return POT_OK;
}

pot_status hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return ok();
  return fail(POT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

constexpr int kE = 6;
constexpr int kMaxF = 12;

pot_status check_format(const pot_format* f) {
  if (!f) return fail(POT_ERR_INVALID_ARG, "fmt is NULL");
  if (f->head_dim != 64) return fail(POT_ERR_UNSUPPORTED, "head_dim %d (only 64)", f->head_dim);
  if (f->exp_bits != 3) return fail(POT_ERR_UNSUPPORTED, "exp_bits %d (only 3)", f->exp_bits);
  if (f->mant_bits < 0 || f->mant_bits > 4)
    return fail(POT_ERR_UNSUPPORTED, "mant_bits %d (0..4)", f->mant_bits);
  if (f->frac_bits < kE)
    return fail(POT_ERR_INVALID_ARG,
                "frac_bits %d < E = %d: a shift F - e would be a right shift", f->frac_bits, kE);
  if (f->frac_bits > kMaxF)
    return fail(POT_ERR_UNSUPPORTED, "frac_bits %d > %d (int32 head-room)", f->frac_bits, kMaxF);
  if (f->hadamard != 0 && f->hadamard != 1)
    return fail(POT_ERR_INVALID_ARG, "hadamard %d (0 or 1)", f->hadamard);
  return POT_OK;
}

struct Plan {
  int n_splits, split_len;
};

// S key splits of T keys, in whole 256-key tiles.
Plan plan_from_count(int T, int S) {
  const int tiles = (T + kTile - 1) / kTile;
  S = std::max(1, std::min(S, tiles));
  const int tiles_per_split = (tiles + S - 1) / S;
  Plan p;
  p.split_len = tiles_per_split * kTile;
  p.n_splits = (T + p.split_len - 1) / p.split_len;
  return p;
}

int split_count_for_slots(long units, long slots) {
  return units >= slots ? 1 : (int)(slots / units);
}

// Upper bound used to size workspaces without a device query: 256 CUs x 8
// resident workgroups (the decode kernels reach at most 4 per CU: 4 waves per SIMD).
constexpr long kMaxSlots = 256L * 8;

Plan plan_bound(int B, int Hkv, int T) {
  return plan_from_count(T, split_count_for_slots((long)B * Hkv, kMaxSlots));
}

std::atomic<int> g_cus[64];
int device_cus() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int cus = g_cus[dev].load(std::memory_order_relaxed);
  if (cus <= 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    g_cus[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

// How a decode call is split: (batch, kv head) units times key splits, on
// four-wave or CU-wide (pw waves, 0: the engine has none) workgroups. Figures:
// graph replays, us, eight heads to a unit, PoT-4 over fp16 values unless said.
//  - Up to one unit per CU: CU-wide workgroups and as many splits as give every
//    CU at most one. More splits cost a second round of prologues, fewer leave
//    CUs idle; four-wave workgroups take longer over the prologue (two heads'
//    queries per wave) and the merge. 64 units T = 4096 11.7 with 4 splits, 14.7
//    with 8 on four waves, 15.3 with 4; 24 units T = 16384 16.1 with 10, 18.4 with
//    32 on four waves; the fp16 comparator (four waves) at 96 units 69.4, 78.0
//    with 4.
//  - That rule rounds down: from half the CUs on it leaves one workgroup per unit
//    and the other CUs without work. For long ranges (from 12288 keys; at 8192 one
//    workgroup is as fast, 132 units 36.7 and 36.5) the fp16 comparator and the
//    engines that are bound by their issue take three splits of four-wave
//    workgroups up to two thirds of the CUs (T = 16384, 160 units: PoT-M1 80.4 ->
//    76.5, PoT-M4 108 -> 93, fp16 119.9 -> 108.4), PoT-4 and INT8 keys over fp16 values,
//    whose stream decides sooner, up to three fifths (132 units 68.6 -> 63.4, 152
//    72.2 -> 70.3, 168 75.2 and 77.8). With INT8 values, where a unit takes a CU the
//    longest, three to four workgroups per CU up to three quarters (132 units 68.0
//    -> 55.1, 160 69.8 -> 61.2, 176 70.7 -> 66.9, 192 72.8 -> 67.7; T = 8192 38.0 ->
//    32.5 and 39.6 -> 40.7).
//  - Where every wave of one workgroup has at most one 64-key tile, one split
//    and no merge: up to 768 keys (T = 512, 4 units 5.8 against 6.8 with two
//    splits, 64 units 6.1 against 7.2; T = 768, 4 units 6.6 against 6.9 with three;
//    on 12 waves PoT-M4 7.4 and 7.6 at 512, but 8.9 and 7.9 at 768), and up to 16
//    tiles on 16 waves if a quarter of the CUs has a unit (T = 1024: 16 units 7.6
//    against 7.2 with four splits, 64 units 7.8 and 7.8, 128 units 8.0 against 9.0
//    with two).
//  - More units than CUs: one split of four-wave workgroups, several of which
//    share a CU, for up to 8191 keys (512 units: T = 256 8.1 against 10.3 CU-wide,
//    T = 4096 57.4 against 59.9; 320 units 41.8 against 47.1); CU-wide above, whose
//    waves claim tiles (512 units, T = 16384 205 against 208), in three splits where
//    those make at most four rounds instead of two whole ones (T = 16384, 320 units
//    145 against 159 with one; 352 units, a fifth round, 168 against 162).
constexpr int kShortKeys = 768, kLongKeys = 8192, kSpreadKeys = 12288;
struct Launch {
  Plan plan;
  bool pool;
};

// Splits of four-wave workgroups, over two and up to four to a CU, that leave the
// smallest share of the CUs' places empty.
int spread_splits(long units, long cus) {
  int best = 1;
  long best_used = 0, best_places = 1;
  for (long S = 2 * cus / units + 1; S * units <= 4 * cus; ++S) {
    const long used = S * units, places = (used + cus - 1) / cus * cus;
    if (used * best_places > best_used * places) {
      best = (int)S;
      best_used = used;
      best_places = places;
    }
  }
  return best;
}

// What of an engine the plan depends on.
struct PlanEngine {
  int pw;            // waves of its CU-wide workgroups, 0: none
  bool int8_values;
  bool light;        // PoT-4 or INT8 keys over fp16 values: the stream decides even on one CU
};

Launch plan_launch(long units, int T, const PlanEngine& e, int cus, int bound) {
  const int pw = e.pw;
  const bool one_tile = pw > 0 && (T <= kShortKeys || (T <= pw * 64 && 4 * units >= cus));
  int S = 1;
  bool pool = pw > 0;
  if (units <= cus) {
    if (!one_tile) S = (int)(cus / units);
    if (S == 1 && T >= kSpreadKeys) {
      if (e.int8_values ? 4 * units <= 3L * cus
                        : (e.light ? 5 * units <= 3L * cus : 3 * units <= 2L * cus)) {
        S = e.int8_values ? spread_splits(units, cus) : 3;
        pool = false;
      }
    }
  } else {
    pool = pool && T >= kLongKeys;
    if (pool && 3 * units <= 4L * cus) S = 3;
  }
  return {plan_from_count(T, std::min(S, bound)), pool};
}

// CU-wide workgroups claim their tiles from a counter when the grid fills the
// chip and every wave has over four (long streams drift apart, graph replays of 256
// units at T = 32768: PoT-4 203 us against 209 in fixed order, PoT-M4 247 against
// 259, PoT-4 over INT8 values 145 against 163; four tiles per wave, 64 units at T =
// 16384: 33.2 against 32.9). In fixed order the sums are the same from call to call.
bool claims_tiles(long units, const Plan& p, int pw, int cus) {
  return units * p.n_splits >= cus && p.split_len > 4 * pw * 64;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct WsLayout {
  size_t part_m, part_l, part_o, total;
};

// Workspace: query_words per decode workgroup (the tickets are in them), then the
// split partials.
WsLayout ws_layout(long B, long Hq, long Hkv, long S) {
  WsLayout w;
  w.part_m = align_up((size_t)(B * Hkv * S) * query_words((int)(Hq / Hkv)) * 4, 256);
  w.part_l = w.part_m + align_up((size_t)(B * Hq * S) * 4, 256);
  w.part_o = w.part_l + align_up((size_t)(B * Hq * S) * 4, 256);
  w.total = w.part_o + align_up((size_t)(B * Hq * S) * 64 * 4, 256);
  return w;
}

// A tag that a workspace does not hold by chance: 52 bits, never 0, another one
// for each call.
unsigned long long next_ticket() {
  static std::atomic<unsigned long long> n{
      (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count()};
  unsigned long long z = n.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;  // splitmix64
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = (z ^ (z >> 31)) >> 12;
  return z != 0 ? z : 1;
}

bool shape_ok(int B, int Hq, int Hkv, int T) {
  return B >= 1 && Hq >= 1 && Hkv >= 1 && T >= 1 && Hq % Hkv == 0;
}

// Validates the GQA head map and fills DecodeArgs::q_of_kv ([Hkv][G]).
pot_status check_heads(const int32_t* map, int Hq, int Hkv, DecodeArgs* a, int* G_out) {
  if (!map) return fail(POT_ERR_INVALID_ARG, "kv_head_of_q is NULL");
  if (Hq > kMaxHqArg) return fail(POT_ERR_UNSUPPORTED, "Hq %d > %d", Hq, kMaxHqArg);
  if (Hq % Hkv) return fail(POT_ERR_UNSUPPORTED, "Hq %d not a multiple of Hkv %d", Hq, Hkv);
  const int G = Hq / Hkv;
  if (G != 1 && G != 2 && G != 4 && G != 8)
    return fail(POT_ERR_UNSUPPORTED, "group size %d (1, 2, 4 or 8)", G);
  int fill[kMaxHqArg] = {};
  for (int i = 0; i < Hq; ++i) {
    const int h = map[i];
    if (h < 0 || h >= Hkv)
      return fail(POT_ERR_INVALID_ARG, "kv_head_of_q[%d] = %d outside [0, %d)", i, h, Hkv);
    if (fill[h] >= G)
      return fail(POT_ERR_UNSUPPORTED, "kv head %d serves more than %d query heads", h, G);
    const int at = h * G + fill[h]++;
    a->q_of_kv[at >> 2] |= (uint32_t)i << (8 * (at & 3));
  }
  *G_out = G;
  return POT_OK;
}

// Shared tail of the three decode entry points.
pot_status decode_common(int mode, int mant_bits, DecodeArgs& a, const int32_t* map, int B,
                         int Hq, int Hkv, int T, int64_t t_cap, void* workspace,
                         size_t ws_bytes, pot_debug* dbg, void* stream, int vf = 0) {
  const bool v8 = vf != 0;
  if (!shape_ok(B, Hq, Hkv, T))
    return fail(POT_ERR_INVALID_ARG, "bad shape B=%d Hq=%d Hkv=%d T=%d", B, Hq, Hkv, T);
  if (t_cap < T) return fail(POT_ERR_INVALID_ARG, "T %d > t_cap %lld", T, (long long)t_cap);
  if (T > kMaxKeys)
    return fail(POT_ERR_UNSUPPORTED, "T %d > %d keys per sequence (32-bit buffer ranges)", T,
                kMaxKeys);
  if (t_cap % 8)
    return fail(POT_ERR_INVALID_ARG, "t_cap %lld is not a multiple of 8 (value-cache groups)",
                (long long)t_cap);
  if (v8) {
    if (!a.q || !a.v8 || !a.v_exp || !a.out)
      return fail(POT_ERR_INVALID_ARG, "q, v_u8, v_exp or out is NULL");
    if (!aligned(a.q, 16) || !aligned(a.v8, 16) || !aligned(a.v_exp, 16) || !aligned(a.out, 16))
      return fail(POT_ERR_INVALID_ARG, "q, v_u8, v_exp and out must be 16-byte aligned");
  } else {
    if (!a.q || !a.v || !a.out) return fail(POT_ERR_INVALID_ARG, "q, v or out is NULL");
    if (!aligned(a.q, 16) || !aligned(a.v, 16) || !aligned(a.out, 16))
      return fail(POT_ERR_INVALID_ARG, "q, v and out must be 16-byte aligned");
  }
  if (!workspace) return fail(POT_ERR_INVALID_ARG, "workspace is NULL");
  if (!aligned(workspace, 256))
    return fail(POT_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
  int G = 0;
  pot_status st = check_heads(map, Hq, Hkv, &a, &G);
  if (st != POT_OK) return st;
  const int force = dbg ? dbg->force_splits : 0;
  if (force < 0) return fail(POT_ERR_INVALID_ARG, "force_splits %d < 0", force);
  const int mbits = (mode == kScorePot || mode == kScoreDs4a) ? mant_bits : 0;
  const int pw = pool_waves(mode, mbits, vf);
  const int want = dbg ? dbg->force_wg_waves : 0;
  if (want != 0 && want != kBlock / 64 && (pw == 0 || want != pw))
    return fail(POT_ERR_INVALID_ARG, "force_wg_waves %d is neither 0, %d nor %d", want,
                kBlock / 64, pw);
  const long units = (long)B * Hkv;
  const int cus = device_cus();
  Plan p;
  bool pool;
  if (force > 0) {
    p = plan_from_count(T, force);
    pool = pw > 0 && want != kBlock / 64 && (want == pw || units * p.n_splits <= cus);
  } else {
    const PlanEngine e{want == kBlock / 64 ? 0 : pw, v8,
                       mbits == 0 && mode != kScoreFp16 && !v8};
    const Launch l = plan_launch(units, T, e, cus, plan_bound(B, Hkv, T).n_splits);
    p = l.plan;
    pool = pw > 0 && (want == pw || l.pool);
  }
  const WsLayout w = ws_layout(B, Hq, Hkv, p.n_splits);
  if (ws_bytes < w.total)
    return fail(POT_ERR_WORKSPACE, "workspace %zu bytes < %zu needed for %d splits", ws_bytes,
                w.total, p.n_splits);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  a.tickets = reinterpret_cast<unsigned long long*>(ws);
  a.ticket = pool && p.n_splits > 1 && p.n_splits <= kMaxMergedSplits ? next_ticket() : 0;
  a.part_m = reinterpret_cast<int32_t*>(ws + w.part_m);
  a.part_l = reinterpret_cast<float*>(ws + w.part_l);
  a.part_o = reinterpret_cast<float*>(ws + w.part_o);
  a.t_cap = t_cap;
  a.B = B;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.T = T;
  a.n_splits = p.n_splits;
  a.split_len = p.split_len;
  a.wg_waves = pool ? pw : kBlock / 64;
  a.claim_tiles = pool && claims_tiles(units, p, pw, cus);
  bool debug = false;
  hipEvent_t ev_begin = nullptr, ev_end = nullptr;
  if (dbg) {
    ev_begin = static_cast<hipEvent_t>(dbg->decode_begin);
    ev_end = static_cast<hipEvent_t>(dbg->decode_end);
    a.dbg_qhat = dbg->qhat;
    a.dbg_delta = dbg->delta;
    a.dbg_scores = dbg->scores;
    a.dbg_m_final = dbg->m_final;
    a.dbg_m_split = dbg->m_split;
    debug = dbg->qhat || dbg->delta || dbg->scores || dbg->m_final || dbg->m_split;
    dbg->n_splits = p.n_splits;
    dbg->split_len = p.split_len;
    dbg->wg_waves = a.wg_waves;
    if (debug && mode == kScoreFp16)
      return fail(POT_ERR_UNSUPPORTED, "debug taps are not available on the fp16 path");
  }
  return hip_status(
      launch_decode(mode, G, mant_bits, debug, vf, a, static_cast<hipStream_t>(stream), ev_begin,
                    ev_end),
      "decode launch");
}

// Shared body of the INT8-value entry points; vf 1: softmax weights, 2:
// power-of-two weights.
pot_status decode_v8(int vf, const pot_format* fmt, int32_t engine, const float* q,
                                   const uint8_t* codes_se, const uint8_t* codes_m,
                                   const float* key_scale, const uint8_t* v_u8,
                                   const int8_t* v_exp, int64_t t_cap,
                                   const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                   int32_t Hkv, int32_t T, float* out, void* workspace,
                                   size_t ws_bytes, pot_debug* dbg, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (engine != 0 && engine != 1)
    return fail(POT_ERR_INVALID_ARG, "engine %d (0 shift-accumulate, 1 byte decode)", engine);
  if (engine == 1 && fmt->mant_bits != 0)
    return fail(POT_ERR_UNSUPPORTED, "the byte-decode path scores PoT-4 codes only (mant_bits 0)");
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4) || (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale / codes_m");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.codes_m = codes_m;
  a.key_scale = key_scale;
  a.v8 = v_u8;
  a.v_exp = v_exp;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  return decode_common(engine == 0 ? kScorePot : kScoreDs4a, fmt->mant_bits, a, kv_head_of_q, B,
                       Hq, Hkv, T, t_cap, workspace, ws_bytes, dbg, stream, vf);
}

}  // namespace

extern "C" {

const char* pot_status_string(pot_status s) {
  switch (s) {
    case POT_OK: return "POT_OK";
    case POT_ERR_INVALID_ARG: return "POT_ERR_INVALID_ARG";
    case POT_ERR_UNSUPPORTED: return "POT_ERR_UNSUPPORTED";
    case POT_ERR_WORKSPACE: return "POT_ERR_WORKSPACE";
    case POT_ERR_HIP: return "POT_ERR_HIP";
  }
  return "POT_ERR_UNKNOWN";
}

const char* pot_last_error(void) { return g_last_error.c_str(); }

size_t pot_code_bytes_per_row(const pot_format* fmt) {
  if (check_format(fmt) != POT_OK) return 0;
  return 32 + 8 * (size_t)fmt->mant_bits;
}

pot_status pot_encode_keys(const pot_format* fmt, const uint16_t* k_fp16, int64_t n_rows,
                           int64_t out_row_stride, int32_t scale_mode, float* key_scale,
                           uint8_t* codes_se, uint8_t* codes_m, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (n_rows < 0) return fail(POT_ERR_INVALID_ARG, "n_rows %lld < 0", (long long)n_rows);
  if (out_row_stride < 1)
    return fail(POT_ERR_INVALID_ARG, "out_row_stride %lld < 1", (long long)out_row_stride);
  if (scale_mode != 0 && scale_mode != 1)
    return fail(POT_ERR_INVALID_ARG, "scale_mode %d (0 or 1)", scale_mode);
  if (n_rows == 0) return ok();
  if (!k_fp16 || !key_scale || !codes_se)
    return fail(POT_ERR_INVALID_ARG, "k_fp16, key_scale or codes_se is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(k_fp16, 16) || !aligned(codes_se, 16) || !aligned(key_scale, 4) ||
      (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned k_fp16 / codes_se / key_scale / codes_m");
  if (n_rows > (int64_t)1 << 36) return fail(POT_ERR_INVALID_ARG, "n_rows too large");
  const EncodeTables& tab = encode_tables(fmt->mant_bits);
  return hip_status(launch_encode_pot(k_fp16, n_rows, out_row_stride, scale_mode, fmt->hadamard,
                                      key_scale, codes_se, codes_m, tab,
                                      static_cast<hipStream_t>(stream)),
                    "encode launch");
}

pot_status pot_store_values(const uint16_t* v_fp16, int64_t n_seq, int64_t n_tok, int64_t t_cap,
                            int64_t t0, uint16_t* v_cache, void* stream) {
  if (n_seq < 0 || n_tok < 0)
    return fail(POT_ERR_INVALID_ARG, "n_seq %lld / n_tok %lld < 0", (long long)n_seq,
                (long long)n_tok);
  if (t_cap < 8 || t_cap % 8)
    return fail(POT_ERR_INVALID_ARG, "t_cap %lld is not a positive multiple of 8",
                (long long)t_cap);
  if (t0 < 0 || t0 + n_tok > t_cap)
    return fail(POT_ERR_INVALID_ARG, "tokens [%lld, %lld) outside [0, t_cap = %lld)",
                (long long)t0, (long long)(t0 + n_tok), (long long)t_cap);
  if (n_seq == 0 || n_tok == 0) return ok();
  if (!v_fp16 || !v_cache) return fail(POT_ERR_INVALID_ARG, "v_fp16 or v_cache is NULL");
  if (!aligned(v_fp16, 16) || !aligned(v_cache, 16))
    return fail(POT_ERR_INVALID_ARG, "v_fp16 and v_cache must be 16-byte aligned");
  return hip_status(launch_store_values(v_fp16, n_seq, n_tok, t_cap, t0, v_cache,
                                        static_cast<hipStream_t>(stream)),
                    "store values launch");
}

pot_status pot_store_values_int8(const uint16_t* v_fp16, int64_t n_seq, int64_t n_tok,
                                 int64_t t_cap, int64_t t0, uint8_t* v_u8, int8_t* v_exp,
                                 void* stream) {
  if (n_seq < 0 || n_tok < 0)
    return fail(POT_ERR_INVALID_ARG, "n_seq %lld / n_tok %lld < 0", (long long)n_seq,
                (long long)n_tok);
  if (t_cap < 8 || t_cap % 8)
    return fail(POT_ERR_INVALID_ARG, "t_cap %lld is not a positive multiple of 8",
                (long long)t_cap);
  if (t0 < 0 || t0 + n_tok > t_cap)
    return fail(POT_ERR_INVALID_ARG, "tokens [%lld, %lld) outside [0, t_cap = %lld)",
                (long long)t0, (long long)(t0 + n_tok), (long long)t_cap);
  if (n_seq == 0 || n_tok == 0) return ok();
  if (!v_fp16 || !v_u8 || !v_exp)
    return fail(POT_ERR_INVALID_ARG, "v_fp16, v_u8 or v_exp is NULL");
  if (!aligned(v_fp16, 16) || !aligned(v_u8, 16) || !aligned(v_exp, 16))
    return fail(POT_ERR_INVALID_ARG, "v_fp16, v_u8 and v_exp must be 16-byte aligned");
  if (n_seq > ((int64_t)1 << 31) / n_tok)
    return fail(POT_ERR_INVALID_ARG, "n_seq * n_tok too large");
  return hip_status(launch_store_values_i8(v_fp16, n_seq, n_tok, t_cap, t0, v_u8, v_exp,
                                           static_cast<hipStream_t>(stream)),
                    "store values launch");
}

size_t pot_decode_workspace_bytes(int32_t B, int32_t Hq, int32_t Hkv, int32_t T) {
  if (!shape_ok(B, Hq, Hkv, T)) return 0;
  return ws_layout(B, Hq, Hkv, plan_bound(B, Hkv, T).n_splits).total;
}

size_t pot_decode_workspace_bytes_for_splits(int32_t B, int32_t Hq, int32_t Hkv, int32_t T,
                                             int32_t n_splits) {
  if (!shape_ok(B, Hq, Hkv, T) || n_splits < 0) return 0;
  const Plan p = n_splits > 0 ? plan_from_count(T, n_splits) : plan_bound(B, Hkv, T);
  return ws_layout(B, Hq, Hkv, p.n_splits).total;
}

pot_status pot_workspace_init(void* workspace, size_t ws_bytes, void* stream) {
  if (!workspace) return fail(POT_ERR_INVALID_ARG, "workspace is NULL");
  return hip_status(launch_fill_zero(workspace, ws_bytes, static_cast<hipStream_t>(stream)),
                    "workspace init");
}

pot_status pot_decode_attention(const pot_format* fmt, const float* q, const uint8_t* codes_se,
                                const uint8_t* codes_m, const float* key_scale,
                                const uint16_t* v_cache, int64_t t_cap,
                                const int32_t* kv_head_of_q, int32_t B, int32_t Hq, int32_t Hkv,
                                int32_t T, float* out, void* workspace, size_t ws_bytes,
                                pot_debug* dbg, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4) || (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale / codes_m");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.codes_m = codes_m;
  a.key_scale = key_scale;
  a.v = v_cache;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  return decode_common(kScorePot, fmt->mant_bits, a, kv_head_of_q, B, Hq, Hkv, T, t_cap,
                       workspace, ws_bytes, dbg, stream);
}

pot_status pot_append_decode_attention(const pot_format* fmt, const float* q,
                                       const uint16_t* k_new, const uint16_t* v_new,
                                       uint8_t* codes_se, uint8_t* codes_m, float* key_scale,
                                       uint16_t* v_cache, int64_t t_cap,
                                       const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                       int32_t Hkv, int32_t T, float* out, void* workspace,
                                       size_t ws_bytes, pot_debug* dbg, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (!k_new || !v_new) return fail(POT_ERR_INVALID_ARG, "k_new or v_new is NULL");
  if (!aligned(k_new, 16) || !aligned(v_new, 16))
    return fail(POT_ERR_INVALID_ARG, "k_new and v_new must be 16-byte aligned");
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4) || (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale / codes_m");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.codes_m = codes_m;
  a.key_scale = key_scale;
  a.v = v_cache;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  a.app_k = k_new;
  a.app_v = v_new;
  a.app_codes_se = codes_se;
  a.app_codes_m = codes_m;
  a.app_key_scale = key_scale;
  a.app_v_cache = v_cache;
  a.app_tab = encode_tables(fmt->mant_bits);
  return decode_common(kScorePot, fmt->mant_bits, a, kv_head_of_q, B, Hq, Hkv, T, t_cap,
                       workspace, ws_bytes, dbg, stream);
}

pot_status pot_decode_attention_v8(const pot_format* fmt, int32_t engine, const float* q,
                                   const uint8_t* codes_se, const uint8_t* codes_m,
                                   const float* key_scale, const uint8_t* v_u8,
                                   const int8_t* v_exp, int64_t t_cap,
                                   const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                   int32_t Hkv, int32_t T, float* out, void* workspace,
                                   size_t ws_bytes, pot_debug* dbg, void* stream) {
  return decode_v8(1, fmt, engine, q, codes_se, codes_m, key_scale, v_u8, v_exp, t_cap,
                   kv_head_of_q, B, Hq, Hkv, T, out, workspace, ws_bytes, dbg, stream);
}

pot_status pot_decode_attention_v8_pow2(const pot_format* fmt, int32_t engine, const float* q,
                                        const uint8_t* codes_se, const uint8_t* codes_m,
                                        const float* key_scale, const uint8_t* v_u8,
                                        const int8_t* v_exp, int64_t t_cap,
                                        const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                        int32_t Hkv, int32_t T, float* out, void* workspace,
                                        size_t ws_bytes, pot_debug* dbg, void* stream) {
  return decode_v8(2, fmt, engine, q, codes_se, codes_m, key_scale, v_u8, v_exp, t_cap,
                   kv_head_of_q, B, Hq, Hkv, T, out, workspace, ws_bytes, dbg, stream);
}

pot_status pot_append_decode_attention_v8(const pot_format* fmt, int32_t engine,
                                          const float* q, const uint16_t* k_new,
                                          const uint16_t* v_new, uint8_t* codes_se,
                                          uint8_t* codes_m, float* key_scale, uint8_t* v_u8,
                                          int8_t* v_exp, int64_t t_cap,
                                          const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                          int32_t Hkv, int32_t T, float* out, void* workspace,
                                          size_t ws_bytes, pot_debug* dbg, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (engine != 0 && engine != 1)
    return fail(POT_ERR_INVALID_ARG, "engine %d (0 shift-accumulate, 1 byte decode)", engine);
  if (engine == 1 && fmt->mant_bits != 0)
    return fail(POT_ERR_UNSUPPORTED, "the byte-decode path scores PoT-4 codes only (mant_bits 0)");
  if (!k_new || !v_new) return fail(POT_ERR_INVALID_ARG, "k_new or v_new is NULL");
  if (!aligned(k_new, 16) || !aligned(v_new, 16))
    return fail(POT_ERR_INVALID_ARG, "k_new and v_new must be 16-byte aligned");
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4) || (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale / codes_m");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.codes_m = codes_m;
  a.key_scale = key_scale;
  a.v8 = v_u8;
  a.v_exp = v_exp;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  a.app_k = k_new;
  a.app_v = v_new;
  a.app_codes_se = codes_se;
  a.app_codes_m = codes_m;
  a.app_key_scale = key_scale;
  a.app_v8 = v_u8;
  a.app_v_exp = v_exp;
  a.app_tab = encode_tables(fmt->mant_bits);
  return decode_common(engine == 0 ? kScorePot : kScoreDs4a, fmt->mant_bits, a, kv_head_of_q, B,
                       Hq, Hkv, T, t_cap, workspace, ws_bytes, dbg, stream, 1);
}

pot_status pot_ds4a_decode_attention(const pot_format* fmt, const float* q,
                                     const uint8_t* codes_se, const float* key_scale,
                                     const uint16_t* v_cache, int64_t t_cap,
                                     const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                     int32_t Hkv, int32_t T, float* out, void* workspace,
                                     size_t ws_bytes, pot_debug* dbg, void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (fmt->mant_bits != 0)
    return fail(POT_ERR_UNSUPPORTED, "the byte-decode path scores PoT-4 codes only (mant_bits 0)");
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.key_scale = key_scale;
  a.v = v_cache;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  return decode_common(kScoreDs4a, 0, a, kv_head_of_q, B, Hq, Hkv, T, t_cap, workspace, ws_bytes,
                       dbg, stream);
}

pot_status pot_dot_decode_attention(const pot_format* fmt, const float* q,
                                    const uint8_t* codes_se, const uint8_t* codes_m,
                                    const float* key_scale, const uint16_t* v_cache,
                                    int64_t t_cap, const int32_t* kv_head_of_q, int32_t B,
                                    int32_t Hq, int32_t Hkv, int32_t T, float* out,
                                    void* workspace, size_t ws_bytes, pot_debug* dbg,
                                    void* stream) {
  pot_status st = check_format(fmt);
  if (st != POT_OK) return st;
  if (!codes_se || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes_se or key_scale is NULL");
  if ((fmt->mant_bits > 0) != (codes_m != nullptr))
    return fail(POT_ERR_INVALID_ARG, "codes_m must be non-NULL exactly when mant_bits > 0");
  if (!aligned(codes_se, 16) || !aligned(key_scale, 4) || (codes_m && !aligned(codes_m, 8)))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes_se / key_scale / codes_m");
  DecodeArgs a{};
  a.q = q;
  a.codes_se = codes_se;
  a.codes_m = codes_m;
  a.key_scale = key_scale;
  a.v = v_cache;
  a.out = out;
  a.frac_bits = fmt->frac_bits;
  a.hadamard = fmt->hadamard;
  return decode_common(kScoreDs4a, fmt->mant_bits, a, kv_head_of_q, B, Hq, Hkv, T, t_cap,
                       workspace, ws_bytes, dbg, stream);
}

pot_status pot_int8_encode_keys(const uint16_t* k_fp16, int64_t n_rows, int64_t out_row_stride,
                                int32_t hadamard, float* key_scale, int8_t* codes, void* stream) {
  if (n_rows < 0) return fail(POT_ERR_INVALID_ARG, "n_rows %lld < 0", (long long)n_rows);
  if (out_row_stride < 1)
    return fail(POT_ERR_INVALID_ARG, "out_row_stride %lld < 1", (long long)out_row_stride);
  if (hadamard != 0 && hadamard != 1)
    return fail(POT_ERR_INVALID_ARG, "hadamard %d (0 or 1)", hadamard);
  if (n_rows == 0) return ok();
  if (!k_fp16 || !key_scale || !codes)
    return fail(POT_ERR_INVALID_ARG, "k_fp16, key_scale or codes is NULL");
  if (!aligned(k_fp16, 16) || !aligned(codes, 16) || !aligned(key_scale, 4))
    return fail(POT_ERR_INVALID_ARG, "misaligned k_fp16 / codes / key_scale");
  return hip_status(launch_encode_int8(k_fp16, n_rows, out_row_stride, hadamard, key_scale,
                                       codes, static_cast<hipStream_t>(stream)),
                    "int8 encode launch");
}

pot_status pot_int8_decode_attention(const float* q, const int8_t* codes, const float* key_scale,
                                     const uint16_t* v_cache, int64_t t_cap,
                                     const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                     int32_t Hkv, int32_t T, int32_t hadamard, float* out,
                                     void* workspace, size_t ws_bytes, pot_debug* dbg,
                                     void* stream) {
  if (hadamard != 0 && hadamard != 1)
    return fail(POT_ERR_INVALID_ARG, "hadamard %d (0 or 1)", hadamard);
  if (!codes || !key_scale) return fail(POT_ERR_INVALID_ARG, "codes or key_scale is NULL");
  if (!aligned(codes, 16) || !aligned(key_scale, 4))
    return fail(POT_ERR_INVALID_ARG, "misaligned codes / key_scale");
  DecodeArgs a{};
  a.q = q;
  a.codes_i8 = codes;
  a.key_scale = key_scale;
  a.v = v_cache;
  a.out = out;
  a.hadamard = hadamard;
  return decode_common(kScoreInt8, 0, a, kv_head_of_q, B, Hq, Hkv, T, t_cap, workspace, ws_bytes,
                       dbg, stream);
}

pot_status pot_fp16_decode_attention(const float* q, const uint16_t* k_fp16,
                                     const uint16_t* v_cache, int64_t t_cap,
                                     const int32_t* kv_head_of_q, int32_t B, int32_t Hq,
                                     int32_t Hkv, int32_t T, float* out, void* workspace,
                                     size_t ws_bytes, void* stream) {
  if (!k_fp16) return fail(POT_ERR_INVALID_ARG, "k_fp16 is NULL");
  if (!aligned(k_fp16, 16)) return fail(POT_ERR_INVALID_ARG, "k_fp16 must be 16-byte aligned");
  DecodeArgs a{};
  a.q = q;
  a.k_f16 = k_fp16;
  a.v = v_cache;
  a.out = out;
  return decode_common(kScoreFp16, 0, a, kv_head_of_q, B, Hq, Hkv, T, t_cap, workspace, ws_bytes,
                       nullptr, stream);
}

}  // extern "C"
