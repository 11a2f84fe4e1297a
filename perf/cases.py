"""The work that a decoder with a power-of-two key cache has this library do, as timed cases.

Three kinds of call, at the head shapes, key formats and value formats of the tests and the benchmark:

- "append": one decode step of one layer. The new token's key and values are appended to the cache and its queries
  attend over all T keys, in one call (pot_append_decode_attention, pot_append_decode_attention_v8).
- "decode": attention over a cache that stands as it is (pot_decode_attention, pot_decode_attention_v8,
  pot_decode_attention_v8_pow2) and the decoded-code engines over the same cache (pot_ds4a_decode_attention,
  pot_dot_decode_attention).
- "prefill": a prompt's keys are encoded and its values stored (pot_encode_keys with pot_store_values or
  pot_store_values_int8).

Keys are N(0, 1) times a per-channel scale from U[0.5, 4] (outlier channels), values and queries N(0, 1).
"""
import math

import numpy as np
import torch

import paper_2609_09208_amd as pa

DEV = "cuda:0"
D = 64


def _case(kind, B, Hq, Hkv, T, t_cap, k, hadamard=False, values="fp16", engine="sac", name=None):
    c = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, T=T, t_cap=t_cap, k=k, hadamard=hadamard, values=values, engine=engine)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one short chat: latency of a step, a few hundred kilobytes of cache
        _case("append", 1, 32, 4, 1024, 2048, 0, name="append_pot4_b1_t1024"),
        # one long document
        _case("append", 1, 32, 4, 32768, 32768, 0, name="append_pot4_b1_t32768"),
        # a few sequences of odd length, four query heads per kv head, with a mantissa bit
        _case("decode", 3, 16, 4, 3001, 4096, 1, name="decode_m1_b3_t3001_g4"),
        # an ordinary serving batch, ordinary context
        _case("append", 16, 32, 4, 4096, 4096, 0, name="append_pot4_b16_t4096"),
        # the same batch, long context, the two accurate formats: one mantissa bit, and Hadamard with four
        _case("append", 16, 32, 4, 16384, 16384, 1, name="append_m1_b16_t16384"),
        _case("append", 8, 32, 4, 32768, 32768, 4, hadamard=True, name="append_m4_hadamard_b8_t32768"),
        # codes for the values too: the smallest cache
        _case("append", 16, 32, 4, 16384, 16384, 0, values="int8", name="append_pot4_int8v_b16_t16384"),
        # the largest step: 64 sequences of 32768 keys (the benchmark's layer)
        _case("append", 64, 32, 4, 32768, 32768, 0, name="append_pot4_b64_t32768"),
        # the decoded-weight engine, for programs that want the accurate format and do not mind a multiply
        _case("decode", 16, 32, 4, 8192, 8192, 4, engine="dot", name="decode_dot_m4_b16_t8192"),
        # prefill: four prompts of ordinary length; one long prompt in the most accurate formats; one short odd prompt
        # at the head of a longer cache (one encode call per kv head, since its rows are not one dense block)
        _case("prefill", 4, 32, 4, 8192, 8192, 0, name="prefill_pot4_b4_t8192"),
        _case("prefill", 1, 32, 4, 32768, 32768, 4, hadamard=True, values="int8",
              name="prefill_m4_hadamard_int8v_t32768"),
        _case("prefill", 1, 32, 4, 777, 2048, 1, values="int8", name="prefill_m1_int8v_t777"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["append", "append", "decode", "prefill"])
    Hq, Hkv = rng.choice([(32, 4), (32, 4), (32, 8), (16, 4), (16, 8), (8, 8), (64, 8)])
    k = rng.choice([0, 0, 1, 2, 3, 4])
    hadamard = rng.random() < 0.25
    values = rng.choice(["fp16", "fp16", "int8"])
    engine = "sac"
    if kind == "decode":
        engine = rng.choice(["sac", "sac", "bytes", "dot", "pow2"])
        if engine == "bytes":
            k = 0
        elif engine == "pow2":
            values = "int8"
        elif engine == "dot":
            values = "fp16"
    # B and T over their whole range, together at most a quarter of the largest listed step's keys
    most = 2 ** 21 if kind != "prefill" else 2 ** 17
    T = _log_int(rng, 130, 32768)
    B = _log_int(rng, 1, max(1, min(64, most // (T * Hkv))))
    room = rng.choice([0, 0, 1000])
    t_cap = (T + room + 7) // 8 * 8
    if kind == "prefill" and t_cap != T:
        B = min(B, 4)
    return _case(kind, B, Hq, Hkv, T, t_cap, k, hadamard, values, engine)


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _keys_values(case, g):
    """fp16 keys and values [B * Hkv][rows][64] of the cache: all t_cap rows, or the prompt's T rows."""
    B, Hkv = case["B"], case["Hkv"]
    rows = case["T"] if case["kind"] == "prefill" else case["t_cap"]
    c = torch.rand((Hkv, 1, D), generator=g, device=DEV) * 3.5 + 0.5
    k = torch.empty((B, Hkv, rows, D), dtype=torch.float16, device=DEV)
    v = torch.empty((B, Hkv, rows, D), dtype=torch.float16, device=DEV)
    for b in range(B):
        k[b] = torch.randn((Hkv, rows, D), generator=g, device=DEV) * c
        v[b] = torch.randn((Hkv, rows, D), generator=g, device=DEV)
    return k.view(B * Hkv, rows, D), v.view(B * Hkv, rows, D), c


def _step_inputs(case, g, c):
    """The queries and, for an appending step, the new token's key and values."""
    B, Hq, Hkv = case["B"], case["Hq"], case["Hkv"]
    q = torch.randn((B, Hq, D), generator=g, device=DEV)
    k_new = (torch.randn((B, Hkv, D), generator=g, device=DEV) * c.view(1, Hkv, D)).to(torch.float16)
    v_new = torch.randn((B, Hkv, D), generator=g, device=DEV).to(torch.float16)
    return q, k_new, v_new


def _empty_cache(case):
    B, Hkv, t_cap = case["B"], case["Hkv"], case["t_cap"]
    cache = pa.alloc_pot_cache(B, Hkv, t_cap, case["k"], DEV)
    if case["values"] == "int8":
        cache["v_u8"], cache["v_exp"] = pa.alloc_value_cache_int8(B, Hkv, t_cap, DEV)
    else:
        cache["v"] = pa.alloc_value_cache(B, Hkv, t_cap, DEV)
    return cache


def _fill(case, fmt, cache, k, v):
    """Encodes the keys and stores the values of a prompt (rows 0 .. of every sequence)."""
    n_seq, rows, _ = k.shape
    t_cap = case["t_cap"]
    se, cm, sc = cache["codes_se"], cache["codes_m"], cache["key_scale"]
    if rows == t_cap:
        pa.pot_encode_keys(fmt, k, n_seq * rows, 1, 0, sc, se, cm)
    else:
        kb = case["k"] * 8
        for s in range(n_seq):
            pa.pot_encode_keys(fmt, k.data_ptr() + s * rows * D * 2, rows, 1, 0, sc.data_ptr() + s * t_cap * 4,
                               se.data_ptr() + s * t_cap * 32, cm.data_ptr() + s * t_cap * kb if kb else None)
    if case["values"] == "int8":
        pa.pot_store_values_int8(v, n_seq, rows, t_cap, 0, cache["v_u8"], cache["v_exp"])
    else:
        pa.pot_store_values(v, n_seq, rows, t_cap, 0, cache["v"])


def prepare(case, seed):
    g = _generator(seed)
    fmt = pa.make_format(mant_bits=case["k"], hadamard=case["hadamard"])
    k, v, c = _keys_values(case, g)
    state = dict(case=case, fmt=fmt, cache=_empty_cache(case))
    if case["kind"] == "prefill":
        state.update(k=k, v=v)
        return state
    _fill(case, fmt, state["cache"], k, v)
    B, Hq, Hkv, T = case["B"], case["Hq"], case["Hkv"], case["T"]
    state["q"], state["k_new"], state["v_new"] = _step_inputs(case, g, c)
    state["heads"] = np.arange(Hq, dtype=np.int32) // (Hq // Hkv)
    state["out"] = torch.empty((B, Hq, D), dtype=torch.float32, device=DEV)
    state["ws"] = pa.alloc_workspace(pa.pot_decode_workspace_bytes(B, Hq, Hkv, T), DEV)
    return state


def run(state):
    case, fmt, cache = state["case"], state["fmt"], state["cache"]
    if case["kind"] == "prefill":
        _fill(case, fmt, cache, state["k"], state["v"])
        return {n: t for n, t in cache.items() if t is not None}
    q, heads, out, ws = state["q"], state["heads"], state["out"], state["ws"]
    B, Hq, Hkv, T, t_cap = case["B"], case["Hq"], case["Hkv"], case["T"], case["t_cap"]
    se, cm, sc = cache["codes_se"], cache["codes_m"], cache["key_scale"]
    if case["kind"] == "append":
        if case["values"] == "int8":
            pa.pot_append_decode_attention_v8(fmt, 0, q, state["k_new"], state["v_new"], se, cm, sc, cache["v_u8"],
                                              cache["v_exp"], t_cap, heads, B, Hq, Hkv, T, out, ws)
        else:
            pa.pot_append_decode_attention(fmt, q, state["k_new"], state["v_new"], se, cm, sc, cache["v"], t_cap,
                                           heads, B, Hq, Hkv, T, out, ws)
        return dict(out=out, **{n: t for n, t in cache.items() if t is not None})
    engine = case["engine"]
    if engine == "pow2":
        pa.pot_decode_attention_v8_pow2(fmt, 0, q, se, cm, sc, cache["v_u8"], cache["v_exp"], t_cap, heads, B, Hq,
                                        Hkv, T, out, ws)
    elif case["values"] == "int8":
        pa.pot_decode_attention_v8(fmt, 1 if engine == "bytes" else 0, q, se, cm, sc, cache["v_u8"], cache["v_exp"],
                                   t_cap, heads, B, Hq, Hkv, T, out, ws)
    elif engine == "bytes":
        pa.pot_ds4a_decode_attention(fmt, q, se, sc, cache["v"], t_cap, heads, B, Hq, Hkv, T, out, ws)
    elif engine == "dot":
        pa.pot_dot_decode_attention(fmt, q, se, cm, sc, cache["v"], t_cap, heads, B, Hq, Hkv, T, out, ws)
    else:
        pa.pot_decode_attention(fmt, q, se, cm, sc, cache["v"], t_cap, heads, B, Hq, Hkv, T, out, ws)
    return dict(out=out)


def work(case):
    rows = case["B"] * case["Hkv"] * case["T"]
    cache = 32 + 8 * case["k"] + 4 + (65 if case["values"] == "int8" else 128)  # bytes of one cache row
    if case["kind"] == "prefill":
        return {"bytes": rows * (256 + cache), "flops": rows * D * (12 if case["hadamard"] else 4)}
    heads = case["B"] * case["Hq"]
    new = case["B"] * case["Hkv"] * (256 + cache) if case["kind"] == "append" else 0
    return {"bytes": rows * cache + heads * D * 8 + new, "flops": heads * case["T"] * D * 4}


def tolerance(case):
    # Codes, scales and stored values are exact (whole values may not differ at all; a scale is a maximum, or one
    # rounding of an exact sum). The attention output is made of fp32 sums over up to 32768 keys, of weights from a
    # hardware exp2: 1.8e-7 to 6.4e-7 was measured against 64 bits. Values held as bytes reach the matrix cores with an
    # offset of 1152 that is taken off the fp32 sums: 1.9e-5 to 2.0e-5 was measured.
    return {"rel": 8e-5 if case["values"] == "int8" else 2.5e-6}


def _fwht(x):
    """Walsh-Hadamard transform of the last axis (64 elements), stages of span 1, 2, 4, .. 32."""
    h = 1
    while h < D:
        y = x.reshape(*x.shape[:-1], D // (2 * h), 2, h)
        x = torch.stack((y[..., 0, :] + y[..., 1, :], y[..., 0, :] - y[..., 1, :]), dim=-2).reshape(x.shape)
        h *= 2
    return x


def _rotated(case, x):
    """The vectors that the quantisers see, as the fp32 numbers they are rounded to, in fp64."""
    x = x.double()
    return (_fwht(x) / 8).float().double() if case["hadamard"] else x


def _decoded_keys(case, k):
    """fp64 keys as the codes hold them: sign, (1 + j / 2^k) 2^-e nearest in log2 distance, times the row's absmax."""
    x = _rotated(case, k)
    s = x.abs().amax(-1, keepdim=True)
    n = 2 ** case["k"]
    u = (x.abs() / s).float().double()
    m, e = torch.frexp(u)  # m in [0.5, 1)
    m, e = m * 2 * n, (e - 1).double()
    t = m.floor()
    t = t + ((m * m) > t * (t + 1)).double()
    val = (t / n) * torch.exp2(e)
    low = 2.0 ** -6
    val = torch.where(val < low, torch.full_like(val, low), val)
    val = torch.where(u * u > 2.0 ** -13, val.clamp(max=2 - 1 / n), torch.zeros_like(val))
    return torch.sign(x) * val * s, s[..., 0]


def _decoded_values(case, v):
    v = v.double()
    if case["values"] != "int8":
        return v
    amax = v.abs().amax(-1, keepdim=True)
    g = torch.floor(torch.log2(127.0 / amax))
    g = torch.where(amax * torch.exp2(g) > 127, g - 1, g)
    g = torch.where(amax * torch.exp2(g + 1) <= 127, g + 1, g)
    g = torch.where(amax > 0, g, torch.zeros_like(g))
    return torch.round(v * torch.exp2(g)) * torch.exp2(-g)


def _decoded_queries(case, q):
    x = _rotated(case, q)
    amax = x.abs().amax(-1, keepdim=True)
    step = (amax / 127).float().double()
    inv = (127 / amax).float().double()
    return torch.round((x * inv).float().double()).clamp(-127, 127) * step


def exact(case, seed):
    if case["engine"] == "pow2":
        return None  # its weights are steps: a tie that 32 and 64 bits see differently is no error
    g = _generator(seed)
    k, v, c = _keys_values(case, g)
    n_seq, rows, _ = k.shape
    t_cap = case["t_cap"]
    none = {n: None for n in ("codes_se", "codes_m", "v_u8", "v_exp", "key_scale", "v")
            if not ((n == "codes_m" and not case["k"]) or (n == "v" and case["values"] == "int8")
                    or (n in ("v_u8", "v_exp") and case["values"] != "int8"))}
    if case["kind"] == "prefill":
        scale = torch.zeros((n_seq, t_cap), dtype=torch.float64, device=DEV)
        for s in range(n_seq):
            scale[s, :rows] = _decoded_keys(case, k[s])[1]
        got = dict(none, key_scale=scale.view(case["B"], case["Hkv"], t_cap))
        if case["values"] != "int8":
            out = torch.zeros((n_seq, t_cap, D), dtype=torch.float64, device=DEV)
            out[:, :rows] = v
            out = out.view(n_seq, t_cap // 8, 8, D).transpose(2, 3)
            got["v"] = out.reshape(case["B"], case["Hkv"], t_cap, D)
        return got
    B, Hq, Hkv, T = case["B"], case["Hq"], case["Hkv"], case["T"]
    q, k_new, v_new = _step_inputs(case, g, c)
    G = Hq // Hkv
    qd = _decoded_queries(case, q).view(B * Hkv, G, D)
    out = torch.empty((B * Hkv, G, D), dtype=torch.float64, device=DEV)
    for s in range(n_seq):
        ks, vs = k[s, :T], v[s, :T]
        if case["kind"] == "append":
            ks, vs = ks.clone(), vs.clone()
            ks[T - 1], vs[T - 1] = k_new.view(-1, D)[s], v_new.view(-1, D)[s]
        kd, vd = _decoded_keys(case, ks)[0], _decoded_values(case, vs)
        p = torch.softmax(qd[s] @ kd.t().contiguous() / 8, dim=-1)
        out[s] = p @ vd
    got = dict(out=out.view(B, Hq, D))
    return dict(got, **none) if case["kind"] == "append" else got
