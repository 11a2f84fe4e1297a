"""The launch plan's cases at their borders: one split of CU-wide workgroups up
to 768 keys (and up to 16 tiles when a quarter of the CUs has a unit), splits
that give each CU at most one workgroup, one split of four-wave workgroups above
one unit per CU and CU-wide ones from 8192 keys on, in three splits just above;
between half the CUs and all of them more splits of four-wave workgroups for long
ranges. Each call is compared with four-wave workgroups at one split on the same cache:
scores and maxima bit-identical, O to fp32 rounding. A wave whose first tile
holds the appended row loads it after the others: the appended calls go over
lengths that put that row in every wave's place.
"""
import numpy as np
import pytest
import torch

import paper_2609_09208_amd as pa
from parity_util import DEV, gpu_encode, gpu_pot_decode, to_dev
from workloads import make_decode_inputs, make_decode_inputs_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,T,k,splits,waves", [
    (1, 8, 1, 768, 0, 1, 16), (1, 8, 1, 769, 0, 4, 16), (1, 8, 1, 768, 4, 1, 12),
    (16, 32, 4, 1024, 0, 1, 16), (15, 32, 4, 1024, 0, 4, 16), (16, 32, 4, 1025, 0, 3, 16),
    (16, 32, 4, 1024, 3, 4, 12), (64, 16, 4, 300, 1, 1, 16), (65, 16, 4, 300, 1, 1, 4)])
def test_plan_matches_one_split_of_four_waves(B, Hq, Hkv, T, k, splits, waves):
    d = make_decode_inputs(900 + T + B, B=B, Hq=Hq, Hkv=Hkv, T=T)
    se, cm, sc = gpu_encode(d["k_bits"].reshape(-1, 64), k)
    a = gpu_pot_decode(d, se, cm, sc, mant_bits=k)
    b = gpu_pot_decode(d, se, cm, sc, mant_bits=k, force_splits=1, wg_waves=4)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (a["n_splits"], a["wg_waves"]) == (splits, waves)
    for key in ("qhat", "scores", "m_final"):
        assert np.array_equal(a[key], b[key]), key
    assert np.abs(a["out"] - b["out"]).max() <= 1e-5


@pytest.mark.parametrize("B,T", [(33, 8191), (33, 8192), (42, 8192), (43, 8192), (46, 8192)])
def test_plan_above_one_unit_per_cu(B, T):
    Hq = Hkv = 8
    d = make_decode_inputs_device(77, B, Hq, Hkv, T, DEV, t_cap=8192)
    fmt = pa.make_format(0)
    c = pa.alloc_pot_cache(B, Hkv, 8192, 0, DEV)
    pa.pot_encode_keys(fmt, d["k"], B * Hkv * 8192, 1, 0, c["key_scale"], c["codes_se"], None)
    v = pa.alloc_value_cache(B, Hkv, 8192, DEV)
    pa.pot_store_values(d["v"], B * Hkv, 8192, 8192, 0, v)
    outs = []
    for splits, waves in ((0, 0), (1, 4)):
        dbg = pa.pot_debug()
        dbg.force_splits, dbg.force_wg_waves = splits, waves
        m = torch.empty((B, Hq), dtype=torch.int32, device=DEV)
        dbg.m_final = m.data_ptr()
        out = torch.empty((B, Hq, 64), dtype=torch.float32, device=DEV)
        ws = pa.alloc_workspace(pa.pot_decode_workspace_bytes(B, Hq, Hkv, T), DEV)
        pa.pot_decode_attention(fmt, d["q"], c["codes_se"], None, c["key_scale"], v, 8192,
                                d["kv_head_of_q"], B, Hq, Hkv, T, out, ws, dbg=dbg)
        torch.cuda.synchronize()
        outs.append((out.cpu().numpy(), m.cpu().numpy(), dbg.n_splits, dbg.wg_waves))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        want = {(33, 8191): (1, 4), (33, 8192): (3, 16), (42, 8192): (3, 16), (43, 8192): (1, 16),
                (46, 8192): (1, 16)}[(B, T)]
        assert outs[0][2:] == want
    assert np.array_equal(outs[0][1], outs[1][1])
    assert np.abs(outs[0][0] - outs[1][0]).max() <= 1e-5


@pytest.mark.parametrize("units,T,k,values,want", [
    (136, 12287, 0, "fp16", (1, 16)), (136, 12288, 0, "fp16", (3, 4)), (152, 12288, 0, "fp16", (3, 4)),
    (160, 12288, 0, "fp16", (1, 16)), (168, 12288, 1, "fp16", (3, 4)), (176, 12288, 4, "fp16", (1, 12)),
    (128, 12288, 0, "int8", (2, 16)), (136, 12288, 0, "int8", (7, 4)), (160, 12288, 1, "int8", (6, 4)),
    (192, 12288, 0, "int8", (4, 4)), (200, 12288, 0, "int8", (1, 16))])
def test_plan_between_half_the_cus_and_all(units, T, k, values, want):
    # one CU-wide workgroup per unit would leave up to half of the CUs without work
    B, Hkv = units // 8, 8
    cap = -(-T // 8) * 8
    d = make_decode_inputs_device(78, B, Hkv, Hkv, T, DEV, t_cap=cap)
    fmt = pa.make_format(k)
    c = pa.alloc_pot_cache(B, Hkv, cap, k, DEV)
    pa.pot_encode_keys(fmt, d["k"], units * cap, 1, 0, c["key_scale"], c["codes_se"], c["codes_m"])
    v = (pa.alloc_value_cache_int8(B, Hkv, cap, DEV) if values == "int8"
         else (pa.alloc_value_cache(B, Hkv, cap, DEV),))
    (pa.pot_store_values_int8 if values == "int8" else pa.pot_store_values)(d["v"], units, cap, cap,
                                                                            0, *v)
    ws = pa.alloc_workspace(pa.pot_decode_workspace_bytes(B, Hkv, Hkv, T), DEV)
    outs = []
    for splits, waves in ((0, 0), (1, 4)):
        dbg = pa.pot_debug()
        dbg.force_splits, dbg.force_wg_waves = splits, waves
        m = torch.empty((B, Hkv), dtype=torch.int32, device=DEV)
        dbg.m_final = m.data_ptr()
        out = torch.empty((B, Hkv, 64), dtype=torch.float32, device=DEV)
        a = (cap, d["kv_head_of_q"], B, Hkv, Hkv, T, out, ws)
        if values == "int8":
            pa.pot_decode_attention_v8(fmt, 0, d["q"], c["codes_se"], c["codes_m"], c["key_scale"],
                                       *v, *a, dbg=dbg)
        else:
            pa.pot_decode_attention(fmt, d["q"], c["codes_se"], c["codes_m"], c["key_scale"], *v, *a,
                                    dbg=dbg)
        torch.cuda.synchronize()
        outs.append((out.cpu().numpy(), m.cpu().numpy(), dbg.n_splits, dbg.wg_waves))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert outs[0][2:] == want
    assert np.array_equal(outs[0][1], outs[1][1])
    assert np.abs(outs[0][0] - outs[1][0]).max() <= 1e-5


@pytest.mark.parametrize("values", ["fp16", "int8"])
@pytest.mark.parametrize("waves", [4, 16])
def test_appended_row_in_every_place(values, waves):
    # T = 1 .. 1025 over one split: the appended row is the first tile's last, a later tile's
    # first, or alone in its tile; the reference appends with the separate calls
    B, Hq, Hkv, t_cap = 2, 8, 2, 1040
    d = make_decode_inputs(5, B=B, Hq=Hq, Hkv=Hkv, T=t_cap)
    fmt = pa.make_format(1)
    kk = to_dev(d["k_bits"].reshape(B * Hkv, t_cap, 64)).view(torch.float16)
    vv = to_dev(d["v_bits"].reshape(B * Hkv, t_cap, 64)).view(torch.float16)
    q = to_dev(d["q"])
    ws = pa.alloc_workspace(pa.pot_decode_workspace_bytes(B, Hq, Hkv, t_cap), DEV)

    def cache(n):
        c = pa.alloc_pot_cache(B, Hkv, t_cap, 1, DEV)
        c["codes_se"].fill_(0x5A)  # rows past n look like other keys
        c["key_scale"].fill_(3.0)
        for s in range(B * Hkv):
            o = s * t_cap
            if n:
                pa.pot_encode_keys(fmt, kk[s, :n].contiguous(), n, 1, 0,
                                   c["key_scale"].data_ptr() + 4 * o,
                                   c["codes_se"].data_ptr() + 32 * o,
                                   c["codes_m"].data_ptr() + 8 * o)
        if values == "int8":
            v = pa.alloc_value_cache_int8(B, Hkv, t_cap, DEV)
            v[1].fill_(-100)  # a stale exponent would be the minimum
            if n:
                pa.pot_store_values_int8(vv[:, :n].contiguous(), B * Hkv, n, t_cap, 0, *v)
        else:
            v = (pa.alloc_value_cache(B, Hkv, t_cap, DEV),)
            v[0].fill_(1000.0)
            if n:
                pa.pot_store_values(vv[:, :n].contiguous(), B * Hkv, n, t_cap, 0, *v)
        return c, v

    for T in (1, 2, 63, 64, 65, 128, 129, 257, 640, 1024, 1025):
        kn, vn = kk[:, T - 1].contiguous(), vv[:, T - 1].contiguous()
        dbg = pa.pot_debug()
        dbg.force_splits, dbg.force_wg_waves = 1, waves
        got, want = (torch.empty((B, Hq, 64), dtype=torch.float32, device=DEV) for _ in range(2))
        c, v = cache(T - 1)
        r, w = cache(T)
        a = (t_cap, d["kv_head_of_q"], B, Hq, Hkv, T)
        if values == "int8":
            pa.pot_append_decode_attention_v8(fmt, 0, q, kn, vn, c["codes_se"], c["codes_m"],
                                              c["key_scale"], *v, *a, got, ws, dbg=dbg)
            pa.pot_decode_attention_v8(fmt, 0, q, r["codes_se"], r["codes_m"], r["key_scale"], *w,
                                       *a, want, ws, dbg=dbg)
        else:
            pa.pot_append_decode_attention(fmt, q, kn, vn, c["codes_se"], c["codes_m"],
                                           c["key_scale"], *v, *a, got, ws, dbg=dbg)
            pa.pot_decode_attention(fmt, q, r["codes_se"], r["codes_m"], r["key_scale"], *w, *a,
                                    want, ws, dbg=dbg)
        torch.cuda.synchronize()
        assert torch.equal(got, want), (T, values, waves)
        for name in ("codes_se", "codes_m", "key_scale"):
            assert torch.equal(c[name], r[name]), (T, name)
        assert all(torch.equal(x, y) for x, y in zip(v, w)), T
