"""The kernels that take eight rows or tokens per wave, at the edges of a group:
the INT8 value store over ranges that start and end inside a group, over more
sequences than one grid dimension holds and over NaN, infinite and zero tokens;
the INT8 key encoder over row counts beside a multiple of eight, with a row
stride; the PoT key encoder likewise, plain and rotated (by butterflies and, 16
rows per wave, on the matrix cores), over
values that fall on both of the rotation's paths, and with caller scales that put
the ratios one ulp below, at and above every cut point.
Bytes and scales are exact against the oracle; nothing else is written.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2609_09208_amd as pa
from parity_util import DEV, gpu_encode, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,n_tok,t0,t_cap", [(1, 1, 0, 8), (3, 1, 7, 16), (2, 9, 6, 24),
                                                  (5, 16, 8, 32), (2, 23, 5, 40), (4, 777, 3, 784),
                                                  (33000, 1, 2, 8),
                                                  # over 2048 tokens: eight tokens per wave
                                                  (256, 8, 8, 16), (257, 8, 8, 16), (300, 9, 6, 24),
                                                  (130, 16, 8, 32), (129, 23, 5, 40), (700, 3, 7, 16),
                                                  (1025, 2, 6, 8), (33000, 2, 3, 8), (1, 4099, 5, 4104)])
def test_store_int8_ranges(n_seq, n_tok, t0, t_cap):
    rng = np.random.default_rng(n_seq + 10 * n_tok + t0)
    v = (rng.standard_normal((n_seq, n_tok, 64)) * 2.0 ** rng.integers(-12, 9, (n_seq, n_tok, 1)))
    v = v.astype(np.float16)
    v[rng.random((n_seq, n_tok)) < 0.1] = 0.0
    vu = torch.full((n_seq, t_cap, 64), 77, dtype=torch.uint8, device=DEV)
    ve = torch.full((n_seq, t_cap), 55, dtype=torch.int8, device=DEV)
    pa.pot_store_values_int8(to_dev(v), n_seq, n_tok, t_cap, t0, vu, ve)
    torch.cuda.synchronize()
    vh, g = oracle.quantize_values(v.view(np.uint16).reshape(-1, 64))
    want_u = np.full((n_seq, t_cap, 64), 77, np.uint8)
    want_u[:, t0:t0 + n_tok] = (vh.reshape(n_seq, n_tok, 64).astype(np.int16) + 128)
    want_e = np.full((n_seq, t_cap), 55, np.int8)
    want_e[:, t0:t0 + n_tok] = g.reshape(n_seq, n_tok)
    got = vu.cpu().numpy().reshape(n_seq, t_cap // 8, 64, 8).transpose(0, 1, 3, 2)
    assert np.array_equal(got.reshape(n_seq, t_cap, 64), want_u)
    assert np.array_equal(ve.cpu().numpy(), want_e)


def test_store_int8_tokens_alone_and_in_a_group():
    # NaN, infinities and mixed signs: what a token becomes depends on nothing but itself
    # (one-token calls take a wave per token, the whole range of 129 sequences the group
    # stores, a range that starts and ends inside groups the partial ones)
    v = np.zeros((1, 16, 64), np.float16)
    v[0, 1] = np.nan
    v[0, 2, ::3] = np.nan
    v[0, 2, 1::3] = 3.25
    v[0, 3, 5] = 65504.0
    v[0, 4] = -(2.0 ** -24)
    v[0, 5:] = np.random.default_rng(3).standard_normal((11, 64)).astype(np.float16)
    n = 300
    v = np.repeat(v, n, axis=0)
    u1, e1 = pa.alloc_value_cache_int8(n, 1, 16, DEV)
    u2, e2 = pa.alloc_value_cache_int8(1, 1, 16, DEV)
    u3, e3 = pa.alloc_value_cache_int8(n, 1, 16, DEV)
    src = to_dev(v)
    pa.pot_store_values_int8(src, n, 16, 16, 0, u1, e1)
    for t in range(16):
        pa.pot_store_values_int8(src[0, t].contiguous(), 1, 1, 16, t, u2, e2)
    pa.pot_store_values_int8(src[:, 3:13].contiguous(), n, 10, 16, 3, u3, e3)
    torch.cuda.synchronize()
    assert torch.equal(u1, u2.expand_as(u1)) and torch.equal(e1, e2.expand_as(e1))
    byte = lambda u: u.view(-1, 2, 64, 8).transpose(2, 3).reshape(-1, 16, 64)  # [seq][token][dim]
    assert torch.equal(byte(u3)[:, 3:13], byte(u1)[:, 3:13]) and torch.equal(e3[:, 0, 3:13], e1[:, 0, 3:13])
    assert not byte(u3)[:, :3].any() and not byte(u3)[:, 13:].any() and not e3[:, 0, 13:].any()


@pytest.mark.parametrize("had", [False, True])
@pytest.mark.parametrize("n,stride", [(1, 1), (7, 3), (8, 1), (9, 2), (33, 5), (4099, 1)])
def test_int8_encode_row_counts(n, stride, had):
    rng = np.random.default_rng(n)
    k = (rng.standard_normal((n, 64)) * 2.0 ** rng.integers(-10, 10, (n, 1))).astype(np.float16)
    k[rng.random(n) < 0.05] = 0.0
    codes = torch.full((n * stride, 64), 99, dtype=torch.int8, device=DEV)
    sc = torch.full((n * stride,), -5.0, dtype=torch.float32, device=DEV)
    pa.pot_int8_encode_keys(to_dev(k), n, stride, int(had), sc, codes)
    torch.cuda.synchronize()
    oc, osc = oracle.int8_encode_keys(k.view(np.uint16), hadamard=had)
    want = np.full((n * stride, 64), 99, np.int8)
    want[::stride][:n] = oc
    want_s = np.full(n * stride, -5.0, np.float32)
    want_s[::stride][:n] = osc
    assert np.array_equal(codes.cpu().numpy(), want)
    assert np.array_equal(sc.cpu().numpy().view(np.uint32), want_s.view(np.uint32))


def pot_rows(n, had):
    """Rows over the whole fp16 range, some all zero, tiny, subnormal or constant (the
    rotation then leaves one element); for the rotation, which is exact on the matrix cores
    up to 4096, rows at and above that bound beside others; NaN and infinities."""
    rng = np.random.default_rng(n + 1000 * had)
    k = rng.standard_normal((n, 64)) * 2.0 ** rng.integers(-26, 9, (n, 1))
    k *= 2.0 ** rng.integers(-9, 2, (n, 64))
    k = np.clip(k, -4096, 4096).astype(np.float16)
    pick = rng.random(n)
    k[pick < 0.05] = 0.0
    k[(pick > 0.1) & (pick < 0.15)] = -3.25
    if n >= 16:
        k[3, 5], k[3, 9], k[3, 11] = 4096.0, 2.0 ** -24, 15.992
    if n >= 33:  # the second group of 16 takes the butterflies
        k[17, 1], k[18, 2], k[19, 3], k[20, 4] = 4098.0, 65504.0, np.inf, np.nan
        k[21] = np.nan
        k[22, 0::2], k[22, 1::2] = 65504.0, -65504.0
    return k


@pytest.mark.parametrize("had", [False, True])
@pytest.mark.parametrize("mant_bits", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n,stride", [(1, 1), (7, 3), (15, 1), (16, 2), (17, 1), (33, 5),
                                      (4099, 1)])
def test_pot_encode_row_counts(n, stride, mant_bits, had):
    check_pot_encode(n, stride, mant_bits, had)


# rotated on the matrix cores, 16 rows per wave (butterflies up to 24576 rows)
@pytest.mark.parametrize("mant_bits", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n,stride", [(24576, 1), (24577, 1), (24583, 3), (24591, 1), (24592, 2),
                                      (24593, 1), (24609, 1)])
def test_pot_encode_rotated_on_the_matrix_cores(n, stride, mant_bits):
    check_pot_encode(n, stride, mant_bits, True)


def check_pot_encode(n, stride, mant_bits, had):
    k = pot_rows(n, had)
    se = torch.full((n * stride, 32), 99, dtype=torch.uint8, device=DEV)
    cm = torch.full((n * stride, 8 * max(mant_bits, 1)), 98, dtype=torch.uint8, device=DEV)
    sc = torch.full((n * stride,), -5.0, dtype=torch.float32, device=DEV)
    fmt = pa.make_format(mant_bits=mant_bits, hadamard=had)
    pa.pot_encode_keys(fmt, to_dev(k), n, stride, 0, sc, se, cm if mant_bits else None)
    torch.cuda.synchronize()
    ose, ocm, osc = oracle.encode_keys(k.view(np.uint16), mant_bits, hadamard=had)
    for got, ref, fill in ((se, ose, 99), (cm, ocm if mant_bits else None, 98)):
        want = np.full(got.shape, fill, np.uint8)
        if ref is not None:
            want[::stride][:n] = ref
        assert np.array_equal(got.cpu().numpy(), want)
    want_s = np.full(n * stride, -5.0, np.float32)
    want_s[::stride][:n] = osc
    assert np.array_equal(sc.cpu().numpy().view(np.uint32), want_s.view(np.uint32))


def cut_points(k):
    """The fp32 cut points between neighbouring grid values, and the zero cut: the largest fp32
    below sqrt((n + i)(n + i + 1)) / n * 2^-e (n = 2^k) and below sqrt(2) 2^-7."""
    n = 1 << k
    # below sqrt(num / den^2) in [1, 2), rounded down to 24 bits; never a whole root
    root = lambda num, den: math.ldexp(math.isqrt((num << 46) // den ** 2), -23)
    cuts = [root((n + i) * (n + i + 1), n) for i in range(n)]
    return ([np.float32(c * 2.0 ** -e) for c in cuts for e in range(0, 8)]
            + [np.float32(root(2, 1) * 2.0 ** -7)])


def ulps(x, d):
    return (np.float32(x).view(np.int32) + np.int32(d)).view(np.float32)


@pytest.mark.parametrize("path", ["plain", "butterflies", "matrix cores"])
@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])
def test_ratios_beside_every_cut_point(k, path):
    # a row with one element x (rotated: x / 8 times a row of the Hadamard matrix) and a scale s
    # such that RN(x / s) is the cut, its neighbours and theirs
    rng = np.random.default_rng(40 + k)
    rows, scales = [], []
    for cut in cut_points(k):
        seen = set()
        for mant in (1.0, 1.3125, 1.9990234375, 1.5 + 2.0 ** -10):
            x = np.float32(mant * 2.0 ** rng.integers(-3, 4))
            for d in range(-6, 7):
                s = ulps(np.float32(x / cut), d)
                u = np.float32(x / s)
                off = int(u.view(np.int32)) - int(cut.view(np.int32))
                if abs(off) <= 2:
                    seen.add(off)
                    m, sign = rng.integers(64), rng.choice([-1.0, 1.0])
                    if path == "plain":
                        row = np.zeros(64, np.float16)
                        row[m] = sign * x
                    else:                # H row m times x / 8: (H r / 8)_m = 64 x / 64
                        row = np.array([sign * x / 8 * (-1) ** bin(m & j).count("1")
                                        for j in range(64)], np.float16)
                    rows.append(row)
                    scales.append(s)
        assert {-1, 0, 1} <= seen, (k, float(cut), seen)
    rows, scales = np.stack(rows), np.array(scales, np.float32)
    n = 24700 if path == "matrix cores" else len(rows)
    reps = -(-n // len(rows))
    rows, scales = np.tile(rows, (reps, 1)), np.tile(scales, reps)
    assert (len(rows) > 24576) == (path == "matrix cores")
    had = path != "plain"
    se, cm, _ = gpu_encode(rows.view(np.uint16), k, had, scales)
    ose, ocm, _ = oracle.encode_keys(rows.view(np.uint16), k, hadamard=had, key_scale=scales)
    assert np.array_equal(se, ose)
    if k:
        assert np.array_equal(cm, ocm)
