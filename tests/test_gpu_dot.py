"""GPU parity of the decoded-weight score path (pot_dot_decode_attention).

Codes are decoded to fp16 weights sigma (1 + j / 2^k) 2^(-8-e) and scored by
fp16 matrix instructions, exactly. The int32 scores are exactly those of eq. (sac)
with eq. (mant), so the bar is pot_decode_attention's: codes, q^, Delta,
scores and integer maxima bit-exact against the oracle, O within 2e-3, over
every mantissa width and head-group size, ragged tails, head-room, Hadamard,
forced splits and degenerate rows.
"""
import numpy as np
import pytest

import oracle
from parity_util import assert_pot_parity, gpu_encode, gpu_pot_decode
from workloads import make_decode_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (8, 4), (8, 2), (32, 4)])
def test_dot_every_mantissa_width_and_group(k, Hq, Hkv):
    d = make_decode_inputs(300 + 10 * k + Hq // Hkv, B=2, Hq=Hq, Hkv=Hkv, T=700)
    assert_pot_parity(d, mant_bits=k, engine="dot")


def test_dot_tinyllama_layer_t32768_potm1():
    d = make_decode_inputs(320, B=1, Hq=32, Hkv=4, T=32768)
    err, g = assert_pot_parity(d, mant_bits=1, engine="dot")
    print(f"dot PoT-M1 T=32768 splits={g['n_splits']} O err {err:.3e}")


def test_dot_batch8_hadamard_potm4_t2048():
    d = make_decode_inputs(321, B=8, Hq=32, Hkv=4, T=2048)
    err, g = assert_pot_parity(d, mant_bits=4, hadamard=True, engine="dot")
    print(f"dot Hadamard PoT-M4 B=8 T=2048 splits={g['n_splits']} O err {err:.3e}")


@pytest.mark.parametrize("T,t_cap", [(1, 8), (63, 64), (257, 320), (4099, 4104)])
@pytest.mark.parametrize("k", [1, 4])
def test_dot_ragged(T, t_cap, k):
    d = make_decode_inputs(330 + T + k, B=2, Hq=8, Hkv=2, T=T, t_cap=t_cap)
    assert_pot_parity(d, mant_bits=k, engine="dot")


@pytest.mark.parametrize("F", [6, 12])
def test_dot_head_room(F):
    d = make_decode_inputs(340 + F, B=1, Hq=8, Hkv=1, T=600)
    assert_pot_parity(d, mant_bits=2, frac_bits=F, engine="dot")


def test_dot_forced_splits_and_degenerate_rows():
    d = make_decode_inputs(350, B=2, Hq=8, Hkv=1, T=2000)
    k = d["k_bits"].reshape(2, 1, -1, 64)
    k[0, 0, 5] = 0          # all-zero key row (s = 0, all zero codes)
    k[1, 0, :50] = 0
    d["q"][1, 3] = 0.0      # zero query (q^ = 0, Delta = 0)
    assert_pot_parity(d, mant_bits=3, force_splits=7, engine="dot")


@pytest.mark.parametrize("k", [1, 4])
def test_dot_scores_equal_shift_path(k):
    d = make_decode_inputs(360 + k, B=2, Hq=32, Hkv=4, T=1500)
    rows = d["k_bits"].reshape(-1, 64)
    se, cm, sc = gpu_encode(rows, k)
    a = gpu_pot_decode(d, se, cm, sc, mant_bits=k, engine="sac")
    b = gpu_pot_decode(d, se, cm, sc, mant_bits=k, engine="dot")
    assert np.array_equal(a["scores"], b["scores"])
    assert np.array_equal(a["m_final"], b["m_final"])
    assert float(np.abs(a["out"] - b["out"]).max()) <= 1e-5


@pytest.mark.parametrize("k,waves", [(1, 16), (2, 16), (3, 16), (4, 16), (1, 4), (4, 4)])
def test_dot_zero_codes_ignore_their_planes(k, waves):
    # e = 7 is zero whatever its sign bit and mantissa bits hold (the encoder writes zeros
    # there, another producer of the cache may not): in every place of a row, all at once too
    d = make_decode_inputs(370 + k, B=1, Hq=8, Hkv=1, T=300)
    se, cm, sc = gpu_encode(d["k_bits"].reshape(-1, 64), k)
    rng = np.random.default_rng(k)
    nib = np.stack([se & 15, se >> 4], axis=-1).reshape(-1, 64)
    zero = rng.random(nib.shape) < 0.2
    zero[:64] = np.eye(64, dtype=bool)
    zero[64] = True
    nib = np.where(zero, 7 | (nib & 8), nib).astype(np.uint8)
    se = nib[:, 0::2] | (nib[:, 1::2] << 4)
    bits = np.unpackbits(cm.reshape(-1, k, 8), axis=-1, bitorder="little") | zero[:, None, :]
    cm = np.packbits(bits, axis=-1, bitorder="little").reshape(-1, 8 * k)
    want = oracle.pot_decode(d["q"], se, cm, sc, d["v_bits"], d["t_cap"], d["kv_head_of_q"], 1, 8, 1,
                             300, mant_bits=k)
    for engine in ("dot", "sac"):
        g = gpu_pot_decode(d, se, cm, sc, mant_bits=k, engine=engine, force_splits=1,
                           wg_waves=4 if waves == 4 else (16 if engine == "dot" or k <= 2 else 12))
        assert np.array_equal(g["scores"], want["scores"]), engine
        assert np.array_equal(g["m_final"], want["m_final"]), engine
        assert float(np.abs(g["out"] - want["out"]).max()) <= 2e-3, engine
