"""The shift-accumulate scores on the matrix cores at the ends of their range.

The scores are formed as 7 + k ternary sums scaled by powers of two, in fp32
matrix instructions over q^ split as 16 hi + lo. They have to be the exact
integers: every partial sum is an integer (in units of 2^(F - 6)) of magnitude
at most 64 * 128 * (2^(k+1) - 1) * 64 <= 16 252 928 < 2^24 at k = 4. These rows
reach the largest sums of either sign, and put a single least significant unit
beside them; q^ = 120 .. 127 has hi = 8 and a negative lo.
"""
import numpy as np
import pytest

from parity_util import assert_pot_parity
from workloads import make_decode_inputs

pytestmark = pytest.mark.gpu


def extreme_rows(rng, rows, k):
    """Keys for a caller scale of 1: magnitude 4 saturates at the top code,
    2^-6 (1 + 2^-k) is the smallest magnitude with its lowest bit set."""
    low = 2.0 ** -6 * (1 + (2.0 ** -k if k else 0))
    out = np.empty((rows, 64), np.float32)
    for r in range(rows):
        kind = r % 8
        sign = np.ones(64, np.float32)
        if kind in (1, 5):
            sign = -sign
        elif kind in (2, 6):
            sign[1::2] = -1
        elif kind in (3, 7):
            sign = rng.choice([-1.0, 1.0], 64).astype(np.float32)
        mag = np.full(64, 4.0, np.float32)
        if kind >= 4:
            mag[rng.integers(64)] = low  # one unit beside the largest sum
            mag[rng.integers(64)] = 0.0
        out[r] = sign * mag
    return out


@pytest.mark.parametrize("F", [6, 7, 12])
@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])
def test_scores_at_the_ends_of_the_range(k, F):
    rng = np.random.default_rng(100 + k)
    G = (8, 4, 2, 1, 8)[k]
    T = 200
    d = make_decode_inputs(7, B=1, Hq=G, Hkv=1, T=T)
    keys = extreme_rows(rng, d["t_cap"], k)
    d["k_bits"] = keys.astype(np.float16).view(np.uint16).reshape(d["k_bits"].shape)
    # q^: +127 everywhere, -127 everywhere, signs of the alternating rows, and 120 .. 127
    q = np.full((8, 64), 1.0, np.float32)
    q[1] = -1.0
    q[2, 1::2] = -1.0
    q[3] = np.where(np.arange(64) % 2, 120.0 / 127, 1.0)
    q[4:] = rng.uniform(-1, 1, (4, 64))
    q[4:, 0] = 1.0
    d["q"] = np.ascontiguousarray(q[:G].reshape(1, G, 64)) * 1e-3
    err, g = assert_pot_parity(d, mant_bits=k, frac_bits=F,
                               key_scale=np.ones(d["t_cap"], np.float32))
    print(f"k={k} F={F} max |score| {np.abs(g['scores']).max()} O err {err:.2e}")
