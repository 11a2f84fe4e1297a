"""The softmax denominator and the value sums at the ends of the weights' range.

Keys whose codes are all +1 (e = 0) and a query of ones give the score 64 s q / 8 of a
caller's row scale s, so the scales set every weight.
"""
import numpy as np
import pytest
import torch

import paper_2609_09208_amd as pa
from parity_util import DEV, store_values, to_dev

pytestmark = pytest.mark.gpu

Q = 1.0                                     # every query element: q^ = 127, Delta = 1 / 127
X_PER_S = 64 * Q / 8 / np.log(2.0)          # log2-domain score of a key with scale 1


def decode(scales, v_bits, waves, negative=None):
    """O of one sequence of such keys (codes -1 where negative), eight query heads, one split."""
    T = scales.size
    cap = -(-T // 8) * 8
    codes = np.zeros((cap, 32), np.uint8)
    if negative is not None:
        codes[:T][negative] = 0x88
    se = to_dev(codes)
    sc = np.zeros(cap, np.float32)
    sc[:T] = scales
    v = store_values(v_bits, 1, 1, cap)
    q = torch.full((1, 8, 64), Q, dtype=torch.float32, device=DEV)
    out = torch.empty((1, 8, 64), dtype=torch.float32, device=DEV)
    ws = pa.alloc_workspace(pa.pot_decode_workspace_bytes_for_splits(1, 8, 1, T, 1), DEV)
    dbg = pa.pot_debug()
    dbg.force_splits, dbg.force_wg_waves = 1, waves
    pa.pot_decode_attention(pa.make_format(0), q, se, None, to_dev(sc), v, cap, np.zeros(8, np.int32),
                            1, 8, 1, T, out, ws, dbg=dbg)
    torch.cuda.synchronize()
    return out.cpu().numpy()[0]


@pytest.mark.parametrize("waves", [4, 16])
def test_constant_values_come_back(waves):
    # every wave meets a large weight, 2^12 as it is formed, in its first tile and then only
    # weights of 2^-18.3, which its fp32 sums next to the large one cannot take up: numerator
    # and denominator have to lose the same ones. O / v is then 1 but for the merge of at most
    # 16 waves and a division, whose roundings (2^-24 each) may differ: below 2^-19. Summing
    # the denominator lane by lane instead makes O smaller by half of the small weights' share,
    # T / (2 waves) 2^-30.3: 4e-6 at 16 waves.
    T = 1 << 18
    scales = np.full(T, (40 - 12 - 18.3) / X_PER_S)
    scales[:waves * 64:64] = 39.99 / X_PER_S
    v = np.broadcast_to(2.0 ** (np.arange(64) % 8 - 4), (T, 64)).astype(np.float16)
    out = decode(scales, np.ascontiguousarray(v).view(np.uint16), waves)
    rel = np.abs(out / v[0].astype(np.float64) - 1).max()
    print(f"waves={waves} |O / v - 1| {rel:.2e}")
    assert rel <= 2.0 ** -19


@pytest.mark.parametrize("waves", [4, 16])
def test_scores_at_minus_two_to_the_31(waves):
    # -2^31 is its own ceiling and the integer maximum's "none yet". A wave whose first tile
    # holds only such scores and that meets a higher one later has to drop their weights.
    step = np.float32(Q) / np.float32(127)
    c = np.float32(np.float32(step * np.float32(1.44269502162933349609375)) * np.float32(2.0 ** -10))
    acc = np.float32(-64 * 127 * 128)
    s = np.float32(2.0 ** 31 / (64 * 127 * 128 * float(c)))
    near = (s.view(np.int32) + np.arange(-8, 9)).astype(np.int32).view(np.float32)
    x = (acc * near).astype(np.float32) * c
    s = near[x == np.float32(-2.0 ** 31)][0]
    T = 64 * waves * 2
    scales = np.full(T, s, np.float32)
    best = 64 * waves + 7                    # wave 0's second tile
    scales[best] = 3.0 / X_PER_S
    v = np.random.default_rng(0).standard_normal((T, 64)).astype(np.float16)
    out = decode(scales, v.view(np.uint16), waves, negative=np.ones(T, bool))
    assert np.abs(out - v[best].astype(np.float32)).max() <= 1e-6
