"""Merge of the key splits by a unit's last workgroup (CU-wide workgroups, up to 32
splits; the combine kernel otherwise): whatever the workspace holds before a call, over one
workspace used by calls of different shapes, in replays of a captured call with
eager calls on the same workspace between them, and on two streams with a
workspace each. The order of the sums does not depend on which workgroup is
last, so repeated calls are bit-identical.
"""
import numpy as np
import pytest
import torch

import paper_2609_09208_amd as pa
from parity_util import DEV, assert_pot_parity
from workloads import make_decode_inputs, make_decode_inputs_device

pytestmark = pytest.mark.gpu


class Call:
    """A PoT-4 decode call on device buffers of its own."""

    def __init__(self, seed, B, Hq, Hkv, T):
        d = make_decode_inputs_device(seed, B, Hq, Hkv, T, DEV, t_cap=-(-T // 8) * 8)
        self.shape, self.t_cap, self.heads, self.q = (B, Hq, Hkv, T), d["t_cap"], d["kv_head_of_q"], d["q"]
        self.fmt = pa.make_format(0)
        self.c = pa.alloc_pot_cache(B, Hkv, self.t_cap, 0, DEV)
        n = B * Hkv * self.t_cap
        pa.pot_encode_keys(self.fmt, d["k"], n, 1, 0, self.c["key_scale"], self.c["codes_se"], None)
        self.v = pa.alloc_value_cache(B, Hkv, self.t_cap, DEV)
        pa.pot_store_values(d["v"], B * Hkv, self.t_cap, self.t_cap, 0, self.v)
        self.out = torch.zeros((B, Hq, 64), dtype=torch.float32, device=DEV)

    def workspace_bytes(self, splits=0):
        B, Hq, Hkv, T = self.shape
        return pa.pot_decode_workspace_bytes_for_splits(B, Hq, Hkv, T, splits)

    def run(self, ws, splits=0, stream=None):
        dbg = pa.pot_debug()
        dbg.force_splits = splits
        pa.pot_decode_attention(self.fmt, self.q, self.c["codes_se"], None, self.c["key_scale"],
                                self.v, self.t_cap, self.heads, *self.shape, self.out, ws, dbg=dbg,
                                stream=stream)
        return dbg.n_splits


@pytest.mark.parametrize("S", [2, 3, 16, 17, 31, 32, 33, 65])
@pytest.mark.parametrize("G", [1, 8])
def test_merge_of_s_splits(S, G):
    d = make_decode_inputs(300 + S, B=1, Hq=2 * G, Hkv=2, T=256 * S - 37)
    for waves in (16, 4):
        err, g = assert_pot_parity(d, force_splits=S, wg_waves=waves)
        assert g["n_splits"] == S
    print(f"S={S} G={G} O err {err:.2e}")


def test_any_workspace_contents():
    call = Call(11, 2, 16, 2, 4000)
    n = call.workspace_bytes()
    ws = pa.alloc_workspace(n, DEV)
    assert call.run(ws) > 1
    torch.cuda.synchronize()
    want = call.out.clone()
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    for fill in ("zeros", "ones", "random", "left", "left", "random"):
        if fill == "zeros":
            ws.zero_()
        elif fill == "ones":
            ws.fill_(255)
        elif fill == "random":
            ws.random_(0, 256, generator=g)
        call.out.zero_()
        call.run(ws)
        torch.cuda.synchronize()
        assert torch.equal(call.out, want), fill
    for _ in range(50):  # back to back, nothing between
        call.run(ws)
    torch.cuda.synchronize()
    assert torch.equal(call.out, want)


def test_one_workspace_for_calls_of_different_shapes():
    calls = [Call(20, 1, 32, 4, 2000), Call(21, 3, 16, 4, 3001), Call(22, 1, 8, 8, 5000)]
    ws = pa.alloc_workspace(max(c.workspace_bytes() for c in calls), DEV)
    wants = []
    for c in calls:
        assert c.run(pa.alloc_workspace(c.workspace_bytes(), DEV)) > 1
        torch.cuda.synchronize()
        wants.append(c.out.clone())
    for _ in range(5):
        for c in calls:
            c.run(ws)
        torch.cuda.synchronize()
        for c, w in zip(calls, wants):
            assert torch.equal(c.out, w)
            c.out.zero_()


def test_replays_with_eager_calls_between():
    a, b = Call(30, 2, 32, 4, 3000), Call(31, 1, 32, 4, 4096)
    ws = pa.alloc_workspace(max(a.workspace_bytes(), b.workspace_bytes()), DEV)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert a.run(ws) > 1 and b.run(ws) > 1
        torch.cuda.synchronize()
        wa, wb = a.out.clone(), b.out.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            a.run(ws)
            a.run(ws)  # the captured calls follow each other on one workspace
    for i in range(6):
        a.out.zero_()
        graph.replay()
        if i % 2:
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(a.out, wa), i
        b.out.zero_()
        b.run(ws)
        torch.cuda.synchronize()
        assert torch.equal(b.out, wb), i


def test_two_streams_with_a_workspace_each():
    calls = [Call(40, 4, 32, 4, 3000), Call(41, 4, 32, 4, 2500)]
    spaces = [pa.alloc_workspace(c.workspace_bytes(), DEV) for c in calls]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    wants = []
    for c, w in zip(calls, spaces):
        assert c.run(w) > 1
        torch.cuda.synchronize()
        wants.append(c.out.clone())
        c.out.zero_()
    torch.cuda.synchronize()
    for _ in range(20):
        for c, w, s in zip(calls, spaces, streams):
            c.run(w, stream=s)
    torch.cuda.synchronize()
    for c, w in zip(calls, wants):
        assert torch.equal(c.out, w)
        assert np.isfinite(c.out.cpu().numpy()).all()
