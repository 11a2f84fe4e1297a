"""Host model of the decode kernel's buffer windows (no GPU).

The decode kernel reads each tile's cache rows through a raw buffer resource
whose base is the tile's first row and whose record count ends at the key
range's last row (codes, mantissa planes, comparator keys) or at the end of its
last 8-key group (scales, values, exponents: rows that exist, since t_cap is a
multiple of 8). The lane's whole offset is the vector operand, which is what the
hardware compares with the record count (the scalar offset is not part of that
check, so the kernel passes 0 there). A load whose offset is at or past the
count returns zeros and touches no memory.

The model replays, for every split, wave and tile (also the prefetch of the
next tile, clamped to the last, and any order in which waves claim tiles: a
tile's loads depend on the tile alone), the offsets each lane uses for every
stream, and checks at ragged T = t_cap rounded up to 8 (the tightest legal cache):
* every performed access lies inside the sequence's rows [0, t_cap);
* a multi-byte load is either wholly in range or wholly out;
* every byte that a matrix operand needs arrives in the lane and register that
  needs it: half `half` of key KEY(lane, set) of the tile for the key streams,
  the 8 keys of the lane's group for scales, exponents and value fragments.
The offsets mirror those of decode_kernel.hpp (load_keys, load_scales,
load_values_buf); the needs are stated from the operand layout.
"""
import pytest

TILE = 256          # keys of the split unit
WTILE = 64          # keys per wave tile
LANES = range(64)


def plan(T, S):
    tiles = (T + TILE - 1) // TILE
    S = max(1, min(S, tiles))
    split_len = (tiles + S - 1) // S * TILE
    return (T + split_len - 1) // split_len, split_len


# What a lane has to hold. Set s: row i = lane % 16 of the key operand is key 8 (i / 4) + 4 s +
# i % 4 of the tile in blocks 0-1, plus 32 in blocks 2-3; odd blocks hold the second half.
def key_of(lane, s):
    return 8 * (lane % 16 // 4) + 4 * s + lane % 4 + 32 * (lane // 32)


def half_of(lane):
    return lane // 16 % 2


def group_of(lane):                 # first of the 8 keys whose scores the lane gets
    return 32 * (lane // 8 % 2) + 8 * (lane // 16)


# ---- loads: (register name, [(lane's offset, bytes)]), as the kernel issues them ------------
def key_offset(l):
    i, blk = l & 15, l >> 4
    return 32 * (blk >> 1) + 8 * (i >> 2) + (i & 3)


def code_loads():
    return [(("c", s), lambda l, s=s: key_offset(l) * 32 + 16 * (l >> 4 & 1) + 128 * s, 16)
            for s in range(2)]


def comparator_loads(row):
    n = row // 32
    return [(("k", s, c), lambda l, s=s, c=c: key_offset(l) * row + 16 * n * (l >> 4 & 1)
             + 4 * s * row + 16 * c, 16) for s in range(2) for c in range(n)]


def plane_loads(K):
    out = []
    for s in range(2):
        if K == 4:
            out.append((("quad", s), lambda l, s=s: key_offset(l) * 32 + 16 * (l >> 4 & 1)
                        + 128 * s, 16))
            continue
        if K >= 2:
            out.append((("pair", s), lambda l, s=s: key_offset(l) * 8 * K + 8 * (l >> 4 & 1)
                        + 32 * K * s, 8))
        if K & 1:
            out.append((("last", s), lambda l, s=s: key_offset(l) * 8 * K + 8 * (K - 1)
                        + 4 * (l >> 4 & 1) + 32 * K * s, 4))
    return out


def scale_loads():
    return [(("s", i), lambda l, i=i: (32 * (l >> 3 & 1) + 8 * (l >> 4)) * 4 + 16 * i, 16)
            for i in range(2)]


def value_loads(v8):
    gb, frag = (512, 8) if v8 else (1024, 16)
    return [(("f", kb, nb), lambda l, kb=kb, nb=nb: (l >> 4) * gb + (l & 15) * frag + kb * 4 * gb
             + nb * 16 * frag, frag) for kb in range(2) for nb in range(4)]


def exp_loads():
    return [(("g",), lambda l: 32 * ((l & 15) >> 3) + 8 * (l >> 4), 8)]


# ---- needs: the bytes of the tile (from its first row) that a register has to hold ----------
def plane_dword(K, key, plane, half):
    at = key * 8 * K + 8 * plane + 4 * half
    return [at, at + 1, at + 2, at + 3]


def plane_need(K):
    """Register contents after the exchange of the block pairs (v_permlane16_swap: odd blocks of
    the first register with even blocks of the second), from what each lane loaded: dword d of
    the quad, or of the pair, is plane_order[block parity][d] of half d_half[d]."""
    def check(loaded, lane, s):
        other = lane ^ 16           # the same row of the neighbouring block
        assert key_of(other, s) == key_of(lane, s) and half_of(other) != half_of(lane)
        lo, hi = (lane, other) if not lane & 16 else (other, lane)   # even, odd block
        mine = lane >> 4 & 1
        planes = {}
        regs = {l: [loaded[(("quad" if K == 4 else "pair"), s)][l][4 * d:4 * d + 4]
                    for d in range(4 if K == 4 else 2)] for l in (lo, hi)} if K >= 2 else {}
        for a in range(0, 4 if K == 4 else 2 if K >= 2 else 0, 2):
            # swap(x = reg a, y = reg a + 1): x's odd block <-> y's even block
            x = {lo: regs[lo][a], hi: regs[lo][a + 1]}
            y = {lo: regs[hi][a], hi: regs[hi][a + 1]}
            first, second = (a // 2, 2 + a // 2) if K == 4 else (0, 1)
            planes[first], planes[second] = x[lane], y[lane]
        if K & 1:
            planes[K - 1] = loaded[("last", s)][lane]
        assert sorted(planes) == list(range(K))
        for p in range(K):
            assert planes[p] == plane_dword(K, key_of(lane, s), p, mine), (K, s, lane, p)
    return check


def check_operands(K, key_row, v8):
    """Which byte of the tile every lane gets in every register (whole tiles)."""
    def load(loads):
        return {name: {l: list(range(off(l), off(l) + size)) for l in LANES}
                for name, off, size in loads}
    if key_row == 32:
        got = load(code_loads())
        for s in range(2):
            for l in LANES:
                at = key_of(l, s) * 32 + 16 * half_of(l)
                assert got[("c", s)][l] == list(range(at, at + 16))
        if K:
            got, check = load(plane_loads(K)), plane_need(K)
            for s in range(2):
                for l in LANES:
                    check(got, l, s)
    else:
        got, n = load(comparator_loads(key_row)), key_row // 32
        for s in range(2):
            for l in LANES:
                at = key_of(l, s) * key_row + key_row // 2 * half_of(l)
                assert sum((got[("k", s, c)][l] for c in range(n)), []) == list(
                    range(at, at + key_row // 2))
    got = load(scale_loads())
    for l in LANES:
        assert got[("s", 0)][l] + got[("s", 1)][l] == list(
            range(4 * group_of(l), 4 * group_of(l) + 32))
    # value fragments: 8 keys 32 kb + 8 (l / 16) .. of dim 16 nb + l % 16, in the interleaved cache
    frag = 8 if v8 else 16
    got = load(value_loads(v8))
    for kb in range(2):
        for nb in range(4):
            for l in LANES:
                at = ((32 * kb + 8 * (l // 16)) // 8 * 64 + 16 * nb + l % 16) * frag
                assert got[("f", kb, nb)][l] == list(range(at, at + frag))
    if v8:
        got = load(exp_loads())
        for l in LANES:
            assert got[("g",)][l] == list(range(group_of(l), group_of(l) + 8))


def streams(K, key_row, v8):
    """(name, row bytes, limit kind, loads)."""
    out = [("keys", key_row, "t", code_loads() if key_row == 32 else comparator_loads(key_row))]
    if key_row != 128:
        out.append(("scales", 4, "v", scale_loads()))
    if K:
        out.append(("planes", 8 * K, "t", plane_loads(K)))
    out.append(("values", 64 if v8 else 128, "v", value_loads(v8)))
    if v8:
        out.append(("exps", 1, "v", exp_loads()))
    return out


def check_windows(T, t_cap, S, K, key_row, v8):
    n_splits, split_len = plan(T, S)
    for split in range(n_splits):
        t_begin = split * split_len
        t_end = min(T, t_begin + split_len)
        v_end = ((t_end - 1) & ~7) + 8
        assert v_end <= t_cap                 # t_cap is a multiple of 8
        n_tiles = (t_end - t_begin + WTILE - 1) // WTILE
        for waves in (4, 12, 16):             # the tiles some wave loads, prefetches among them
            first = range(min(waves, n_tiles))
            tiles = {t for w in first for j in range(w, n_tiles, waves)
                     for t in (j, min(j + waves, n_tiles - 1))}
            assert tiles == set(range(n_tiles))
        for name, rb, kind, loads in streams(K, key_row, v8):
            lim = t_end if kind == "t" else v_end
            read = bytearray((lim - t_begin) * rb)
            for j in range(n_tiles):
                t0 = t_begin + WTILE * j
                assert t0 < lim
                base, n_rec = t0 * rb, (lim - t0) * rb
                for reg, off, size in loads:
                    for lane in LANES:
                        o = off(lane)
                        if o >= n_rec:
                            continue              # returns zeros, no access
                        assert o + size <= n_rec, (name, reg, lane, o, size, n_rec)
                        assert 0 <= base + o and base + o + size <= t_cap * rb, (name, reg, lane)
                        at = base + o - t_begin * rb
                        read[at:at + size] = b"\x01" * size
            assert all(read), (name, read.index(0))   # every byte of the range arrives


# K (None: a comparator), key row bytes, INT8 values
ENGINES = [(0, 32, False), (1, 32, False), (2, 32, False), (3, 32, False), (4, 32, False),
           (0, 32, True), (1, 32, True), (2, 32, True), (3, 32, True), (4, 32, True),
           (0, 64, False), (0, 128, False)]


@pytest.mark.parametrize("K,key_row,v8", ENGINES)
def test_every_register_gets_its_key(K, key_row, v8):
    check_operands(K, key_row, v8)


@pytest.mark.parametrize("T,S", [(4104, 1), (4104, 3), (4104, 16), (64, 1), (65, 1), (63, 1),
                                 (1000, 2), (8, 1), (1, 1), (7, 1), (257, 2), (3001, 12),
                                 (32768, 4), (33016, 5)])
@pytest.mark.parametrize("K,key_row,v8", ENGINES)
def test_buffer_windows_stay_inside_the_sequence(T, S, K, key_row, v8):
    t_cap = (T + 7) // 8 * 8                    # the tightest legal capacity
    check_windows(T, t_cap, S, K, key_row, v8)
