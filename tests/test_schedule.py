"""The kernel's tile schedule, compiled for the host, against a model in
unbounded integers: the ranges partition the tiles at the model's costs, none
is empty, and every shared unit's first and last owner are the ranges that hold
its ends.  Up to totals just below 2^31 in cost and 2^30 in tiles."""
import bisect
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2508_21706_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("schedule") / "schedule_host.so")
    res = subprocess.run([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                          "-I" + os.path.join(build.HERE, "csrc"), os.path.join(HERE, "schedule_host.hip"), "-o", out],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return ctypes.CDLL(out)


def check(host, g, Hkv, C_max, P, flat, tile, ctx, chunk):
    B = len(ctx)
    T = np.asarray(ctx, np.int64) + np.asarray(chunk, np.int64)
    seqs = (T.astype(np.uint32) << np.uint32(8)) | np.asarray(chunk, np.uint32)
    head = (ctypes.c_int64 * 5)()
    rows = np.zeros((P, 11), np.int32)
    host.host_schedule(g, Hkv, C_max, P, flat, tile, B, seqs.ctypes.data_as(ctypes.c_void_p), head,
                       rows.ctypes.data_as(ctypes.c_void_p))
    Pe, whole = head[0], head[1]

    # the model: per sequence its tiles n, a tile's cost w, a unit's start S and
    # end E, and the tiles and the cost before it
    n = [int(-(-t // tile)) if c else 0 for t, c in zip(T.tolist(), chunk)]
    count = bool(whole or flat)
    w = [1 if count else 10 + -(-int(c) * g // 16) for c in chunk]
    S = [0 if count else 3] * B
    E = [0 if count else 9 if int(c) * g <= 32 else 6 for c in chunk]
    U = [-(-a // whole) * whole if whole else a * x + s + e if a else 0 for a, x, s, e in zip(n, w, S, E)]
    t0, c0 = [0], [0]
    for b in range(B):
        t0.append(t0[-1] + Hkv * n[b])
        c0.append(c0[-1] + Hkv * U[b])
    N, Wt = t0[-1], c0[-1]
    assert head[2] == Wt and Wt < 1 << 31
    if N == 0:
        assert Pe == 0
        return whole
    assert 1 <= Pe <= P and head[3] * Pe + head[4] == Wt and 0 <= head[4] < Pe
    bound = [q * head[3] + min(q, head[4]) for q in range(Pe + 1)]

    def place(t):      # sequence, KV head and index of tile t, and its start cost
        b = bisect.bisect_right(t0, t) - 1
        kvh, j = divmod(t - t0[b], n[b])
        return b, kvh, j, c0[b] + kvh * U[b] + (S[b] + j * w[b] if j else 0)

    rows = rows[:Pe].tolist()
    starts = [r[0] for r in rows]
    assert starts[0] == 0 and rows[-1][1] == N
    for q, (g0, g1, b, kvh, j, bl, kvl, qf0, ql0, qf1, ql1) in enumerate(rows):
        assert g0 < g1 and (q + 1 == Pe or g1 == rows[q + 1][0])
        assert place(g0)[:3] == (b, kvh, j) and place(g1 - 1)[:2] == (bl, kvl)
        assert bound[q] <= place(g0)[3] and place(g1 - 1)[3] < bound[q + 1]
        for bb, kk, qf, ql in ((b, kvh, qf0, ql0), (bl, kvl, qf1, ql1)):
            unit = t0[bb] + kk * n[bb]
            assert qf == bisect.bisect_right(starts, unit) - 1
            assert ql == bisect.bisect_right(starts, unit + n[bb] - 1) - 1
        if whole:
            assert (b, kvh) == (bl, kvl) and g1 - g0 <= whole
    if whole > 4:
        # no range costs over 3.5 of its tiles more than the average one, which
        # counts for three quarters, and the average over all workgroups
        w = [10 + -(-int(c) * g // 16) for c in chunk]
        E = [12 if int(c) * g <= 32 else 9 for c in chunk]
        total = sum(Hkv * (a * x + e) for a, x, e in zip(n, w, E) if a)
        most = max((min(a, whole) - 3.5) * x + e for a, x, e in zip(n, w, E) if a)
        assert most <= 0.75 * total / Pe + 0.25 * total / P + 1e-6
    return whole
    assert 1 <= Pe <= P and head[3] * Pe + head[4] == Wt and 0 <= head[4] < Pe
    bound = [q * head[3] + min(q, head[4]) for q in range(Pe + 1)]

    def place(t):      # sequence, KV head and index of tile t, and its start cost
        b = bisect.bisect_right(t0, t) - 1
        kvh, j = divmod(t - t0[b], n[b])
        return b, kvh, j, c0[b] + kvh * U[b] + (S[b] + j * w[b] if j else 0)

    rows = rows[:Pe].tolist()
    starts = [r[0] for r in rows]
    assert starts[0] == 0 and rows[-1][1] == N
    for q, (g0, g1, b, kvh, j, bl, kvl, qf0, ql0, qf1, ql1) in enumerate(rows):
        assert g0 < g1 and (q + 1 == Pe or g1 == rows[q + 1][0])
        assert place(g0)[:3] == (b, kvh, j) and place(g1 - 1)[:2] == (bl, kvl)
        assert bound[q] <= place(g0)[3] and place(g1 - 1)[3] < bound[q + 1]
        for bb, kk, qf, ql in ((b, kvh, qf0, ql0), (bl, kvl, qf1, ql1)):
            unit = t0[bb] + kk * n[bb]
            assert qf == bisect.bisect_right(starts, unit) - 1
            assert ql == bisect.bisect_right(starts, unit + n[bb] - 1) - 1
        if whole:
            assert (b, kvh) == (bl, kvl) and g1 - g0 <= whole
    if whole > 4:
        # no range costs over 3.5 of its tiles more than the average one
        w = [10 + -(-int(c) * g // 16) for c in chunk]
        E = [12 if int(c) * g <= 32 else 9 for c in chunk]
        mean = sum(Hkv * (a * x + e) for a, x, e in zip(n, w, E) if a) / Pe
        assert max((min(a, whole) - 3.5) * x + e for a, x, e in zip(n, w, E) if a) <= mean
    return whole


def test_random_launches(host):
    rng = np.random.default_rng(7)
    forms = {0: 0, 1: 0}
    for _ in range(1500):
        B = int(rng.choice([1, 2, 5, 11, 63, 64, 65, 200, 1024]))
        g, Hkv = int(rng.choice([1, 3, 4, 7, 16])), int(rng.choice([1, 2, 8, 32]))
        C_max = int(rng.integers(1, 128 // g + 1))
        chunk = rng.integers(0 if rng.random() < 0.5 else 1, C_max + 1, size=B)
        ctx = rng.integers(0, int(np.exp(rng.uniform(1, 10.5))), size=B)
        P = int(rng.choice([1, 2, 7, 64, 256, 300, 2048]))
        flat = int(rng.random() < 0.2)
        whole = check(host, g, Hkv, C_max, P, flat, int(rng.choice([64, 128, 256])), ctx, chunk)
        forms[int(whole > 0)] += 1
    assert min(forms.values()) > 50   # both forms occur


@pytest.mark.parametrize("P", [7, 256, 2048])
@pytest.mark.parametrize("ragged", [False, True])
def test_largest_totals(host, P, ragged):
    """16 KV heads of 64768 tiles: the last batch whose costs are added up,
    the first that counts tiles, and the largest."""
    tiles = 64768
    B0 = next(b for b in range(1, 1025) if host.host_counts_tiles(1, 16, 2, b, tiles))
    assert (B0 - 1) * 16 * (tiles * 11 + 12) < 1 << 31 <= B0 * 16 * (tiles * 11 + 12)
    rng = np.random.default_rng(P)
    for B, flat in ((B0 - 1, 0), (B0, 1), (1024, 1)):
        ctx = np.full(B, 256 * tiles - 2)
        chunk = np.full(B, 2)
        if ragged:
            ctx -= rng.integers(0, 3000, size=B)
            chunk[rng.random(B) < 0.01] = 0
        check(host, 1, 16, 2, P, flat, 256, ctx, chunk)


def test_counts_tiles_only_past_31_bits(host):
    for g, Hkv, C_max, tiles in ((4, 8, 5, 4096), (7, 4, 16, 60000), (1, 128, 128, 8000), (16, 1, 8, 65536)):
        unit = tiles * (10 + -(-C_max * g // 16)) + 12
        for B in (1, 64, 500, 1024):
            assert host.host_counts_tiles(g, Hkv, C_max, B, tiles) == int(B * Hkv * unit >= 1 << 31)


@pytest.mark.parametrize("Hkv,g,C,tile,ctx,chunk,even", [
    (8, 4, 5, 128, [3800] * 12, [5] * 12, True),       # 192 equal ranges
    (8, 4, 5, 128, [300] * 16, [5] * 16, True),        # whole units
    (4, 7, 16, 128, [3800] * 24, [16] + [1] * 23, False),                        # rows differ
    (2, 4, 4, 64, [3000 - 50 * i for i in range(56)], [4] * 56, False),          # lengths differ
])
def test_uneven_ranges_fall_back_to_equal_cost(host, Hkv, g, C, tile, ctx, chunk, even):
    whole = check(host, g, Hkv, C, 256, 0, tile, ctx, chunk)
    assert (whole > 0) == even
