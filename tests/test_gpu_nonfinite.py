"""GPU parity where inputs hold infinities and NaN: they reach the rows that
see them, and no row of another sequence, wherever the schedule puts tiles."""
import numpy as np
import pytest

from oracle import verify_attn_ref
from test_gpu_parity import _custom, compare, note, run_gpu

pytestmark = pytest.mark.gpu

INF = {"bf16": np.uint16(0x7f80), "f16": np.uint16(0x7c00), "f32": np.float32(np.inf)}
NAN = {"bf16": np.uint16(0x7fc0), "f16": np.uint16(0x7e00), "f32": np.float32(np.nan)}


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("C", [2, 8, 40])   # one, two and more row blocks
def test_sequences_do_not_reach_each_other(C, dtype, D):
    """Every key, value and query of two sequences is Inf or NaN; the tiles
    of the others take over their LDS stages, full and partial ones, and
    give what they give alone."""
    ctx = [1500, 3, 40, 700, 77, 130, 1, 15]
    chunk = [C, 1, C, C, C - 1, C, 1, C]
    inp = _custom(len(ctx), 6, 2, D, dtype, ctx, chunk, C)
    ref_o, ref_l = verify_attn_ref(inp["q"], inp["k_cache"], inp["v_cache"], inp["ctx_lens"], inp["chunk_lens"],
                                   inp["scale"], dtype)
    for b in (0, 3):
        for name in ("q", "k_cache", "v_cache"):
            inp[name][b, ..., ::2] = INF[dtype]
            inp[name][b, ..., 1::2] = NAN[dtype]
    ok = [b for b in range(len(ctx)) if b not in (0, 3)]
    for grid in (1, 2, 3, 7, 0):
        note(f"case C={C} {dtype} D={D} grid_blocks={grid}")
        o, s = run_gpu(inp, dtype, grid)
        compare(o[ok], s[ok], ref_o[ok], ref_l[ok], dtype, f"grid={grid}")


def test_piece_without_visible_keys():
    """A unit's last tile holds draft tokens only: rows before them see no key
    of it.  As a piece of its own it weighs nothing there, whatever the values
    of its tokens are.  (64-key tiles; with ranges of two tiles, units of seven
    and three tiles leave the last one alone.)"""
    C, ctx = 100, [7 * 64 - 100, 3 * 64 - 100, 7 * 64 - 100]
    inp = _custom(3, 1, 1, 128, "f32", ctx, [C] * 3, C)
    ref_o, ref_l = verify_attn_ref(inp["q"], inp["k_cache"], inp["v_cache"], inp["ctx_lens"], inp["chunk_lens"],
                                   inp["scale"], "f32")
    for b, l in enumerate(ctx):
        inp["v_cache"][b, :, l + C - 8:l + C] = np.inf
    rows = C - 64   # of every sequence: no key of the last tile is visible
    note("case last tile invisible")
    o, s = run_gpu(inp, "f32", 0)
    compare(o[:, :rows], s[:, :rows], ref_o[:, :rows], ref_l[:, :rows], "f32", "last tile invisible")
