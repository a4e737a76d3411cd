"""GPU parity where inputs hold infinities and NaN: they reach the rows that
see them, and no row of another sequence or KV head, wherever the schedule
puts tiles."""
import numpy as np
import pytest
import torch

import paper_2508_21706_amd as pkg
from oracle import verify_attn_ref
from paper_2508_21706_amd import workloads as wl
from test_gpu_parity import _custom, compare, dev, nan_outputs, note, run_gpu, to_dev

pytestmark = pytest.mark.gpu

INF = {"bf16": np.uint16(0x7f80), "f16": np.uint16(0x7c00), "f32": np.float32(np.inf)}
NAN = {"bf16": np.uint16(0x7fc0), "f16": np.uint16(0x7e00), "f32": np.float32(np.nan)}


def run_paged(inp, dtype, page, grid):
    nan = {"bf16": wl.BF16_NAN, "f16": wl.F16_NAN, "f32": np.float32(np.nan)}[dtype]
    kp, table = wl.paginate(inp["k_cache"], page, 3, nan)
    vp, _ = wl.paginate(inp["v_cache"], page, 3, nan)
    i32 = [torch.from_numpy(np.asarray(a, np.int32)).to(dev()) for a in (table, inp["ctx_lens"], inp["chunk_lens"])]
    out, lse = nan_outputs(*inp["q"].shape)
    pkg.verify_attn_paged(to_dev(inp["q"], dtype), to_dev(kp, dtype), to_dev(vp, dtype), *i32, inp["scale"], out=out,
                          lse=lse, grid_blocks=grid)
    torch.cuda.synchronize()
    return out.cpu().double().numpy(), lse.cpu().double().numpy()


@pytest.mark.parametrize("dtype,D,page", [("bf16", 128, 0), ("f16", 64, 0), ("f32", 128, 0), ("f32", 64, 0),
                                          ("f16", 128, 16), ("f32", 64, 8)])
@pytest.mark.parametrize("C", [2, 8, 40])   # one, two and more row blocks
def test_units_do_not_reach_each_other(C, dtype, D, page):
    """Every key, value and query of two sequences, and the keys and values of
    one KV head of a third, are Inf or NaN; the tiles of the other units take
    over their LDS stages, full and partial ones, and give what they give
    alone."""
    ctx = [1500, 3, 40, 700, 77, 130, 1, 15]
    chunk = [C, 1, C, C, C - 1, C, 1, C]
    inp = _custom(len(ctx), 6, 2, D, dtype, ctx, chunk, C)
    ref_o, ref_l = verify_attn_ref(inp["q"], inp["k_cache"], inp["v_cache"], inp["ctx_lens"], inp["chunk_lens"],
                                   inp["scale"], dtype)
    for a in [inp[name][b] for name in ("q", "k_cache", "v_cache") for b in (0, 3)] + [inp["k_cache"][5, 0],
                                                                                       inp["v_cache"][5, 0]]:
        a[..., ::2] = INF[dtype]
        a[..., 1::2] = NAN[dtype]
    ok = [b for b in range(len(ctx)) if b not in (0, 3, 5)]
    for grid in (1, 2, 3, 7, 0):
        note(f"case C={C} {dtype} D={D} page={page} grid_blocks={grid}")
        o, s = run_paged(inp, dtype, page, grid) if page else run_gpu(inp, dtype, grid)
        compare(o[ok], s[ok], ref_o[ok], ref_l[ok], dtype, f"grid={grid}")
        compare(o[5, :, 3:], s[5, :, 3:], ref_o[5, :, 3:], ref_l[5, :, 3:], dtype, f"grid={grid}, second KV head")


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
