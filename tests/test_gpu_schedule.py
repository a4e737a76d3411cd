"""GPU parity where the tile schedule changes its form: batches of one and of
several sequences per lane with runs of empty ones, and launches whose total
cost could pass 31 bits, which are split by tile counts.  (The split itself, up
to the largest totals, is checked on the CPU in test_schedule.py.)"""
import numpy as np
import pytest
import torch

import paper_2508_21706_amd as pkg
from test_gpu_parity import _custom, check_case, compare, dev, nan_outputs, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 63, 64, 65, 129, 1024])
def test_sequences_per_lane(B):
    rng = np.random.default_rng(B)
    ctx = rng.integers(0, 400, size=B)
    chunk = rng.integers(1, 4, size=B)
    chunk[rng.random(B) < 0.4] = 0          # empty sequences, among them ...
    chunk[: B // 3], chunk[B - B // 5:] = 0, 0   # ... the first and the last of the batch
    chunk[B // 3] = 3
    inp = _custom(B, 4, 2, 64, "bf16", ctx.tolist(), chunk.tolist(), 3)
    for grid in (0, 3, 700):
        check_case(inp, "bf16", f"B={B}", grid_blocks=grid)


@pytest.mark.parametrize("B", [188, 190])
def test_total_cost_at_31_bits(B):
    """The kernel on both sides of the host's choice of the schedule's form: 16
    KV heads of up to 64768 tiles of 256 keys, at least 11 cost units each, stay
    below 2^31 with B = 188 and could pass it with B = 190.  The lengths are
    short (all sequences share one page of 65536 tokens), so this runs the
    form that counts tiles, not the totals that call for it."""
    d = dev()
    Hq = Hkv = 16
    D, C, ps, pages = 64, 2, 65536, 253
    g = torch.Generator(device=d).manual_seed(B)
    q = torch.randn((B, C, Hq, D), generator=g, device=d).to(torch.bfloat16)
    k = torch.randn((1, Hkv, ps, D), generator=g, device=d).to(torch.bfloat16)
    v = torch.randn((1, Hkv, ps, D), generator=g, device=d).to(torch.bfloat16)
    table = torch.zeros((B, pages), dtype=torch.int32, device=d)
    rng = np.random.default_rng(B)
    ctx, chunk = rng.integers(0, 900, size=B), rng.integers(0, C + 1, size=B)
    dctx, dchunk = (torch.from_numpy(a.astype(np.int32)).to(d) for a in (ctx, chunk))
    k64, v64 = k[0, :, :1024].double(), v[0, :, :1024].double()
    ref_o = torch.zeros((B, C, Hq, D), dtype=torch.float64, device=d)
    ref_l = torch.full((B, C, Hq), -np.inf, dtype=torch.float64, device=d)
    for b in range(B):
        for i in range(chunk[b]):
            T = int(ctx[b]) + i + 1
            s = (k64[:, :T] * q[b, i].double()[:, None]).sum(-1) * 0.125
            ref_l[b, i] = torch.logsumexp(s, -1)
            ref_o[b, i] = (torch.softmax(s, -1)[..., None] * v64[:, :T]).sum(1)
    for grid in (0, 7):
        note(f"case B={B} grid_blocks={grid}")
        out, lse = nan_outputs(B, C, Hq, D)
        pkg.verify_attn_paged(q, k, v, table, dctx, dchunk, 0.125, out=out, lse=lse, grid_blocks=grid)
        torch.cuda.synchronize()
        compare(out.cpu().double().numpy(), lse.cpu().double().numpy(), ref_o.cpu().numpy(), ref_l.cpu().numpy(),
                "bf16", f"B={B}")


def test_no_sequence_takes_a_step():
    d = dev()
    q = torch.zeros((70, 2, 4, 64), dtype=torch.bfloat16, device=d)
    k = torch.zeros((70, 2, 256, 64), dtype=torch.bfloat16, device=d)
    zeros = torch.zeros(70, dtype=torch.int32, device=d)
    for grid in (0, 1):
        out, lse = nan_outputs(70, 2, 4, 64)
        pkg.verify_attn(q, k, k, zeros + 9, zeros, 0.125, out=out, lse=lse, grid_blocks=grid)
        assert (out == 0).all() and (lse == -np.inf).all()


@pytest.mark.parametrize("grid", [4, 8, 9, 14, 15, 24, 40, 256])
@pytest.mark.parametrize("ctx", [[0, 61, 2000, 700], [1100, 3, 64, 128], [60, 61, 100, 20]])
def test_ranges_inside_units(ctx, grid):
    """Few units: ranges of a fixed number of tiles inside units, from the
    first grid with two workgroups per unit (8) over those where no small
    number leaves a range per workgroup to one with whole units."""
    inp = _custom(4, 2, 1, 128, "f32", ctx, [2, 1, 2, 2], 2)   # 64-key tiles
    check_case(inp, "f32", f"ctx={ctx}", grid_blocks=grid)
