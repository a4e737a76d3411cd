"""GPU parity of launches that store their results with device scope: 8 MB and
more of output, four units and more per workgroup, and units too large for the
held piece.  One sequence is much longer than the others, so that its units are
cut over several ranges and merged through the workspace and from registers."""
import numpy as np
import pytest

from paper_2508_21706_amd import workloads as wl
from test_gpu_paged import check_paged
from test_gpu_parity import _custom, check_case
from test_gpu_tree import check_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,tree,page", [
    ("f16", 128, False, 0), ("bf16", 64, False, 0), ("f32", 128, False, 0),
    ("bf16", 128, True, 0), ("f32", 64, True, 0),
    ("f16", 64, False, 16), ("f32", 128, False, 64), ("bf16", 128, True, 8),
])
def test_device_scope_results(dtype, D, tree, page):
    g, Hkv = 4, 2
    B, C, grids = (90, 24, (40, 9)) if D == 128 else (132, 32, (60, 11))
    assert B * C * g * Hkv * D * 4 >= 8 << 20 and B * Hkv >= 4 * max(grids) and C * g > 32
    rng = np.random.default_rng([D, page, tree])
    ctx, chunk = rng.integers(0, 150, size=B), rng.integers(0, C + 1, size=B)
    ctx[B // 2], chunk[B // 2] = 2000, C
    inp = _custom(B, g * Hkv, Hkv, D, dtype, ctx.tolist(), chunk.tolist(), C)
    words = wl.tree_draft_masks(5, chunk, C) if tree else None
    for grid in grids:
        label = f"{dtype} D={D} tree={tree}"
        if page:
            check_paged(inp, dtype, page, label, grid_blocks=grid, words=words)
        elif tree:
            check_tree(inp, dtype, words, label, grid_blocks=grid)
        else:
            check_case(inp, dtype, label, grid_blocks=grid)
