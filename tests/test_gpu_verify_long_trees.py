"""Verification attention of trees over long splits (blocks of 128 rows, heads of 128, more than ten steps of 64 tokens
per split), whose two token streams run half a step apart, and in step for one block over token-major K/V.  Splits of an odd number of 32-token tiles
(one stream has a tile less than the other), last splits that end in, at and just behind a tile, row blocks
in which some wavefronts have no rows."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import check_attn, run_verify  # noqa: E402

PIECE = 672                    # 21 tiles


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _case(nodes, total, seed):
    cfg = wl.Config("L", "bf16", 28, 4, 128, 1, None, 16, 4, False, 64, 128)
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2, 1, 1))
    return wl.verify_case(cfg, seed=seed, layouts=(((wl.TEXT, total - len(parent)),),), n_q=len(parent), parent=parent)


@pytest.mark.parametrize("nodes,splits", [(56, 16), (30, 32), (16, 64)])        # 392, 210, 112 rows: 4, 2, 1 blocks
@pytest.mark.parametrize("short", [0, 1, 31, 33, 64, 607])
def test_split_ends(sp, oracle, nodes, splits, short):
    if splits == 64 and short not in (0, 33):
        pytest.skip("two ends are enough for the longest context")
    c = _case(nodes, splits * PIECE - short, seed=nodes + short)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
    check_attn(out, ref, "bf16", f"{nodes} nodes, {short} short")
    assert np.abs(lse - ref_lse).max() <= 4e-3


def test_infinite_value_at_the_end_of_a_split(sp):
    c = _case(56, 16 * PIECE, seed=5)
    c.v[PIECE - 1, :, 0] = np.inf                       # last row of the first split, visible to every draft row
    out, _ = run_verify(sp, c)
    assert np.all(np.isposinf(out[:, :, 0]))            # and no 0 * inf from rows behind the split's end
    assert np.all(np.isfinite(out[:, :, 1:]))
