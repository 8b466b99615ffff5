"""Verification attention of trees over long splits (blocks of 128 rows, heads of 128).  Several blocks from 14 steps of
64 tokens on: the two token streams of a workgroup run half a step apart; one block, or shorter splits: in step.  Splits
of an odd number of 32-token tiles (one stream has a tile less than the other) and of an even one, last splits that end
in, at and just behind a tile or hold one row, row blocks in which some wavefronts have no rows; batches on both grids,
with short sequences and splits without a row beside long ones, a tree per sequence, every layout of K and V.
test_dispatch.py holds the cases against the library's plan: the instance, the splits, the rows of the last one."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import check_attn, dev, host, run_verify  # noqa: E402

# (query heads, KV heads, nodes), splits, rows of a split, rows that the last split is short
ONE_SEQUENCE = (
    [((28, 4, 56), 16, 864, short) for short in (0, 1, 31, 33, 64, 511)]        # four blocks, 27 tiles
    + [((28, 4, 30), 32, 896, short) for short in (0, 1, 33, 895)]              # two blocks, 28 tiles
    + [((16, 2, 50), 32, 864, short) for short in (0, 500, 832, 863)]           # four blocks
    + [((28, 4, 30), 32, 672, short) for short in (0, 607)]                     # in step: short splits
    + [((28, 4, 16), 64, 672, short) for short in (0, 33)]                      # in step: one block
)
# (query heads, KV heads, nodes), rows of each sequence, splits of each, the flat grid
BATCHES = [
    ((28, 4, 30), (13824, 13824), (16, 16), False),
    ((28, 4, 30), (22131, 1085, 64), (30, 1, 1), True),          # the long sequence's last split has no row
    ((28, 4, 60), (14000, 13900), (8, 8), False),
    ((16, 2, 50), (26500, 51, 900, 82), (30, 1, 1, 1), True),    # one context row; draft rows behind a tile's end
    ((32, 8, 30), (9000, 14000, 7000), (10, 15, 7), True),       # in step: one block
]


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _config(Hq, Hkv):
    return wl.Config("L", "bf16", Hq, Hkv, 128, 1, None, 16, 4, False, 64, 128)


def _case(heads, total, seed):
    Hq, Hkv, nodes = heads
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2, 1, 1))
    return wl.verify_case(_config(Hq, Hkv), seed=seed, layouts=(((wl.TEXT, total - nodes),),), n_q=nodes, parent=parent)


@pytest.mark.parametrize("heads,splits,piece,short", ONE_SEQUENCE)
def test_split_ends(sp, oracle, heads, splits, piece, short):
    c = _case(heads, splits * piece - short, seed=heads[2] + short)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
    check_attn(out, ref, "bf16", f"{heads}, {splits} x {piece}, {short} short")
    assert np.abs(lse - ref_lse).max() <= 4e-3


def _laid_out(x, y, layout):
    """K and V [T, Hkv, d] on the device as views of [T, Hkv, d], [Hkv, T, d] or [Hkv, T, 2, d]."""
    import torch
    k, v = dev(x, "bf16"), dev(y, "bf16")
    if layout == "token":
        return k, v
    if layout == "head":
        return tuple(t.permute(1, 0, 2).contiguous().permute(1, 0, 2) for t in (k, v))
    kv = torch.stack([k.permute(1, 0, 2), v.permute(1, 0, 2)], dim=2).contiguous()
    return kv[:, :, 0].permute(1, 0, 2), kv[:, :, 1].permute(1, 0, 2)


@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_batches_of_own_trees(sp, oracle, batch):
    import torch
    (Hq, Hkv, nodes), lens, _, _ = BATCHES[batch]
    trees = np.stack([wl.pruned_tree(40 + b, nodes, (4, 3, 2, 2, 1, 1)) for b in range(len(lens))])
    c = wl.verify_case(_config(Hq, Hkv), seed=batch, layouts=tuple(((wl.TEXT, n - nodes),) for n in lens), n_q=nodes,
                       parent=trees)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, trees, nodes)
    first = None
    for layout in ("token", "head", "pair"):
        k, v = _laid_out(c.k, c.v, layout)
        out, lse = sp.verify_attn(dev(c.q, "bf16"), k, v, c.cu_seqlens, dev(trees), nodes)
        torch.cuda.synchronize()
        check_attn(host(out), ref, "bf16", f"{lens} {layout}")
        assert np.abs(host(lse) - ref_lse).max() <= 4e-3
        first = out if first is None else first
        assert torch.equal(out, first)                  # the layout moves no sum


def test_infinite_value_at_the_end_of_a_split(sp):
    heads, piece = (28, 4, 56), 864
    c = _case(heads, 16 * piece, seed=5)
    c.v[piece - 1, :, 0] = np.inf                       # last row of the first split, visible to every draft row
    out, _ = run_verify(sp, c)
    assert np.all(np.isposinf(out[:, :, 0]))            # and no 0 * inf from rows behind the split's end
    assert np.all(np.isfinite(out[:, :, 1:]))
