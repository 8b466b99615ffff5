"""Verification attention of sequences short enough to be one piece (the partial pass writes the result
itself): both head sizes, chains and trees, row counts around the 16- and 64-row tiles, lengths around
the tile, the step and the line of the rule; and the two passes asked for one by one, which never take
that way."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import check_attn, dev, host, run_verify  # noqa: E402


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


@pytest.mark.parametrize("Hq,Hkv,d,n_q,nodes", [(4, 4, 128, 1, 0), (28, 4, 128, 5, 0), (28, 4, 128, 0, 10), (28, 4, 128, 0, 25),
                                                (32, 8, 64, 3, 0), (28, 4, 64, 0, 30), (16, 16, 128, 9, 0)])
@pytest.mark.parametrize("lengths", [(0,), (31,), (60, 65), (144,), (150, 3, 200), (500,) * 16, (511, 300) * 8])
def test_short_sequences(sp, oracle, Hq, Hkv, d, n_q, nodes, lengths):
    import torch
    cfg = wl.Config("S", "bf16", Hq, Hkv, d, 1, None, 16, 4, False, 64, 128)
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2)) if nodes else None
    c = wl.verify_case(cfg, seed=sum(lengths) + Hq, layouts=tuple(((wl.TEXT, n),) for n in lengths),
                       n_q=len(parent) if nodes else n_q, parent=parent)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
    what = f"{Hq}/{Hkv}/{d} {lengths} n_q={c.n_q}"
    check_attn(out, ref, "bf16", what)
    assert np.abs(lse - ref_lse).max() <= (4e-3 if d == 128 else 2e-5), what     # as in the split passes
    q, k, v = dev(c.q, "bf16"), dev(c.k, "bf16"), dev(c.v, "bf16")
    par = None if parent is None else dev(parent)
    ws = torch.empty(sp.verify_attn_workspace_bytes(q, k, v, len(lengths), c.n_q, len(c.k)), dtype=torch.uint8, device="cuda")
    out2 = torch.zeros_like(q)
    for p in (1, 2):
        sp.verify_attn(q, k, v, c.cu_seqlens, par, c.n_q, out=out2, workspace=ws, passes=p)
    check_attn(host(out2), ref, "bf16", what + ", pass by pass")
