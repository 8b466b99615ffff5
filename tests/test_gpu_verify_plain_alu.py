"""The plain-ALU verification kernels (K/V that span 2 GiB or more, scratch too small for the matrix-core
kernels' partials) over what the matrix-core kernels take otherwise: trees of several row blocks, one tree
per sequence, ragged batches, many splits; fp32 and heads of 64, against the oracle."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import TORCH_DTYPE, check_attn, dev, host  # noqa: E402


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("Hq,Hkv,lengths,n_q,nodes", [(16, 4, (300,), 5, 0), (28, 4, (257, 40), 0, 25), (4, 1, (2101,), 0, 60),
                                                      (8, 2, (700, 0, 3, 1290, 64), 0, 12), (8, 8, (1, 31, 33), 17, 0)])
def test_trees_batches_and_splits(sp, oracle, dtype, d, Hq, Hkv, lengths, n_q, nodes):
    import torch
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2, 1, 1)) if nodes else None
    cfg = wl.Config("P", dtype, Hq, Hkv, d, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=sum(lengths) + Hq, layouts=tuple(((wl.TEXT, n),) for n in lengths),
                       n_q=len(parent) if nodes else n_q, parent=parent)
    T, dt = len(c.k), TORCH_DTYPE[dtype]
    esize = torch.empty(0, dtype=dt).element_size()
    stride = -(-(1 << 31) // (T * esize)) // 512 * 512 + 512          # rows far enough apart to span 2 GiB
    buf = torch.empty(T * stride, dtype=dt, device="cuda").view(T, stride)
    at = Hkv * d
    k, v = buf[:, :at].view(T, Hkv, d), buf[:, at:2 * at].view(T, Hkv, d)
    k.copy_(dev(c.k, dtype))
    v.copy_(dev(c.v, dtype))
    q = dev(c.q, dtype)
    for par in [None] if parent is None else [dev(parent), dev(np.tile(parent, (len(lengths), 1)))]:
        out, lse = sp.verify_attn(q, k, v, c.cu_seqlens, par, c.n_q)
        ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
        check_attn(host(out), ref, dtype, f"{Hq}/{Hkv}/{d} {lengths}")
        assert np.abs(host(lse) - ref_lse).max() <= 2e-5          # fp32 throughout
    del buf, k, v
