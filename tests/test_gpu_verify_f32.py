"""Verification attention in fp32 on the matrix cores, against the oracle: row counts around the 16-, 64-
and 128-row tiles, contexts around the 32-token tile, ragged batches, one piece and split, and the scratch
rule that leaves a call with the plain-ALU kernels."""
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


def _case(Hq, Hkv, d, lengths, n_q, nodes, **kw):
    cfg = wl.Config("F32", "f32", Hq, Hkv, d, 1, None, 16, 4, False, 64, 128)
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2, 1, 1)) if nodes else None
    return wl.verify_case(cfg, seed=sum(lengths) + Hq, layouts=tuple(((wl.TEXT, n),) for n in lengths),
                          n_q=len(parent) if nodes else n_q, parent=parent, **kw)


def _run(sp, oracle, *args, **kw):
    c = _case(*args, **kw)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
    check_attn(out, ref, "f32", str(args))
    assert np.abs(lse - ref_lse).max() <= 2e-5, str(args)


@pytest.mark.parametrize("Hq,Hkv,d,n_q,nodes", [(4, 4, 64, 1, 0), (16, 4, 128, 4, 0), (28, 4, 128, 0, 10), (8, 2, 64, 17, 0),
                                                (28, 4, 64, 0, 25), (16, 2, 128, 0, 30), (32, 4, 128, 0, 60)])
@pytest.mark.parametrize("L", [0, 1, 31, 33, 130, 2001])
def test_rows_and_contexts(sp, oracle, Hq, Hkv, d, n_q, nodes, L):
    """1, 16, 68, 70, 175, 240 and 480 rows per KV head: blocks of 64 and of 128."""
    _run(sp, oracle, Hq, Hkv, d, (L,), n_q, nodes, peaked=L == 130)


@pytest.mark.parametrize("Hq,Hkv,d", [(28, 4, 128), (16, 4, 64)])
@pytest.mark.parametrize("lengths,n_q,nodes", [((9000, 300, 40, 2500), 5, 0), ((5000, 4300), 0, 30), ((26112,), 3, 0),
                                               (tuple(20 + 37 * i % 300 for i in range(64)), 2, 0)])
def test_batches_and_long_contexts(sp, oracle, Hq, Hkv, d, lengths, n_q, nodes):
    _run(sp, oracle, Hq, Hkv, d, lengths, n_q, nodes)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [63, 126, 1500])
def test_output_sums_are_short_chains(sp, d, L):
    """Equal probabilities (a zero query): the output is the mean of the values and its error that of the
    sums over the tokens.  A rounding at the sum's size is 2.6e-8 of it (0.3 * 2^-23 over the mantissa), a chain
    of n additions from zero sqrt(n / 2) of them: 16 tokens at a time, a chain over those (at most 16) and some
    six roundings where pieces are merged stay at sqrt(8 + 8 + 6) * 2.6e-8; one chain over 64 is at 1.5e-7."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(L)
    k, v = (torch.randn(L + 1, 16, d, generator=g, device="cuda") for _ in range(2))
    out, _ = sp.verify_attn(torch.zeros(1, 16, d, device="cuda"), k, v, np.array([0, L + 1], dtype=np.int32), None, 1)
    ref = v.double().mean(dim=0)
    assert float((out[0].double() - ref).norm() / ref.norm()) <= 1.25e-7


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_log_sum_exp_is_rounded_once_at_its_size(sp, dtype):
    """Root mean square error of values near 7.9: the last rounding 0.29 * 2^-21 = 1.4e-7, scores and row sums
    2.3e-7; a second rounding at 11.4 (log2 units), 0.29 * 2^-20 * ln 2, would make 3.3e-7 of it."""
    import torch
    L, n, Hq, Hkv, d = 1500, 60, 16, 4, 64
    g = torch.Generator(device="cuda").manual_seed(2)
    q, k, v = (torch.randn(t, h, d, generator=g, device="cuda").to(getattr(torch, dtype)) for t, h in ((n, Hq), (L + n, Hkv), (L + n, Hkv)))
    _, lse = sp.verify_attn(q, k, v, np.array([0, L + n], dtype=np.int32), None, n)
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for h in range(Hq):
        s = q[:, h].double() @ k[:, h // 4].double().t().contiguous() / 8.0
        s[:, L:][hidden] = -float("inf")
        err = lse[:, h].double() - torch.logsumexp(s, dim=1)
        lse[:, h] = err.float()
    assert float(lse.double().pow(2).mean().sqrt()) <= 3.0e-7


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [30, 97, 700, 3000])
def test_an_infinite_value_in_the_last_row_stays_infinite(sp, d, L):
    """The rows that fill up the last tile bring no 0 * inf."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda") for n, h in ((1, 8), (L + 1, 2), (L + 1, 2)))
    v[L, 1, 7] = float("inf")
    out, _ = sp.verify_attn(q, k, v, np.array([0, L + 1], dtype=np.int32), None, 1)
    assert torch.isposinf(out[0, 4:, 7]).all()
    out[0, 4:, 7] = 0
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("d", [64, 128])
def test_scratch_without_room_for_padded_rows_takes_the_plain_alu_kernels(sp, oracle, d):
    import torch
    c = _case(64, 64, d, tuple(200 + 5 * i % 50 for i in range(64)), 1, 0)
    q, k, v = dev(c.q, "f32"), dev(c.k, "f32"), dev(c.v, "f32")
    assert sp.verify_attn_workspace_bytes(q, k, v, 64, 1, int(c.cu_seqlens[-1])) > sp.STATIC_WS_BYTES
    ref, _ = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, 1)
    out = torch.empty_like(q)
    sp.verify_attn_static(q, k, v, c.cu_seqlens, None, 1, out)
    check_attn(host(out), ref, "f32", "static scratch")
    small = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    out2, _ = sp.verify_attn(q, k, v, c.cu_seqlens, None, 1, workspace=small)
    assert torch.equal(out, out2)
    out3, _ = sp.verify_attn(q, k, v, c.cu_seqlens, None, 1)
    check_attn(host(out3), ref, "f32", "matrix cores")
