"""Combine pass of sequences with many splits (1, 2, 4, 8 and 16 wavefronts that merge 16 each), with rows that leave groups of
four and 16-row tiles partly empty, and sequences of one length, whose place the kernels work out without a table, beside
ragged ones.  test_dispatch.py holds the bf16 cases against the library's launches."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import check_attn, dev, host, run_verify  # noqa: E402

# (query heads, KV heads, draft rows), rows of each sequence, most splits of a sequence in bf16 with heads of 128
CASES = [((8, 1, 8), (9001,), 141), ((5, 1, 3), (8100, 8100), 127), ((6, 2, 5), (8000,), 125), ((6, 2, 1), (4161,), 66),
         ((28, 4, 9), (4096,), 64), ((12, 4, 3), (2150,), 34), ((12, 4, 3), (1200,), 19), ((28, 4, 5), (2048, 2048), 32),
         ((4, 1, 7), (3000, 700, 40, 1500), 47), ((16, 4, 4), (1000,) * 8, 8), ((28, 4, 30), (5030,), 27),
         ((12, 4, 3), (600,), 10), ((28, 4, 60), (5030,), 16),
         ((64, 32, 4), (2011,), 8)]                     # fp32: 16 splits of 32 units


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_many_splits(oracle, dtype, d, case):
    import paper_2602_15318_amd as sp
    (Hq, Hkv, n_q), lens, _ = CASES[case]
    cfg = wl.Config("L", dtype, Hq, Hkv, d, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=case + d, layouts=tuple(((wl.TEXT, n - n_q),) for n in lens), n_q=n_q, parent=None)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, n_q)
    check_attn(out, ref, dtype, f"{CASES[case]}")
    assert np.abs(lse - ref_lse).max() <= (4e-3 if dtype == "bf16" else 2e-5)


@pytest.mark.parametrize("half", [0, 1])
def test_large_values_in_one_half_of_a_row(oracle, half):
    """fp16 partials carry a power of two per half of a row's columns: with values of 2^100 in one half, the other half's
    bits are those of a call without them, and the large half's those of small ones, shifted."""
    import paper_2602_15318_amd as sp
    cfg = wl.Config("L", "bf16", 28, 4, 128, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=3, layouts=(((wl.TEXT, 5000),),), n_q=5, parent=None)
    out, _ = run_verify(sp, c)
    cols = slice(64 * half, 64 * half + 64)
    c.v[..., cols] *= 2.0 ** 100
    big, _ = run_verify(sp, c)
    big[..., cols] *= 2.0 ** -100
    assert (big == out).all()


# KV heads, rows of each sequence: 4-row groups, 16-row tiles of four, two and one wavefronts
@pytest.mark.parametrize("Hkv,lens", [(1, (4500,)), (12, (3000, 3000)), (12, (1300,) * 4), (12, (1000, 900) * 4)])
@pytest.mark.parametrize("rows", [1, 4, 5, 13, 16, 17, 32, 33, 48, 63, 64, 65, 69, 81, 128, 130, 193])
def test_workgroups_with_and_without_rows(oracle, Hkv, lens, rows):
    """One draft row, `rows` heads per KV head: workgroups of the combine pass whose rows none, some or all exist.  Outputs and
    scratch are NaN beforehand: every output is written, by what the call itself wrote."""
    import torch

    import paper_2602_15318_amd as sp
    cfg = wl.Config("R", "bf16", Hkv * rows, Hkv, 128, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=rows, layouts=tuple(((wl.TEXT, n - 1),) for n in lens), n_q=1, parent=None)
    q, k, v = (dev(x, "bf16") for x in (c.q, c.k, c.v))
    ws = torch.full((sp.verify_attn_workspace_bytes(q, k, v, len(lens), 1, sum(lens)) // 4,), float("nan"), device="cuda")
    out, lse = sp.verify_attn(q, k, v, c.cu_seqlens, None, 1, out=torch.full_like(q, float("nan")), workspace=ws)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, 1)
    check_attn(host(out), ref, "bf16", f"{rows} rows, {lens}")
    assert np.abs(host(lse) - ref_lse).max() <= 4e-3


@pytest.mark.parametrize("splits", [29, 32])
def test_equal_sequences_by_proportion_and_alike(oracle, splits):
    """Eight sequences of 807 rows over 32 slots: scratch of 29 splits holds the plan by proportion, 32 are cut alike."""
    import torch

    import paper_2602_15318_amd as sp
    cfg = wl.Config("R", "bf16", 32, 8, 128, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=3, layouts=(((wl.TEXT, 802),),) * 8, n_q=5, parent=None)
    q, k, v = (dev(x, "bf16") for x in (c.q, c.k, c.v))
    ws = torch.full((splits * 8 * 64 * (4 * 64 + 12) // 4,), float("nan"), device="cuda")
    out, lse = sp.verify_attn(q, k, v, c.cu_seqlens, None, 5, workspace=ws)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, 5)
    check_attn(host(out), ref, "bf16", f"scratch of {splits} splits")
    assert np.abs(host(lse) - ref_lse).max() <= 4e-3
