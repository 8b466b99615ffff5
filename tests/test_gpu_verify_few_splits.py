"""Combine pass of batches whose sequences have few splits: at most four (one wavefront takes them all) and at most eight
(two), beside sequences of one split and draft rows that leave 16-row tiles without a row.  test_dispatch.py holds the
bf16 cases against the library's launches."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import check_attn, run_verify  # noqa: E402

# (query heads, KV heads, draft rows), rows of each sequence, most splits of a sequence in bf16
CASES = [((16, 8, 5), (1500, 1460, 1400, 1490, 1300, 1444, 1333, 1222, 1111), 4),
         ((16, 8, 20), (1200, 900, 65, 1200, 1190, 1111, 1001, 800, 1134), 4),
         ((32, 4, 6), (2400, 2300, 2200, 2100, 2000, 1900, 1800, 1700), 8),
         ((32, 4, 17), (1900, 70, 1880, 300, 1800, 1890, 1850, 1700, 1750, 1600), 7),
         ((12, 4, 30), (1600, 1500, 1400, 1300, 1250, 1200, 1100, 1000), 8)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_few_splits(oracle, dtype, d, case):
    import paper_2602_15318_amd as sp
    (Hq, Hkv, n_q), lens, _ = CASES[case]
    cfg = wl.Config("F", dtype, Hq, Hkv, d, 1, None, 16, 4, False, 64, 128)
    c = wl.verify_case(cfg, seed=case + d, layouts=tuple(((wl.TEXT, n - n_q),) for n in lens), n_q=n_q, parent=None)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, n_q)
    check_attn(out, ref, dtype, f"{CASES[case]}")
    assert np.abs(lse - ref_lse).max() <= (4e-3 if dtype == "bf16" else 2e-5)
    # f32 has twice the splits: both halves of them run what bf16 runs
    if dtype == "f32":
        half = lens[:len(lens) // 2]
        lens2 = lens + half + half
        c = wl.verify_case(cfg, seed=case, layouts=tuple(((wl.TEXT, n - n_q),) for n in lens2), n_q=n_q, parent=None)
        out, _ = run_verify(sp, c)
        check_attn(out, oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, n_q)[0], dtype, f"{lens2}")
