"""Window attention of the draft: every share of a head between workgroups (up to 64 query heads of the call four, up to
128 two, more one) and both lengths of a round, windows around a round, one token to several rounds, against fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import ATOL, TORCH_DTYPE  # noqa: E402


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _step(dtype, d):
    """Tokens that a workgroup takes side by side."""
    return 16 * 64 * (8 if dtype == "bf16" else 4) // d


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 3, 1), (4, 16, 2), (5, 13, 1), (2, 64, 8), (3, 43, 1), (9, 24, 8)])
@pytest.mark.parametrize("layout", ["token", "pair"])
def test_shares_and_rounds(sp, dtype, d, B, Hq, Hkv, layout):
    import torch
    g = torch.Generator(device="cuda").manual_seed(B * Hq + d)
    rng = np.random.default_rng(Hq)
    step = _step(dtype, d)
    for window in (1, step - 1, 2 * step, 2 * step + 1, 8 * step + 3, 17 * step):
        n_text = [int(x) for x in rng.integers(1, window + 20, size=B)]
        n_text[-1] = window                              # one sequence with the whole window
        lens = [n + int(rng.integers(0, 50)) for n in n_text]
        cu = np.concatenate(([0], np.cumsum(lens))).astype(np.int32)
        ct = np.concatenate(([0], np.cumsum(n_text))).astype(np.int32)
        idx = [np.sort(rng.permutation(L)[:n]).astype(np.int32) for L, n in zip(lens, n_text)]
        q = torch.randn(B, Hq, d, generator=g, device="cuda").to(TORCH_DTYPE[dtype])
        kv = torch.randn(Hkv, int(cu[-1]), 2, d, generator=g, device="cuda").to(TORCH_DTYPE[dtype])
        k, v = kv[:, :, 0].permute(1, 0, 2), kv[:, :, 1].permute(1, 0, 2)
        if layout == "token":
            k, v = k.contiguous(), v.contiguous()
        out, lse = sp.draft_window_attn(q, k, v, cu, torch.from_numpy(np.concatenate(idx)).cuda(), ct, window)
        for b in range(B):
            at = torch.from_numpy(idx[b][-window:]).long().cuda() + int(cu[b])
            kk = k[at].double().repeat_interleave(Hq // Hkv, dim=1).permute(1, 0, 2)             # [Hq, n, d]
            vv = v[at].double().repeat_interleave(Hq // Hkv, dim=1).permute(1, 0, 2)
            s = (kk * q[b].double()[:, None]).sum(dim=2) / d ** 0.5
            ref = (torch.softmax(s, dim=1)[:, :, None] * vv).sum(dim=1)
            err = (out[b].double() - ref).abs().max() / max(1.0, float(ref.abs().max()))
            assert float(err) <= ATOL[dtype], (window, b, float(err))
            assert float((lse[b].double() - torch.logsumexp(s, dim=1)).abs().max()) <= 1e-4


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv", [(2, 6, 2), (3, 32, 4), (9, 24, 8)])
def test_an_infinite_value_in_the_last_token_stays_infinite(sp, dtype, d, B, Hq, Hkv):
    """The token that fills up a window's last round: with no weight there, and nothing of it in the other columns."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d)
    step = _step(dtype, d)
    for window in (1, 5, step + 1, 2 * step + 1, 9 * step - 1):
        n = window + 3
        q, k, v = (torch.randn(m, h, d, generator=g, device="cuda").to(TORCH_DTYPE[dtype]) for m, h in ((B, Hq), (B * n, Hkv), (B * n, Hkv)))
        last = n * torch.arange(1, B + 1, device="cuda") - 1
        v[last, 1, 7] = float("inf")
        at = np.arange(B + 1, dtype=np.int32) * n
        out, _ = sp.draft_window_attn(q, k, v, at, torch.arange(n, dtype=torch.int32, device="cuda").repeat(B), at, window)
        own = out[:, Hq // Hkv:2 * (Hq // Hkv), 7]
        assert torch.isposinf(own).all(), window
        own.zero_()
        assert torch.isfinite(out).all(), window
