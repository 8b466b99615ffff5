"""Draft tree kernels at the edges of their sizes: top-k for vocabularies around every number of logits a
thread owns, with ties; selection and expansion of pools around the 64 entries of a register, up to the
largest, with tied, zero and infinite scores."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


@pytest.mark.parametrize("V", [16, 64, 65, 16384, 16385, 65536, 65537, 152064, 163840, 163841, 262144])
@pytest.mark.parametrize("k", [1, 13, 16])
def test_topk_vocabularies(sp, V, k):
    """Whole-number logits (one-hot hidden rows pick a column of W), so ties are exact: the lowest ids."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(V + k)
    W = torch.randint(-8, 9, (V, 8), generator=g, device="cuda").float()
    W[torch.randint(0, V, (5,), generator=g, device="cuda"), 0] = 20.0
    W[:, 1] = 3.0                                            # every logit tied
    hid = torch.eye(8, device="cuda")[:3].contiguous()
    ids, logp = sp.draft_topk(hid, W, k)
    logits = W[:, :3].t().double()
    order = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k]
    assert torch.equal(ids.long(), order)
    ref = torch.log_softmax(logits, dim=1).gather(1, order)
    assert float((logp.double() - ref).abs().max()) <= 1e-5


def _select_reference(tok, par, score, total):
    order = sorted(range(len(tok)), key=lambda i: (-score[i], i))[:min(total, len(tok))]
    kept = sorted(order)
    new = {i: j for j, i in enumerate(kept)}
    return [new.get(int(par[i]), -1) if par[i] >= 0 else -1 for i in kept], [int(tok[i]) for i in kept], kept


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 300, 689, 1024, 1025, 2047, 2048])
@pytest.mark.parametrize("total", [1, 30, 64])
def test_selection_sizes(sp, n, total):
    import torch
    from paper_2602_15318_amd import binding as b
    rng = np.random.default_rng(n + total)
    for kind in range(4):
        score = -rng.random(n).astype(np.float32) * 9.0
        if kind == 1:
            score = -rng.integers(0, 4, n).astype(np.float32)            # many ties, zeros among them
            score[::3] *= -1.0 if n < 3 else 1.0
        elif kind == 2:
            score[:] = -1.5                                              # all tied
        elif kind == 3:
            score[rng.random(n) < 0.5] = -np.inf
        tok = rng.integers(0, 1000, n).astype(np.int32)
        par = np.array([int(rng.integers(-1, i)) if i else -1 for i in range(n)], dtype=np.int32)
        dev = [torch.from_numpy(x).cuda() for x in (tok, par, score)]
        keep = min(total, n)
        out = [torch.full((keep,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
        b._check(b.lib.sparrow_tree_select(*[b._ptr(t) for t in dev], n, total, *[b._ptr(t) for t in out], b._stream_ptr(None)))
        ref = _select_reference(tok, par, score, total)
        for got, want in zip(out, ref):
            assert got.cpu().tolist() == list(want), (n, total, kind)


@pytest.mark.parametrize("n", [129, 191, 192, 193, 255, 256, 257])
@pytest.mark.parametrize("total", [1, 30, 64])
def test_selection_of_pools_around_four_registers(sp, n, total):
    test_selection_sizes(sp, n, total)


@pytest.mark.parametrize("width", [1, 3, 13, 16])
def test_expansion_widths(sp, width):
    import torch
    rng = np.random.default_rng(width)
    pool = sp.TreePool(width, 3)
    score, front = np.zeros(0, dtype=np.float32), None
    for level in range(3):
        m = 1 if level == 0 else width
        logp = np.sort(-rng.integers(1, 6, (m, width)).astype(np.float32), axis=1)[:, ::-1].copy()   # ties
        ids = rng.integers(0, 99, (m, width)).astype(np.int32)
        got = pool.expand(torch.from_numpy(ids).cuda(), torch.from_numpy(logp).cuda()).cpu().numpy()
        base = np.zeros((m, 1), dtype=np.float32) if front is None else score[front][:, None]
        new = (base + logp).reshape(-1)
        order = sorted(range(len(new)), key=lambda i: (-new[i], i))[:width]
        first = len(score)
        score = np.concatenate([score, new])
        front = np.array([first + i for i in order])
        assert np.array_equal(got, front)
        assert np.array_equal(pool.score[:len(score)].cpu().numpy(), score)
        assert np.array_equal(pool.tok[first:len(score)].cpu().numpy(), ids.reshape(-1))
