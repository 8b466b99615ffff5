"""GPU parity of sparrow_accept_sample_q (stochastic acceptance against a sampled draft
distribution, uniforms from the caller or generated by the library) against the CPU fp64 oracle.

As in the other stochastic tests floating point decides integers, so a case is graded bit for bit
only if the oracle's margin (smallest distance of any decision from its threshold, relative to the
remaining mass) is at least MARGIN; other seeds are replaced on the CPU."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu
MARGIN = 1e-4


@pytest.fixture(scope="module")
def sp():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


from gpu_util import dev  # noqa: E402


def _softmax_rows(x):
    e = np.exp(x - x.max(axis=1, keepdims=True))
    return e / e.sum(axis=1, keepdims=True)


def _case(oracle, cfg, seed, B, n_q, parent, V, H, dtype, T):
    """Hidden rows damped so that a row's likeliest token holds roughly half of the mass.  The
    draft distribution of a row is the target's own with the four likeliest tokens scaled down by
    four and every other token scaled up to compensate: a draft that resembles the target, accepts
    a tail token with probability 1/c (c ~ 2-3) and a top token always, and leaves residuals
    max(p - q, 0) that sit on a handful of tokens, so that the bonus draws of graded seeds are well
    conditioned whatever the vocabulary size.  Children are drawn from it independently."""
    ac = wl.accept_case(cfg, seed, vocab=V, batch=B, n_q=n_q, parent=parent, planted=True)
    f = (np.log(V) + 1.0) / (0.02 * H)
    hidden = wl.to_storage(ac.hidden * np.float32(f), dtype)
    rng = np.random.default_rng(seed + 500)
    lg = oracle.logits(hidden, ac.lm_head)
    p = _softmax_rows(lg / T)
    q = np.empty_like(p)
    for r in range(p.shape[0]):
        top = np.argsort(-p[r])[:4]
        m4 = p[r, top].sum()
        c = (1.0 - 0.25 * m4) / (1.0 - m4)
        q[r] = p[r] * c
        q[r, top] = p[r, top] * 0.25
    q = (q / q.sum(axis=1, keepdims=True)).astype(np.float32)
    par = wl.chain_parent(n_q) if parent is None else parent
    draft = np.zeros((B, n_q), dtype=np.int32)
    for b in range(B):
        pb = par if par.ndim == 1 else par[b]
        for j in range(n_q):
            row = b * (n_q + 1) + pb[j] + 1
            pr = q[row].astype(np.float64)
            draft[b, j] = rng.choice(V, p=pr / pr.sum())
    return hidden, ac.lm_head, lg, q, draft.reshape(-1)


CASES = [
    # dtype, H, V, B, n_q, tree, T
    ("f32", 256, 300, 2, 5, "chain", 1.0),
    ("f32", 256, 1000, 3, 9, "tree", 0.8),
    ("bf16", 512, 4096, 2, 12, "tree", 1.0),
    ("bf16", 3584, 4096, 1, 8, "chain", 1.0),
    ("bf16", 3584, 2048, 3, 13, "per-seq", 1.0),
    ("bf16", 1024, 3001, 2, 6, "chain", 1.3),          # vocabulary not a multiple of 4: scalar loads
]


@pytest.mark.parametrize("dtype,H,V,B,n_q,tree,T", CASES)
@pytest.mark.parametrize("generated", [False, True])
def test_accept_sample_q_matches_oracle(sp, oracle, dtype, H, V, B, n_q, tree, T, generated):
    cfg = wl.Config("asq", dtype, 4, 1, 64, B, (((wl.TEXT, 8),),) * B, 8, n_q, tree != "chain", H, V)
    if tree == "chain":
        parent = None
    elif tree == "tree":
        parent = wl.pruned_tree(9, n_q, (3, 2, 2, 1, 1, 1))
    else:
        parent = np.stack([wl.pruned_tree(60 + i, n_q, (3, 2, 2, 1, 1, 1)) for i in range(B)])
    graded, walked = 0, set()
    for seed in range(16):
        hidden, W, lg, q, draft = _case(oracle, cfg, seed, B, n_q, parent, V, H, dtype, T)
        if generated:
            ua, ub = oracle.philox_uniforms(1234 + seed, 7 * seed, B, n_q)
        else:
            rng = np.random.default_rng(seed + 900)
            ua = rng.random((B, n_q)).astype(np.float32).astype(np.float64)
            ub = rng.random(B).astype(np.float32).astype(np.float64)
        alen, path, bonus, margin = oracle.accept_sample_q(lg, draft, parent, B, n_q, T, q, ua, ub)
        if margin.min() < MARGIN:
            continue
        kw = dict(seed=1234 + seed, offset=7 * seed) if generated else \
            dict(u_accept=dev(ua.astype(np.float32)), u_bonus=dev(ub.astype(np.float32)))
        r = sp.accept_sample_q(dev(hidden, dtype), dev(W, dtype), dev(draft),
                               None if parent is None else dev(parent), B, n_q, T, draft_probs=dev(q), **kw)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(r["accept_len"].cpu().numpy(), alen, err_msg=f"seed {seed}")
        np.testing.assert_array_equal(r["accept_path"].cpu().numpy(), path, err_msg=f"seed {seed}")
        np.testing.assert_array_equal(r["bonus_id"].cpu().numpy(), bonus, err_msg=f"seed {seed}")
        walked.update(alen.tolist())
        graded += 1
        if graded == 4:
            break
    assert graded >= 2, "fewer than two well-conditioned seeds among 16"
    assert len(walked) >= 2, f"all graded walks had the same length {walked}: the cases are too easy"


# Above 32,768 tokens the first residual's sums are the whole chip's work, the walk in front of it and the rest of the
# walk (siblings, nodes below an accepted sibling, the draw) kernels of their own; up to there one workgroup does it all.
@pytest.mark.parametrize("V", [16384, 16385, 20480, 32768, 32769, 40003])
@pytest.mark.parametrize("tree,B,n_q", [("chain", 3, 5), ("tree", 2, 13), ("per-seq", 3, 12)])
def test_vocabularies(sp, oracle, V, tree, B, n_q):
    test_accept_sample_q_matches_oracle(sp, oracle, "bf16", 64, V, B, n_q, tree, 1.0, False)


@pytest.mark.parametrize("V", [20011, 36867])
def test_residuals_of_siblings_over_a_large_vocabulary(sp, oracle, V):
    """Siblings that are rejected one after the other, and accepted after others were: counted on the CPU."""
    dtype, H, B, n_q, T = "bf16", 64, 4, 24, 1.0
    parent = np.array([-1] * 6 + [0, 0, 1, 1, 2, 2, 3, 3, 4, 4, 5, 5, 6, 6, 8, 8, 10, 12], dtype=np.int32)
    cfg = wl.Config("asq", dtype, 4, 1, 64, B, (((wl.TEXT, 8),),) * B, 8, n_q, True, H, V)
    graded, late, nested = 0, 0, 0
    for seed in range(16):
        hidden, W, lg, q, draft = _case(oracle, cfg, seed, B, n_q, parent, V, H, dtype, T)
        rng = np.random.default_rng(seed + 900)
        ua = rng.random((B, n_q)).astype(np.float32).astype(np.float64)
        ub = rng.random(B).astype(np.float32).astype(np.float64)
        alen, path, bonus, margin = oracle.accept_sample_q(lg, draft, parent, B, n_q, T, q, ua, ub)
        ok = margin >= MARGIN
        if not ok.any():
            continue
        r = sp.accept_sample_q(dev(hidden, dtype), dev(W, dtype), dev(draft), dev(parent), B, n_q, T, draft_probs=dev(q),
                               u_accept=dev(ua.astype(np.float32)), u_bonus=dev(ub.astype(np.float32)))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(r["accept_len"].cpu().numpy()[ok], alen[ok], err_msg=f"seed {seed}")
        np.testing.assert_array_equal(r["accept_path"].cpu().numpy()[ok], path.reshape(B, n_q)[ok], err_msg=f"seed {seed}")
        np.testing.assert_array_equal(r["bonus_id"].cpu().numpy()[ok], bonus[ok], err_msg=f"seed {seed}")
        for b in np.flatnonzero(ok):
            first = path.reshape(B, n_q)[b][0]
            late += int(alen[b] > 0 and 0 < first < 6)              # accepted after siblings were rejected
            nested += int(alen[b] > 1 and 0 < first < 6)            # and the walk went on below it
        graded += int(ok.sum())
    assert graded >= 12 and late >= 4 and nested >= 1, (graded, late, nested)


def test_generated_uniforms_without_a_draft_distribution(sp, oracle):
    """draft_probs = NULL with library-generated uniforms: the deterministic-children rule of
    sparrow_accept_sample on the Philox stream the oracle generates on its own."""
    dtype, H, V, B, n_q, T = "bf16", 512, 2000, 3, 10, 1.0
    parent = wl.pruned_tree(5, n_q, (3, 2, 2, 1, 1, 1))
    cfg = wl.Config("asq", dtype, 4, 1, 64, B, (((wl.TEXT, 8),),) * B, 8, n_q, True, H, V)
    graded = 0
    for seed in range(12):
        ac = wl.accept_case(cfg, seed, vocab=V, batch=B, n_q=n_q, parent=parent, planted=True)
        hidden = wl.to_storage(ac.hidden * np.float32((np.log(V) + 1.0) / (0.02 * H)), dtype)
        rng = np.random.default_rng(seed)
        draft = ac.draft_ids.reshape(B, n_q).copy()
        t = ac.planted_ids.reshape(B, n_q + 1)
        for b in range(B):
            for j in range(n_q):
                if rng.random() < 0.6:
                    draft[b, j] = t[b, parent[j] + 1]
        draft = draft.reshape(-1).astype(np.int32)
        ua, ub = oracle.philox_uniforms(99, seed, B, n_q)
        ref = oracle.accept_sample_step(hidden, ac.lm_head, draft, parent, B, n_q, T, ua, ub)
        if ref["margin"].min() < MARGIN:
            continue
        r = sp.accept_sample_q(dev(hidden, dtype), dev(ac.lm_head, dtype), dev(draft), dev(parent), B, n_q, T,
                               seed=99, offset=seed)
        torch.cuda.synchronize()
        for key in ("accept_len", "accept_path", "bonus_id"):
            np.testing.assert_array_equal(r[key].cpu().numpy(), ref[key], err_msg=f"seed {seed}: {key}")
        graded += 1
        if graded == 3:
            break
    assert graded >= 2


def test_full_vocabulary_chain_with_a_sampled_draft(sp, oracle):
    """The benchmarked lm_head (152,064 x 3584), chain of 8 drawn from a draft distribution."""
    cfg = wl.C5
    n_q, V, H = cfg.n_q, cfg.vocab, cfg.hidden
    W = wl.lm_head_weights(cfg, 0)
    Wd = dev(W, "bf16")
    graded = 0
    for seed in range(6):
        ac = wl.accept_case(cfg, seed, lm_head=W, planted=True)
        hidden = wl.to_storage(ac.hidden * np.float32((np.log(V) + 1.0) / (0.02 * H)), "bf16")
        rng = np.random.default_rng(seed + 500)
        lg = oracle.logits(hidden, W)
        p = _softmax_rows(lg)
        q = np.empty_like(p)
        for r in range(p.shape[0]):
            top = np.argsort(-p[r])[:4]
            m4 = p[r, top].sum()
            q[r] = p[r] * ((1.0 - 0.25 * m4) / (1.0 - m4))
            q[r, top] = p[r, top] * 0.25
        q = (q / q.sum(axis=1, keepdims=True)).astype(np.float32)
        draft = np.array([rng.choice(V, p=q[j].astype(np.float64) / q[j].astype(np.float64).sum())
                          for j in range(n_q)], dtype=np.int32)
        ua, ub = oracle.philox_uniforms(5, seed, 1, n_q)
        alen, path, bonus, margin = oracle.accept_sample_q(lg, draft, None, 1, n_q, 1.0, q, ua, ub)
        if margin.min() < 1e-5:
            continue
        r = sp.accept_sample_q(dev(hidden, "bf16"), Wd, dev(draft), None, 1, n_q, 1.0, draft_probs=dev(q),
                               seed=5, offset=seed)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(r["accept_len"].cpu().numpy(), alen)
        np.testing.assert_array_equal(r["accept_path"].cpu().numpy(), path)
        np.testing.assert_array_equal(r["bonus_id"].cpu().numpy(), bonus)
        graded += 1
        if graded == 2:
            break
    assert graded >= 1, "no well-conditioned seed among 6"


def test_accept_sample_q_argument_errors(sp):
    h = torch.zeros(3, 256, device="cuda")
    W = torch.zeros(100, 256, device="cuda")
    d = torch.zeros(2, dtype=torch.int32, device="cuda")
    ua, ub = torch.zeros(1, 2, device="cuda"), torch.zeros(1, device="cuda")
    with pytest.raises(sp.SparrowError) as e:          # only one of the two uniform arrays
        sp.accept_sample_q(h, W, d, None, 1, 2, 1.0, u_accept=ua)
    assert e.value.code == -1 and "both" in str(e.value)
    with pytest.raises(sp.SparrowError) as e:
        sp.accept_sample_q(h, W, d, None, 1, 2, 0.0, u_accept=ua, u_bonus=ub)
    assert e.value.code == -1 and "temperature" in str(e.value)


def test_no_draft_rows_is_plain_sampling(sp, oracle):
    """n_q = 0: no draft to accept, the call draws one token per sequence from softmax(logits / T)
    by inverse CDF -- with and without a (never read) draft distribution, caller-given and
    generated uniforms."""
    dtype, H, V, B, T = "bf16", 512, 1500, 3, 0.9
    cfg = wl.Config("asq0", dtype, 4, 1, 64, B, (((wl.TEXT, 8),),) * B, 8, 0, False, H, V)
    graded = 0
    for seed in range(10):
        ac = wl.accept_case(cfg, seed, vocab=V, batch=B, n_q=0, parent=None, planted=True)
        hidden = wl.to_storage(ac.hidden * np.float32((np.log(V) + 1.0) / (0.02 * H)), dtype)
        lg = oracle.logits(hidden, ac.lm_head)
        ua, ub = oracle.philox_uniforms(77, seed, B, 0)
        draft = np.zeros(0, dtype=np.int32)
        alen, _, bonus, margin = oracle.accept_sample(lg, draft, None, B, 0, T, ua, ub)
        if margin.min() < MARGIN:
            continue
        q = torch.full((B, V), 1.0 / V, dtype=torch.float32, device="cuda")
        for kw in (dict(seed=77, offset=seed), dict(seed=77, offset=seed, draft_probs=q),
                   dict(u_accept=dev(ua.astype(np.float32)), u_bonus=dev(ub.astype(np.float32)))):
            r = sp.accept_sample_q(dev(hidden, dtype), dev(ac.lm_head, dtype), dev(draft), None, B, 0, T, **kw)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(r["accept_len"].cpu().numpy(), np.zeros(B, dtype=np.int32))
            np.testing.assert_array_equal(r["bonus_id"].cpu().numpy(), bonus, err_msg=f"seed {seed} {list(kw)}")
        graded += 1
        if graded == 2:
            break
    assert graded >= 1
