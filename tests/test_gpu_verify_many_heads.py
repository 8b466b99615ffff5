"""Verification with thousands of query heads per KV head, or of KV heads: partials whose splits lie near 2 GiB apart, queries
of more than 4 GiB, numbers of (sequence, KV head) beyond 2^20.  A row's output is a function of its own query, so the oracle
is given a few heads, the first and the last among them.
test_dispatch.py holds the plan against the offsets' limits on the CPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import check_attn  # noqa: E402


def check_heads(oracle, dtype, d, Hkv, g, n_q, tokens):
    import torch

    import paper_2602_15318_amd as sp
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(g)
    q = torch.randn(n_q, Hkv * g, d, device="cuda", dtype=tdt, generator=gen)
    k, v = (torch.randn(tokens, Hkv, d, device="cuda", dtype=tdt, generator=gen) for _ in range(2))
    cu = np.array([0, tokens], dtype=np.int32)
    print(f"{dtype} d={d} {Hkv * g}/{Hkv} heads, {n_q} rows, {tokens} tokens", flush=True)
    out, lse = sp.verify_attn(q, k, v, cu, None, n_q)
    torch.cuda.synchronize()
    some = sorted({0, 1, g // 3, g // 2, g - 2, g - 1})
    heads = torch.tensor([c * g + h for c in range(Hkv) for h in some], device="cuda")
    f64 = lambda t: t.double().cpu().numpy()
    ref, ref_lse = oracle.verify_attn(f64(q[:, heads]), f64(k), f64(v), cu, None, n_q)
    check_attn(f64(out[:, heads]), ref, dtype, f"{Hkv * g}/{Hkv} heads of {d}")
    assert np.abs(f64(lse[:, heads]) - ref_lse).max() <= (4e-3 if dtype == "bf16" else 2e-5)


@pytest.mark.parametrize("dtype,d,g", [("f32", 128, 4367), ("f32", 128, 4400), ("bf16", 128, 18726), ("bf16", 64, 21846)])
def test_splits_near_2_gib_apart(oracle, dtype, d, g):
    check_heads(oracle, dtype, d, 1, g, 64, 2000)


@pytest.mark.parametrize("dtype,d,g,n_q,tokens", [("bf16", 128, 32769, 33, 700), ("bf16", 64, 65537, 17, 90), ("f32", 64, 50021, 9, 700)])
def test_groups_whose_rows_take_more_than_20_bits(oracle, dtype, d, g, n_q, tokens):
    check_heads(oracle, dtype, d, 1, g, n_q, tokens)


def test_queries_of_more_than_4_gib(oracle):
    check_heads(oracle, "bf16", 128, 9, 29600, 64, 80)


def test_ragged_batch_of_70000_kv_heads(oracle):
    """(sequence, KV head) numbers beyond 2^20 on the one axis that such a call is launched on."""
    import torch

    import paper_2602_15318_amd as sp
    Hkv, d, lens = 70000, 64, [15] * 15 + [14]
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn(len(lens), Hkv, d, device="cuda", dtype=torch.bfloat16, generator=gen)
    k, v = (torch.randn(sum(lens), Hkv, d, device="cuda", dtype=torch.bfloat16, generator=gen) for _ in range(2))
    cu = np.cumsum([0] + lens).astype(np.int32)
    print(f"bf16 d={d} {Hkv} KV heads, {len(lens)} sequences", flush=True)
    out, lse = sp.verify_attn(q, k, v, cu, None, 1)
    torch.cuda.synchronize()
    heads = torch.tensor([0, 1, 2, 65534, 65535, 65536, Hkv // 2, Hkv - 2, Hkv - 1], device="cuda")
    f64 = lambda t: t[:, heads].double().cpu().numpy()
    ref, ref_lse = oracle.verify_attn(f64(q), f64(k), f64(v), cu, None, 1)
    check_attn(f64(out), ref, "bf16", f"{Hkv} KV heads")
    assert np.abs(f64(lse) - ref_lse).max() <= 4e-3
