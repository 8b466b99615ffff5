"""Verification attention with heads of 64 in bf16 on the matrix cores, against the oracle: row counts
around the 16- and 64-row tiles, contexts around the 32-token tile and the 128-token step, batches on
both grid shapes, and the scratch rule that leaves a call with the plain-ALU kernels."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import dev, host, run_verify  # noqa: E402


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _cfg(Hq, Hkv):
    return wl.Config("D64", "bf16", Hq, Hkv, 64, 1, None, 16, 4, False, 64, 128)


def _check(out, lse, ref, ref_lse, what):
    # the output's bf16 rounding (8 significant bits: half a unit is at most 2^-8 of the value) is all that is larger than fp32 sums: 2e-5 of the
    # row's largest value covers those
    bound = 2.0 ** -8 * np.abs(ref) + 2e-5 * np.abs(ref).max()
    assert np.all(np.abs(out - ref) <= 1.01 * bound), what
    assert np.abs(lse - ref_lse).max() <= 2e-5, f"{what}: lse"      # row sums stay in fp32


def _run(sp, oracle, Hq, Hkv, lengths, n_q, nodes, peaked=False):
    parent = wl.pruned_tree(3, nodes, (4, 3, 2, 2, 1, 1)) if nodes else None
    lay = tuple(((wl.TEXT, n),) for n in lengths)
    c = wl.verify_case(_cfg(Hq, Hkv), seed=sum(lengths) + Hq, layouts=lay,
                       n_q=len(parent) if nodes else n_q, parent=parent, peaked=peaked)
    out, lse = run_verify(sp, c)
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, c.parent, c.n_q)
    _check(out, lse, ref, ref_lse, f"{Hq}/{Hkv} {lengths} n_q={c.n_q}")


@pytest.mark.parametrize("Hq,Hkv,n_q,nodes", [(4, 4, 1, 0), (16, 4, 4, 0), (16, 4, 5, 0), (8, 2, 16, 0), (28, 4, 0, 10),
                                              (28, 4, 0, 25), (16, 2, 0, 30), (32, 4, 0, 60)])
@pytest.mark.parametrize("L", [0, 1, 63, 65, 129, 3001])
def test_rows_and_contexts(sp, oracle, Hq, Hkv, n_q, nodes, L):
    """1, 16, 20, 64, 70, 175, 240 and 480 rows per KV head: one to eight tiles of 64."""
    _run(sp, oracle, Hq, Hkv, (L,), n_q, nodes, peaked=L == 65)


@pytest.mark.parametrize("lengths,n_q,nodes", [((6001, 5200, 4000, 7400), 8, 0), ((26112,), 8, 0), ((9000, 300, 40, 2500), 5, 0),
                                               ((5000, 4300), 0, 30), ((9000, 20), 0, 19), ((26112,), 0, 19)])
def test_batches_and_long_contexts(sp, oracle, lengths, n_q, nodes):
    _run(sp, oracle, 28, 4, lengths, n_q, nodes)


@pytest.mark.parametrize("Hq,Hkv,n_q,nodes", [(2, 2, 1, 0), (15, 1, 1, 0), (8, 1, 2, 0), (17, 1, 1, 0), (12, 4, 0, 10), (16, 2, 4, 0),
                                              (11, 1, 3, 0)])
@pytest.mark.parametrize("lengths", [(31,), (128, 129), (160, 95, 1), (257,), (420, 33), (5000,), (3301, 2000, 64, 1290), (26080,)])
def test_rows_of_two_wavefronts(sp, oracle, Hq, Hkv, n_q, nodes, lengths):
    """1 to 32 rows per KV head, shared out by token: a wavefront takes one of the two tiles of a step.  33: the other way.
    One piece and several, pieces that end in, at and behind either tile of either stream."""
    _run(sp, oracle, Hq, Hkv, lengths, n_q, nodes, peaked=lengths[0] % 2 == 1)


@pytest.mark.parametrize("Hq,Hkv,lengths,nodes", [(28, 4, (26112,), 60), (32, 8, tuple(4129 + 300 * (i % 3 - 1) for i in range(12)), 30)])
def test_two_row_tiles_over_long_pieces(sp, oracle, Hq, Hkv, lengths, nodes):
    """More than ten steps per piece at blocks of 128 rows: two steps in flight, the number of steps odd (13 at 26k)
    and mixed."""
    _run(sp, oracle, Hq, Hkv, lengths, 0, nodes)


def test_an_infinite_value_row_stays_infinite(sp, oracle):
    """One infinite V element: that output column is infinite, the others are as they were."""
    c = wl.verify_case(_cfg(16, 4), seed=5, layouts=(((wl.TEXT, 700),),), n_q=4, parent=None)
    ref, _ = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, 4)
    c.v[123, 1, 7] = np.inf
    out, _ = run_verify(sp, c)
    hit = np.zeros(out.shape, dtype=bool)
    hit[:, 4:8, 7] = True
    assert np.all(np.isposinf(out[hit])) and np.all(np.isfinite(out[~hit]))
    assert np.all(np.abs(out - ref)[~hit] <= 1.01 * (2.0 ** -8 * np.abs(ref) + 2e-5 * np.abs(ref).max())[~hit])


def test_probabilities_keep_32_bits(sp):
    """Three tokens whose weighted values cancel down to 2^-18 of their sizes: what is left shows the
    probabilities' low bits.  Their own fp32 error (score, exponential) is a few units of 2^-24."""
    import torch
    Hkv, d = 16, 64
    g = torch.Generator().manual_seed(11)
    q, k = (torch.randn(n, Hkv, d, generator=g).bfloat16() for n in (1, 3))
    p = torch.softmax(torch.einsum("hd,thd->ht", q[0].double(), k.double()) / 8.0, dim=1)       # [Hkv, 3]
    v = torch.zeros(3, Hkv, d, dtype=torch.bfloat16)
    v[0] = (1 + torch.rand(Hkv, d, generator=g)).bfloat16()
    for i in (1, 2):
        left = sum(p[:, j, None] * v[j].double() for j in range(i))
        v[i] = (-left / p[:, i, None]).bfloat16()
    ref = sum(p[:, j, None] * v[j].double() for j in range(3))
    size = sum(p[:, j, None] * v[j].double().abs() for j in range(3))
    out, _ = sp.verify_attn(q.cuda(), k.cuda(), v.cuda(), np.array([0, 3], dtype=np.int32), None, 1)
    # each term within 2^-21 of its size, and the output's rounding
    assert torch.all((out[0].cpu().double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -20 * size)


@pytest.mark.parametrize("L", [30, 97, 700, 3000])
def test_an_infinite_value_in_the_last_row_stays_infinite(sp, L):
    """The last draft row, which only itself attends: its infinity reaches its own output and not, through
    the rows that fill up the last tile, as 0 * inf."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn(n, h, 64, generator=g, device="cuda").bfloat16() for n, h in ((1, 8), (L + 1, 2), (L + 1, 2)))
    v[L, 1, 7] = float("inf")
    out, _ = sp.verify_attn(q, k, v, np.array([0, L + 1], dtype=np.int32), None, 1)
    assert torch.isposinf(out[0, 4:, 7]).all()
    out[0, 4:, 7] = 0
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("n_q,at", [(1, (0, 32)), (1, (0, 64)), (1, (32, 64)), (40, (0, 64)), (40, (32, 64))])
@pytest.mark.parametrize("L", [80, 270])
def test_values_near_the_end_of_the_range(sp, n_q, at, L):
    """One piece, two tokens that share the whole weight, in states of their own (up to 32 rows of a KV head four, one per
    tile of a step; 40 rows two, one per stream): their mean is in range, the sum of their values is not."""
    import torch
    Hkv = 32
    q = torch.ones(n_q, Hkv, 64, device="cuda").bfloat16()
    k = torch.full((L + n_q, Hkv, 64), -8.0, device="cuda").bfloat16()
    v = torch.zeros_like(k)
    k[list(at)] = 8.0
    v[list(at)] = 3e38
    out, lse = sp.verify_attn(q, k, v, np.array([0, L + n_q], dtype=np.int32), None, n_q)
    assert torch.all(out == v[at[0], 0, 0])              # (scores 128 apart: the others weigh nothing)
    assert float((lse - (64.0 + np.log(2.0))).abs().max()) <= 2e-5


def test_scratch_without_room_for_padded_rows_takes_the_plain_alu_kernels(sp, oracle):
    """64 sequences of one row over 64 KV heads: the matrix-core partials (64-row units) are far larger
    than the plain-ALU ones.  The static scratch and a caller's small workspace still serve the call."""
    import torch
    lay = tuple(((wl.TEXT, 3 + 5 * i % 50),) for i in range(64))
    c = wl.verify_case(_cfg(64, 64), seed=9, layouts=lay, n_q=1, parent=None)
    q, k, v = dev(c.q, "bf16"), dev(c.k, "bf16"), dev(c.v, "bf16")
    assert sp.verify_attn_workspace_bytes(q, k, v, 64, 1, int(c.cu_seqlens[-1])) > sp.STATIC_WS_BYTES
    ref, ref_lse = oracle.verify_attn(c.q, c.k, c.v, c.cu_seqlens, None, 1)
    out, lse = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    sp.verify_attn_static(q, k, v, c.cu_seqlens, None, 1, out, lse=lse)
    _check(host(out), host(lse), ref, ref_lse, "static scratch")
    small = torch.empty(2 << 20, dtype=torch.uint8, device="cuda")
    out2, lse2 = sp.verify_attn(q, k, v, c.cu_seqlens, None, 1, workspace=small)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)
    out3, lse3 = sp.verify_attn(q, k, v, c.cu_seqlens, None, 1)
    _check(host(out3), host(lse3), ref, ref_lse, "matrix cores")
