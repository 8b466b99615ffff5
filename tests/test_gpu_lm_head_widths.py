"""lm_head on the matrix cores for hidden sizes around the 512-element slice of a wavefront (8 to
8,192, short last slices), row counts around the row blocks of a pass and vocabularies around the
16-row tile: target tokens and top-k log-probabilities against a plain fp64 product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _check(sp, H, V, M, seed, dtype="bfloat16"):
    import torch
    dt = getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = (torch.randn(V, H, generator=g, device="cuda") * H ** -0.5).to(dt)
    hid = (torch.randn(M, H, generator=g, device="cuda") * 2.0).to(dt)
    logits = hid.double() @ W.double().t()
    # fp32 sums of H products: a random walk of H roundings of 2^-24, far below 64 * 2^-24 of the
    # largest possible partial sum |hid| . |W|
    tol = 64 * 2.0 ** -24 * float((hid.double().abs() @ W.double().abs().t()).max())
    drafts = torch.zeros(M - 1, dtype=torch.int32, device="cuda")
    if M <= 65:
        got = sp.accept(hid, W, drafts, None, 1, M - 1)["target_ids"].long()
    else:
        # more rows than one sequence has: M sequences without draft rows
        got = sp.accept(hid, W, drafts[:0], None, M, 0)["target_ids"].long()
    assert int(got.min()) >= 0 and int(got.max()) < V
    best = logits.max(dim=1).values
    picked = logits.gather(1, got[:, None])[:, 0]
    assert torch.all(best - picked <= 2 * tol), "a token that is not the row's best"
    top = torch.topk(logits, min(2, V), dim=1).values
    clear = (top[:, 0] - top[:, -1] > 2 * tol) if V > 1 else torch.ones(M, dtype=torch.bool, device="cuda")
    assert torch.equal(got[clear], logits.argmax(dim=1)[clear])
    k = min(4, V)
    ids, logp = sp.draft_topk(hid, W, k)
    ref = torch.topk(torch.log_softmax(logits, dim=1), k, dim=1).values
    assert float((logp.double() - ref).abs().max()) <= 2 * tol + 2e-6
    assert float((torch.log_softmax(logits, dim=1).gather(1, ids.long()) - ref).abs().max()) <= 2 * tol


@pytest.mark.parametrize("H", [8, 264, 512, 520, 1016, 1536, 2048, 2560, 3072, 4096, 4104, 5120, 8192])
@pytest.mark.parametrize("M,V", [(1, 5003), (17, 777), (33, 4096), (64, 15), (65, 2049)])
def test_hidden_sizes(sp, H, V, M):
    _check(sp, H, V, M, H + V + M)


@pytest.mark.parametrize("H,V,M", [(3584, 152064, 9), (2048, 64003, 36), (2560, 32000, 16), (1024, 40000, 64)])
def test_whole_vocabularies(sp, H, V, M):
    _check(sp, H, V, M, 7)


@pytest.mark.parametrize("H", [64, 328, 2048, 4104])
@pytest.mark.parametrize("M,V", [(128, 130), (129, 5003), (256, 128), (257, 1000), (300, 4099), (512, 777)])
def test_many_rows(sp, H, V, M):
    _check(sp, H, V, M, H + V + M)


@pytest.mark.parametrize("H", [4, 68, 260, 1028, 3584])
@pytest.mark.parametrize("M,V", [(1, 5003), (16, 15), (17, 777), (33, 4096), (64, 130), (65, 2049), (300, 1000), (512, 129)])
def test_fp32(sp, H, V, M):
    _check(sp, H, V, M, H + V + M, "float32")


@pytest.mark.parametrize("M,dtype", [(9, "float32"), (20, "float32"), (50, "float32"), (100, "float32"), (100, "bfloat16"),
                                     (200, "bfloat16")])
def test_tiles_of_128_vocabulary_rows(sp, M, dtype):
    """Vocabularies that give every compute unit a tile of 128 rows."""
    _check(sp, 264, 33001, M, M, dtype)


# Rows, vocabulary, vocabulary rows of a tile: row blocks of 64, 128 and 256 rows, full and not, one tile per workgroup and
# several.  test_dispatch.py holds the instances and the tiles per workgroup against the library.
STRAIGHT_TO_LDS = [(33, 140001, 128), (64, 140001, 128), (50, 30011, 64), (65, 33001, 128), (100, 70001, 128),
                   (128, 33001, 128), (128, 9001, 64), (129, 70001, 128), (200, 5003, 64), (256, 33001, 128), (505, 33001, 128)]
# Width, rows, vocabulary, vocabulary rows of a tile: above 4,096 columns from 17 rows on
STRAIGHT_TO_LDS_WIDE = [(4104, 17, 33001, 128), (5120, 20, 32000, 64), (5120, 24, 70001, 128), (8192, 32, 33001, 128),
                        (4104, 33, 70001, 128), (8192, 50, 20011, 64), (5120, 64, 33001, 128), (4104, 65, 12001, 64),
                        (5120, 100, 33001, 128), (8192, 128, 20011, 128), (5120, 129, 20001, 128), (4104, 300, 33001, 128)]


@pytest.mark.parametrize("H,M,V", [(H, M, V) for H in (8, 64, 72, 200, 1032) for M, V, _ in STRAIGHT_TO_LDS]
                         + [(H, M, V) for H, M, V, _ in STRAIGHT_TO_LDS_WIDE])
def test_rows_straight_to_lds(sp, H, V, M):
    """Loads of two steps in flight: 1 to 128 steps per tile, one to three tiles per workgroup.  What lies behind the
    last row and the last token in memory must not reach the result."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(H + V + M)
    W = torch.full((V + 128, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hid = torch.full((M + 256, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    W[:V] = torch.randn(V, H, generator=g, device="cuda") * H ** -0.5
    hid[:M] = torch.randn(M, H, generator=g, device="cuda") * 2.0
    logits = hid[:M].double() @ W[:V].double().t()
    tol = 64 * 2.0 ** -24 * float((hid[:M].double().abs() @ W[:V].double().abs().t()).max())     # as in _check
    ids, logp = sp.draft_topk(hid[:M], W[:V], 4)
    ref = torch.topk(torch.log_softmax(logits, dim=1), 4, dim=1).values
    assert float((logp.double() - ref).abs().max()) <= 2 * tol + 2e-6
    got = sp.accept(hid[:M], W[:V], torch.zeros(0, dtype=torch.int32, device="cuda"), None, M, 0)["target_ids"].long()
    assert torch.all(logits.max(dim=1).values - logits.gather(1, got[:, None])[:, 0] <= 2 * tol)
    assert torch.all((ids == got[:, None].to(ids.dtype)).any(dim=1))


@pytest.mark.parametrize("H,M", [(1920, 33), (1928, 33), (2040, 64), (2048, 33), (2056, 64), (2176, 40), (2184, 40), (4096, 48),
                                 (6144, 17)])
@pytest.mark.parametrize("V", [30011, 140001])
def test_columns_walked_round(sp, H, V, M):
    """Rows within 256 bytes of a multiple of 4 KB (and just outside): workgroups that start at different columns, with a short
    last step in the middle of a tile's walk, one tile per workgroup and several."""
    test_rows_straight_to_lds(sp, H, V, M)


@pytest.mark.parametrize("H", [256, 520, 1000, 2568, 3584, 5120])
@pytest.mark.parametrize("M", [1, 17, 33, 65, 129, 300])
@pytest.mark.parametrize("dtype,limit", [("bfloat16", 0.62e-7), ("float32", 0.9e-7)])
def test_logits_carry_the_error_of_short_sums_only(sp, H, M, dtype, limit):
    """The 2-norm error of the logits against 64 bits does not grow with the width.  A matrix instruction
    rounds its sums at the size they have reached (about four times per 32 bf16 products, once per fp32
    product, 0.3 * 2^-23 each): two bf16 instructions or four fp32 ones from zero are at 0.5e-7 and 0.77e-7
    of the logit's size, the final rounding and that of the wavefronts' shares at 0.25e-7 each."""
    import torch
    import paper_2602_15318_amd.binding as bd
    V, k, dt = 2049, 2, getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(H + M)
    W = (torch.randn(V, H, generator=g, device="cuda") * 0.02).to(dt)
    hid = torch.randn(M, H, generator=g, device="cuda").to(dt)
    code = bd._dtype_code(W)
    ws = torch.zeros(bd.lib.sparrow_draft_topk_workspace(code, M, H, V, k), dtype=torch.uint8, device="cuda")
    sp.draft_topk(hid, W, k, workspace=ws)
    at = bd.lib.sparrow_accept_workspace(code, 1, M - 1, H, V)          # the logits lie behind the candidates
    logits = ws[at:at + 4 * M * V].view(torch.float32).view(M, V).double()
    ref = hid.double() @ W.double().t()
    assert float((logits - ref).norm() / ref.norm()) <= limit


@pytest.mark.parametrize("M,V,dtype", [(M, V, "bfloat16") for M in (3, 20, 40, 100, 140) for V in (33001, 33002, 33003)]
                         + [(40, 2050, "bfloat16"), (140, 6827, "bfloat16"), (5, 2051, "float32"), (70, 130, "float32")])
def test_stored_logits_of_odd_vocabularies(sp, M, V, dtype):
    """Four logits by one store, the last of a row by fewer: every logit of every row, one slice of a weight row."""
    import torch
    import paper_2602_15318_amd.binding as bd
    H, k, dt = 264, 2, getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(V + M)
    W = (torch.randn(V, H, generator=g, device="cuda") * H ** -0.5).to(dt)
    hid = (torch.randn(M, H, generator=g, device="cuda") * 2.0).to(dt)
    code = bd._dtype_code(W)
    ws = torch.full((bd.lib.sparrow_draft_topk_workspace(code, M, H, V, k),), 0xff, dtype=torch.uint8, device="cuda")
    sp.draft_topk(hid, W, k, workspace=ws)
    at = bd.lib.sparrow_accept_workspace(code, 1, M - 1, H, V)          # the logits lie behind the candidates
    logits = ws[at:at + 4 * M * V].view(torch.float32).view(M, V).double()
    tol = 64 * 2.0 ** -24 * float((hid.double().abs() @ W.double().abs().t()).max())     # as in _check
    assert float((logits - hid.double() @ W.double().t()).abs().max()) <= tol


@pytest.mark.parametrize("H", [2048, 4104, 8192])
@pytest.mark.parametrize("M", [33, 64, 65, 200, 512])
@pytest.mark.parametrize("V", [7, 1000, 3001])
def test_row_blocks_side_by_side(sp, H, M, V):
    """Small vocabularies above 32 rows: the k-split kernel with up to 32 row blocks in one launch."""
    _check(sp, H, V, M, H + V + M)


def test_wider_than_the_matrix_core_kernels(sp):
    _check(sp, 8704, 300, 3, 1)
    _check(sp, (1 << 20) + 4, 20, 2, 1, "float32")


@pytest.mark.parametrize("H", [520, 5120])
def test_columns_past_the_width_do_not_reach_the_result(sp, H):
    """The last slice of a row is short: what lies behind the row in memory (the next row, here an
    infinite one; other tensors behind the last row) must not leak into the sums."""
    import torch
    W = torch.ones(40, H, dtype=torch.bfloat16, device="cuda")
    W[5] = float("inf")
    hid = torch.full((3, H), 0.5, dtype=torch.bfloat16, device="cuda")
    ids, _ = sp.draft_topk(hid, W[:5].contiguous(), 2)
    assert ids.tolist() == [[0, 1]] * 3                      # all rows tie: the lowest ids
    r = sp.accept(hid, W, torch.zeros(2, dtype=torch.int32, device="cuda"), None, 1, 2)
    assert r["target_ids"].tolist() == [5] * 3               # and the infinite row is the only best one
