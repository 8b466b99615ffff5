"""The draft's input side in bf16 for hidden sizes around the 512-element slice of a wavefront (8 to
8,200, short last slices) and row counts around the 16-row block, against plain fp64 products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2602_15318_amd as sp_
    return sp_


def _bf(g, *shape, std=1.0):
    import torch
    return (torch.randn(*shape, generator=g, device="cuda") * std).to(torch.bfloat16)


def _close(got, ref, abs_sum, what):
    # one rounding of the result to bf16 (at most 2^-8 of it) and the fp32 sums: 2^-15 of the sum of the
    # terms' magnitudes covers them
    bound = 1.01 * 2.0 ** -8 * ref.abs() + 2.0 ** -15 * abs_sum
    excess = (got.double() - ref).abs() - bound
    assert float(excess.max()) <= 0, f"{what}: over the bound by {float(excess.max()):.3e}"


@pytest.mark.parametrize("H", [8, 72, 512, 520, 1000, 1280, 2560, 3584, 4104, 5120, 8200])
@pytest.mark.parametrize("M", [1, 2, 16, 17, 64])
def test_hsr_fc(sp, H, M):
    import torch
    g = torch.Generator(device="cuda").manual_seed(H + M)
    embed, h, w, b = _bf(g, 50, H), _bf(g, M, H), _bf(g, H, 2 * H, std=H ** -0.5), _bf(g, H)
    tok = torch.randint(0, 50, (M,), generator=g, device="cuda", dtype=torch.int32)
    x = torch.cat([embed[tok.long()], h], dim=1).double()
    for bias in (b, None):
        z = sp.hsr_fc(embed, tok, h, w, bias)
        add = 0.0 if bias is None else bias.double()
        _close(z, x @ w.double().t() + add, x.abs() @ w.double().abs().t() + abs(add), f"H={H} M={M}")


@pytest.mark.parametrize("H,Hq,Hkv,d", [(8, 2, 1, 64), (72, 6, 2, 128), (512, 4, 2, 64), (1000, 8, 2, 128), (2560, 40, 8, 64),
                                        (3072, 28, 4, 128), (4104, 8, 1, 64), (5120, 40, 8, 128), (8200, 4, 4, 64)])
@pytest.mark.parametrize("M", [1, 2, 16, 17, 64])
def test_draft_qkv_append(sp, H, Hq, Hkv, d, M):
    import torch
    g = torch.Generator(device="cuda").manual_seed(H + M)
    F = (Hq + 2 * Hkv) * d
    z, gam, w, b = _bf(g, M, H, std=1.5), _bf(g, H), _bf(g, F, H, std=H ** -0.5), _bf(g, F)
    ang = torch.rand(M, d // 2, generator=g, device="cuda", dtype=torch.float64) * 6.0
    kc, vc = torch.zeros(80, Hkv, d, dtype=torch.bfloat16, device="cuda"), torch.zeros(80, Hkv, d, dtype=torch.bfloat16, device="cuda")
    rows = np.random.default_rng(M).permutation(80)[:M].astype(np.int32)
    q = sp.draft_qkv_append(z, gam, 1e-6, w, b, ang.cos().float(), ang.sin().float(), rows, Hq, kc, vc)
    x = z.double()
    u = x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + 1e-6) * gam.double()
    f = (u @ w.double().t() + b.double()).view(M, -1, d)
    s = (u.abs() @ w.double().abs().t() + b.double().abs()).view(M, -1, d)
    c, sn = ang.cos().float().double()[:, None], ang.sin().float().double()[:, None]
    lo, hi, slo, shi = f[..., :d // 2], f[..., d // 2:], s[..., :d // 2], s[..., d // 2:]
    rot = torch.cat([lo * c - hi * sn, hi * c + lo * sn], dim=2)
    srot = torch.cat([slo + shi, slo + shi], dim=2)
    at = torch.from_numpy(rows).long().cuda()
    _close(q, rot[:, :Hq], srot[:, :Hq], f"q H={H} M={M}")
    _close(kc[at], rot[:, Hq:Hq + Hkv], srot[:, Hq:Hq + Hkv], f"k H={H} M={M}")
    _close(vc[at], f[:, Hq + Hkv:], s[:, Hq + Hkv:], f"v H={H} M={M}")
    rest = np.setdiff1d(np.arange(80), rows)
    assert not kc[rest].any() and not vc[rest].any()


@pytest.mark.parametrize("M", [1, 2, 17])
def test_normalised_activations_enter_exactly(sp, M):
    """An activation times its gamma has 16 bits.  Three products that cancel exactly leave nothing:
    (1 + 2^-7)^2 - (1 + 2^-6) - 2^-14.  (At most 2^-38: the second bf16 term of a product is never zero.)"""
    import torch
    H, Hq, Hkv, d = 1032, 4, 2, 64
    rng = np.random.default_rng(5)
    z, gam = torch.ones(M, H, dtype=torch.bfloat16), torch.ones(H, dtype=torch.bfloat16)
    z[:, 1::3] = gam[1::3] = 1 + 2.0 ** -7
    w = torch.zeros((Hq + 2 * Hkv) * d, H, dtype=torch.bfloat16)
    for f in range(w.shape[0]):
        c = 3 * rng.integers(0, H // 3, size=3) + np.array([0, 1, 2])
        w[f, c] = torch.tensor([-(1 + 2.0 ** -6), 1.0, -2.0 ** -14], dtype=torch.bfloat16)
    one = torch.ones(M, d // 2, device="cuda")
    kc, vc = (torch.ones(M, Hkv, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q = sp.draft_qkv_append(z.cuda(), gam.cuda(), 1e-6, w.cuda(), None, one, one, np.arange(M), Hq, kc, vc)
    assert max(float(t.abs().max()) for t in (q, kc, vc)) <= 2.0 ** -38


@pytest.mark.parametrize("M", [1, 3])
def test_infinite_weights_give_infinities(sp, M):
    """A weight of infinity beside non-zero activations: its features are infinite, the others finite."""
    import torch
    H, Hq, Hkv, d = 520, 4, 2, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    z, w = _bf(g, M, H).abs() + 0.5, _bf(g, (Hq + 2 * Hkv) * d, H, std=0.05)
    v_feat = (Hq + Hkv) * d + 5
    w[v_feat, 513] = float("inf")
    gam, one = torch.ones(H, dtype=torch.bfloat16, device="cuda"), torch.ones(M, d // 2, device="cuda")
    kc, vc = (torch.zeros(M, Hkv, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sp.draft_qkv_append(z, gam, 1e-6, w, None, one, one, np.arange(M), Hq, kc, vc)
    assert torch.isposinf(vc[:, 0, 5]).all()
    vc[:, 0, 5] = 0
    assert torch.isfinite(vc).all() and torch.isfinite(kc).all()


# Few rows: FC of two to four rows, two features a wavefront, activations in LDS ten slices at a time (four up to 1,024
# columns); QKV of up to eight rows, two lanes a row; more rows the other way.  Widths around a slice, both halves of a
# concatenation in one chunk and in several, workgroups of four to eight wavefronts and a last one with idle ones.
FEW_WIDTHS = [8, 504, 512, 520, 1024, 1032, 2056, 2560, 2568, 4104, 5128]


@pytest.mark.parametrize("H", FEW_WIDTHS)
@pytest.mark.parametrize("M", [3, 4, 5])
def test_hsr_fc_of_few_rows(sp, H, M):
    test_hsr_fc(sp, H, M)


@pytest.mark.parametrize("H,Hq,Hkv,d", [(H, *((6, 3, 64) if i % 2 else (5, 1, 128))) for i, H in enumerate(FEW_WIDTHS)]
                         + [(2048, 40, 8, 128)])
@pytest.mark.parametrize("M", [1, 3, 7, 8, 9])
def test_draft_qkv_of_few_rows(sp, H, Hq, Hkv, d, M):
    test_draft_qkv_append(sp, H, Hq, Hkv, d, M)


@pytest.mark.parametrize("H,Hq,Hkv,d", [(24, 3, 1, 64), (264, 7, 1, 128), (2560, 40, 8, 64), (3072, 24, 8, 128), (3080, 5, 5, 64),
                                        (4088, 9, 3, 64), (4096, 16, 4, 64), (3584, 16, 8, 128)])
@pytest.mark.parametrize("M", [2, 5, 8])
def test_one_slice_a_wavefront(sp, H, Hq, Hkv, d, M):
    """Two to eight rows, all weights at once: 1 to 8 rotary pairs and 2 to 12 features a workgroup, the last one with fewer,
    tiles that cross heads, short last slices, 1 to 16 wavefronts."""
    test_hsr_fc(sp, H, M)
    test_draft_qkv_append(sp, H, Hq, Hkv, d, M)


@pytest.mark.parametrize("H,Hq,Hkv,d", [(3584, 28, 4, 128), (4096, 6, 2, 64)])
def test_draft_qkv_of_one_row_at_whole_slices(sp, H, Hq, Hkv, d):
    test_draft_qkv_append(sp, H, Hq, Hkv, d, 1)


@pytest.mark.parametrize("H", [512, 1024, 3584, 4104])
def test_an_infinite_gamma_gives_infinities(sp, H, M=1):
    """Both terms of an infinite product are infinite: of one sign, not infinity minus infinity."""
    import torch
    Hq, Hkv, d = 4, 2, 64
    g = torch.Generator(device="cuda").manual_seed(H)
    z, w = _bf(g, M, H).abs() + 0.5, _bf(g, (Hq + 2 * Hkv) * d, H, std=0.05).abs() + 0.25
    gam, one = torch.ones(H, dtype=torch.bfloat16, device="cuda"), torch.ones(M, d // 2, device="cuda")
    gam[H - 3] = float("inf")
    kc, vc = (torch.zeros(M, Hkv, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sp.draft_qkv_append(z, gam, 1e-6, w, None, one, one, np.arange(M), Hq, kc, vc)
    assert torch.isposinf(vc).all()


@pytest.mark.parametrize("H", [504, 1024, 3584, 4104])
@pytest.mark.parametrize("M", [1, 2, 3, 8, 9, 17])
@pytest.mark.parametrize("inf", [float("inf"), float("-inf")])
def test_an_infinite_gamma_in_a_batch_gives_infinities(sp, H, M, inf):
    """Of either sign, at one row, two lanes a row, sixteen rows to a block, and a second block.  Beside a product without
    low bits and one with them."""
    import torch
    Hq, Hkv, d = 4, 2, 64
    g = torch.Generator(device="cuda").manual_seed(H)
    z, w = _bf(g, M, H).abs() + 0.5, _bf(g, (Hq + 2 * Hkv) * d, H, std=0.05).abs() + 0.25
    gam, one = torch.ones(H, dtype=torch.bfloat16, device="cuda"), torch.ones(M, d // 2, device="cuda")
    gam[H - 4], gam[H - 3], gam[H - 2] = 1.0078125, inf, 1.0
    kc, vc = (torch.zeros(M, Hkv, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sp.draft_qkv_append(z, gam, 1e-6, w, None, one, one, np.arange(M), Hq, kc, vc)
    assert torch.all(vc == inf)
