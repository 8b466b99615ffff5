"""The kernels that calls are sent to, and how their work is cut, on the CPU (launch_recorder.py)."""
import math
import random

import pytest

from launch_recorder import record


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("recorder")
    return lambda calls: record(calls, tmp)


def verify(Hq, Hkv, n_q, lens, layout="token", own=False, d=128, dtype="bf16"):
    return dict(call="verify", dtype=dtype, Hq=Hq, Hkv=Hkv, d=d, n_q=n_q, lens=list(lens), layout=layout, own=own)


IN_STEP, HALF_STEP = "verify_partial_mfma_kernel<128, 2, 2, false>", "verify_partial_mfma_kernel<128, 2, 2, true>"


@pytest.mark.parametrize("layout", ["token", "head", "pair"])
def test_streams_half_a_step_apart_only_where_they_are_faster(launches, layout):
    """Several blocks of 128 rows over splits of 14 steps of 64 tokens and more.  One block loses 1 to 9 per cent by it
    with every layout of K and V, shorter splits 1 to 4."""
    cases = [((28, 4, 16), 64, 704, IN_STEP), ((28, 4, 16), 64, 1920, IN_STEP), ((32, 8, 30), 32, 1472, IN_STEP),
             ((28, 4, 30), 32, 704, IN_STEP), ((28, 4, 30), 32, 832, IN_STEP), ((28, 4, 30), 32, 864, HALF_STEP),
             ((28, 4, 60), 16, 832, IN_STEP), ((28, 4, 60), 16, 864, HALF_STEP), ((28, 4, 60), 16, 1664, HALF_STEP),
             ((28, 4, 60), 16, 640, "verify_partial_mfma_kernel<128, 1, 2, false>")]
    got = launches([verify(*heads, [splits * piece], layout) for heads, splits, piece, _ in cases])
    for (heads, splits, piece, kernel), run in zip(cases, got):
        assert (run[0]["splits"], run[0]["pieces"]) == ([splits], [piece]), (heads, run[0])
        assert run[0]["kernel"] == kernel, (heads, splits, piece)


def test_long_tree_cases(launches):
    """test_gpu_verify_long_trees.py runs the instances, splits and grids that it names."""
    from test_gpu_verify_long_trees import BATCHES, ONE_SEQUENCE
    got = launches([verify(*heads, [splits * piece - short]) for heads, splits, piece, short in ONE_SEQUENCE])
    for (heads, splits, piece, short), run in zip(ONE_SEQUENCE, got):
        assert (run[0]["splits"], run[0]["pieces"]) == ([splits], [piece]), (heads, short, run[0])
        assert short < piece
        half = heads[0] // heads[1] * heads[2] > 128 and piece > 832
        assert run[0]["kernel"] == (HALF_STEP if half else IN_STEP), (heads, piece, short)
    kinds = set()
    for layout in ("token", "head", "pair"):
        got = launches([verify(*heads, lens, layout, own=True) for heads, lens, _, _ in BATCHES])
        for (heads, lens, splits, flat), run in zip(BATCHES, got):
            assert (run[0]["splits"], run[0]["flat"]) == (list(splits), flat), (heads, lens, run[0])
            last = [n - (s - 1) * p for n, s, p in zip(lens, splits, run[0]["pieces"])]
            kinds.add((run[0]["kernel"], flat, min(last) <= 0))
    assert kinds >= {(HALF_STEP, False, False), (HALF_STEP, True, False), (HALF_STEP, True, True), (IN_STEP, True, False)}


def test_combine_of_few_splits(launches):
    """One wavefront up to four splits a sequence, two up to eight, four up to sixteen;
    test_gpu_verify_few_splits.py runs the first two at both head sizes."""
    from test_gpu_verify_few_splits import CASES
    for d in (64, 128):
        got = launches([verify(*heads, lens, d=d) for heads, lens, _ in CASES])
        for (heads, lens, most), run in zip(CASES, got):
            assert max(run[0]["splits"]) == most, (heads, lens, run[0]["splits"])
            assert run[1]["kernel"] == f"verify_combine_few_kernel<unsigned short, {d}, {1 if most <= 4 else 2}>", (heads, lens)
    got = launches([verify(28, 4, n_q, [n] * B) for B, n, n_q in ((4, 26112, 25), (1, 12000, 60))])
    assert {run[1]["kernel"] for run in got} == {"verify_combine_tiled_kernel<unsigned short, 128, 4>"}


def test_combine_of_many_splits(launches):
    """16 splits a wavefront, and four wavefronts over 16-row tiles where 9 to 16 splits meet many row blocks;
    test_gpu_verify_long_splits.py runs them."""
    from test_gpu_verify_long_splits import CASES
    seen = set()
    for d in (64, 128):
        got = launches([verify(*heads, lens, d=d) for heads, lens, _ in CASES])
        for (heads, lens, most), run in zip(CASES, got):
            if d == 128:
                assert max(run[0]["splits"]) == most, (heads, lens, run[0]["splits"])
            most = max(run[0]["splits"])
            units = heads[1] * -(-heads[0] // heads[1] * heads[2] // 64)
            kernel = run[1]["kernel"]
            if most > 16 or (most > 8 and units <= 8):
                assert kernel == f"verify_combine_long_kernel<unsigned short, {d}, {min(w for w in (1, 2, 4, 8, 16) if 16 * w >= most or w == 16)}>"
            elif most > 8:
                assert kernel == f"verify_combine_tiled_kernel<unsigned short, {d}, 4>"
            seen.add(kernel)
    assert {f"verify_combine_long_kernel<unsigned short, {d}, {w}>" for d in (64, 128) for w in (1, 2, 4, 8, 16)} <= seen


def test_any_number_of_heads_on_the_matrix_cores(launches):
    for dtype in ("bf16", "f32"):
        for run in launches([verify(g, 1, n_q, [900], dtype=dtype) for g in (32767, 32768, 100003) for n_q in (1, 64)]):
            assert run[0]["kernel"].startswith("verify_partial_mfma_kernel" if dtype == "bf16" else "verify_partial_f32_kernel"), run


def test_any_number_of_kv_heads_on_one_grid_axis(launches):
    """Short sequences of very many KV heads are numbered along x, like any others: a grid's other axes end at 65,535."""
    lens = [([15] * 15 + [14], 70000), ([15] * 16, 70000), ([16], 1 << 20), ([40] * 3, 400000)]
    for (ns, heads), run in zip(lens, launches([verify(heads, heads, 1, ns, "head", d=64) for ns, heads in lens])):
        assert run[0]["flat"] and run[0]["grid"] == [len(ns) * heads, 1, 1], run


@pytest.mark.parametrize("dtype,d,unit_bytes,most", [("bf16", 64, 16384, 8), ("bf16", 128, 16384, 8), ("f32", 64, 16384, 16),
                                                      ("f32", 128, 32768, 16)])
def test_combine_offsets(launches, dtype, d, unit_bytes, most):
    """The combine kernels address a sequence's splits by 31-bit offsets from its first one, and those of (m, l, c), 12
    bytes a row, by a product of 24 bits: so many query heads per KV head that the plan's splits lie further apart get fewer."""
    units = sorted({g + i for s in range(1, most) for g in [(2 ** 31 - 1) // (s * unit_bytes)] for i in (-2, -1, 0, 1)} | {64, 2000, 21845, 21846})
    got = launches([verify(u, 1, 64, [26000], d=d, dtype=dtype) for u in units])
    splits = {}
    for u, run in zip(units, got):
        assert run[1]["units"] == u, (u, run)
        splits[u] = run[1]["splits"]
        assert (splits[u] - 1) * u * unit_bytes + unit_bytes <= 2 ** 31 - 1, (u, run)
        assert u * 64 * 12 < 2 ** 24 or splits[u] == 1, (u, run)
    assert splits[2000] == most and splits[21846] == 1


def test_combine_kernels_of_row_counts(launches):
    """test_gpu_verify_long_splits.py runs every combine kernel's workgroups with and without rows."""
    for Hkv, lens, kernels in ((1, [4500], {"long"}), (12, [3000] * 2, {"tiled"}), (12, [1300] * 4, {"few"}), (12, [1000, 900] * 4, {"few"})):
        got = launches([verify(Hkv * rows, Hkv, 1, lens) for rows in (1, 16, 64, 65, 130)])
        assert {run[1]["kernel"].split("_")[2] for run in got} == kernels, (Hkv, lens, [run[1] for run in got])


@pytest.mark.parametrize("d", [64, 128])
def test_pieces(launches, d):
    """Pieces are whole 32-token tiles that cover a sequence.  Sequences of one length get as many as whole 64-token steps allow
    (up to 8 steps): none is empty, and none takes more steps than an even share of the slots."""
    sizes = (70, 300, 642, 1000, 1538, 2049, 4101, 7173, 8197, 11111, 26117, 40000)
    calls = [verify(*heads, 5, lens, d=d) for heads in ((28, 4), (16, 8), (32, 32)) for n in sizes for lens in
             ([n], [n, n], [n] * 4, [n] * 7, [n] * 8, [n, n // 3 + 8], [n, n // 2 + 7, n // 5 + 9, n])
             if sum(lens) * heads[1] * d * 2 < 2 ** 31]
    for c, run in zip(calls, launches(calls)):
        equal = len(set(c["lens"])) == 1
        for n, s, p in zip(c["lens"], run[0]["splits"], run[0]["pieces"]):
            assert p % 32 == 0 and s * p >= n, (c, run[0])
            if equal and len(run) == 2:
                share = -(-n // (256 // c["Hkv"] // len(c["lens"])))
                steps = -(-share // 64) if share <= 512 else -(-share // 32) / 2
                assert s == math.ceil(n / (64 * steps)) and (s - 1) * p < n and p <= 64 * steps, (c, run[0])


def plan_by_proportion(lens, slots):
    """Splits of sequences that differ: about `slots` pieces of whole 32-token tiles dealt in proportion to the lengths, what is
    left to the longest pieces; a sequence's pieces are equal."""
    total = sum(lens)
    budget = -(-total // max(64, -(-(-(-total // slots)) // 32) * 32))
    ns = [max(1, n * budget // total) for n in lens]
    while sum(ns) < budget:
        ns[max(range(len(lens)), key=lambda b: lens[b] / ns[b])] += 1
    return ns


@pytest.mark.parametrize("d", [64, 128])
def test_ragged_batches_use_every_slot(launches, d):
    """Sequences that differ are cut by proportion into as many pieces of 32-token grain as there are slots; a coarser grain
    of their budget leaves compute units idle and makes the longest piece longer."""
    rng = random.Random(d)
    calls = [((28, 4, 1), (1538, 1948, 1219, 903)), ((28, 4, 8), (791, 1218, 734, 1574, 955, 1113, 1699, 1688)),
             ((28, 4, 6), (1448, 1229, 693, 2084, 1911, 2213, 1384, 1933)), ((28, 4, 8), (6110, 6049, 2670, 2093))]
    calls += [((28, 4, rng.randint(1, 9)), tuple(rng.randint(600, 6000) for _ in range(rng.randint(2, 9)))) for _ in range(100)]
    for (heads, lens), run in zip(calls, launches([verify(*heads, lens, d=d) for heads, lens in calls])):
        if len(run) == 2 and len(set(lens)) > 1:
            assert run[0]["splits"] == plan_by_proportion(lens, 64), (heads, lens, run[0])


def test_equal_batches_fit_the_scratch_of_the_proportional_plan(launches):
    """Sequences of one length, cut alike, may take more pieces than by proportion to the chip; scratch that holds no more than
    those is not refused, and more scratch changes nothing."""
    calls = [(Hkv, n_q, [n] * B) for Hkv in (4, 8, 32) for n_q in (1, 5, 9) for B in (1, 2, 4, 6, 8) for n in (66, 85, 100, 260, 807, 4995)]
    tight = [plan_by_proportion(lens, 256 // Hkv) for Hkv, n_q, lens in calls]
    unit = 64 * (4 * 64 + 12)                                # bytes of 64 rows of a split and KV head: fp16 values, (m, l, c)
    few = launches([dict(verify(7 * Hkv, Hkv, n_q, lens), workspace=sum(ns) * Hkv * unit) for (Hkv, n_q, lens), ns in zip(calls, tight)])
    many = launches([verify(7 * Hkv, Hkv, n_q, lens) for Hkv, n_q, lens in calls])
    assert any(sum(m[0]["splits"]) > sum(ns) for m, ns in zip(many, tight) if len(m) == 2)
    for c, ns, f, m in zip(calls, tight, few, many):
        assert f == m or (sum(m[0]["splits"]) > sum(ns) and f[0]["splits"] == ns), (c, ns, f, m)


def test_lm_head_cases_straight_to_lds(launches):
    """test_gpu_lm_head_widths.py runs every instance that loads straight to LDS: each row block with one tile per
    workgroup and, where its tiles have 128 rows, with several; and these instances from 17 rows up above 4,096 columns."""
    from test_gpu_lm_head_widths import STRAIGHT_TO_LDS, STRAIGHT_TO_LDS_WIDE
    cases = [(H, M, V, vt) for H in (8, 1032) for M, V, vt in STRAIGHT_TO_LDS] + STRAIGHT_TO_LDS_WIDE
    seen = {}
    for call in ("accept", "topk"):
        got = launches([dict(call=call, dtype="bf16", M=M, H=H, V=V) for H, M, V, _ in cases])
        for (H, M, V, vt), run in zip(cases, got):
            rows = 64 if M <= 64 else 128 if M <= 128 else 256
            assert run[0]["kernel"] == f"lm_head_tiled_kernel<unsigned short, {vt}, {rows}, 8, 2, 128>", (call, H, M, V)
            workgroups = run[0]["grid"][0] // -(-M // rows)
            seen.setdefault((vt, rows), set()).add(-(-V // vt) > workgroups)
    assert seen == {(64, r): {False} for r in (64, 128, 256)} | {(128, r): {False, True} for r in (64, 128, 256)}
