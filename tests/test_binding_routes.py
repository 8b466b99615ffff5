"""binding.py's native part against its general code: what it leaves to that code (CPU), and that both routes of a call
give the same results, of the same types and shapes, or the same exception (GPU)."""
import os
import shutil
import subprocess
import sys
import types

import numpy as np
import pytest
import torch

import paper_2602_15318_amd as sp
from paper_2602_15318_amd import binding

NAMES = ("verify_attn", "draft_window_attn", "accept", "hsr_fc", "draft_qkv_append")
GENERAL = types.SimpleNamespace(**{n: lambda *a: NotImplemented for n in NAMES})


class Sub(torch.Tensor):
    pass


def _calls(device, dtype=torch.bfloat16):
    """name -> arguments of a call that the native part takes"""
    g = torch.Generator().manual_seed(1)

    def r(*shape, dt=dtype):
        return torch.randn(shape, generator=g).to(dt).to(device)

    def ints(*x):
        return torch.tensor(x, dtype=torch.int32, device=device)

    Hq, Hkv, d, H, V, n_q = 8, 2, 64, 256, 512, 3
    lens = np.array([0, 70, 200], np.int32)
    kv = r(2, 200, Hkv, d)
    return {
        "verify_attn": [r(2 * n_q, Hq, d), kv[0], kv[1], lens, ints(-1, 0, 0), n_q],
        "draft_window_attn": [r(2, Hq, d), kv[0], kv[1], lens, ints(0, 3, 69, 1, 2, 129), np.array([0, 3, 6], np.int32), 8],
        "accept": [r(2 * (n_q + 1), H), r(V, H), ints(*range(2 * n_q)), None, 2, n_q],
        "hsr_fc": [r(V, H), ints(5, 9), r(2, H), r(H, 2 * H), r(H)],
        "draft_qkv_append": [r(2, H), r(H), 1e-6, r((Hq + 2 * Hkv) * d, H), None, r(2, d // 2, dt=torch.float32),
                             r(2, d // 2, dt=torch.float32), np.array([69, 199], np.int32), Hq, kv[0], kv[1]],
    }


# arguments whose type neither route looks at
UNCHECKED = {("accept", 2), ("verify_attn", 1), ("verify_attn", 2), ("draft_window_attn", 1), ("draft_window_attn", 2),
             ("draft_qkv_append", 9), ("draft_qkv_append", 10)}


def _odd_forms(name, args):
    """(what, arguments) that binding.py's own code converts or refuses, one argument at a time"""
    for i, a in enumerate(args):
        if isinstance(a, np.ndarray):
            yield f"{i} list", i, a.tolist()
            yield f"{i} int64", i, a.astype(np.int64)
            yield f"{i} every other", i, np.repeat(a, 2)[::2]
            yield f"{i} short", i, a[:-1]
        elif isinstance(a, torch.Tensor):
            yield f"{i} subclass", i, a.as_subclass(Sub)
            if (name, i) not in UNCHECKED:
                yield f"{i} float64", i, a.double()
            if a.dim() > 1:
                yield f"{i} transposed", i, a.transpose(0, -1)
        elif isinstance(a, int):
            yield f"{i} numpy", i, np.int64(a)


def _native_args(name, a):
    tail = {"verify_attn": (0.0, None, None, True, None, 0), "draft_window_attn": (0.0, None, None, True, 0), "accept": (None, 0),
            "hsr_fc": (None, 0), "draft_qkv_append": (None, 0)}[name]
    return [*a, *tail]


@pytest.mark.parametrize("name", NAMES)
def test_what_is_left_to_the_general_code(name):
    args = _calls("cpu")[name]
    fn = getattr(binding._native, name)
    n = 0
    for what, i, x in _odd_forms(name, args):
        if name == "draft_window_attn" and what.endswith("short"):
            continue                                     # (B follows from q: the general code refuses it)
        a = list(args)
        a[i] = x
        if name == "verify_attn" and what.endswith("short"):
            continue                                     # (a call of one sequence: the library looks at its rows)
        assert fn(*_native_args(name, a)) is NotImplemented, what
        n += 1
    assert n >= 4
    with torch.overrides.TorchFunctionMode():
        assert fn(*_native_args(name, args)) is NotImplemented


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _python(code, **env):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env={**os.environ, **env}, stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout.splitlines(), r.stderr


def test_both_routes_call_the_library_beside_the_package(tmp_path):
    """Also with another libsparrow.so on the loader's search path: one is mapped, and a refusal by the native part's route
    reads that one's error text."""
    shutil.copy(sp.library_path(), tmp_path / "libsparrow.so")
    out, _ = _python("""
import types
import numpy as np, torch
import paper_2602_15318_amd as sp
z, one = torch.zeros(1, 4, 64), np.array([0, 1], np.int32)
try:
    sp.draft_window_attn(z, z, z, one, torch.zeros(1, dtype=torch.int32), one, -1, stream=types.SimpleNamespace(cuda_stream=0))
except sp.SparrowError as e:
    print(e)
for path in sorted({l.split()[-1] for l in open("/proc/self/maps") if l.rstrip().endswith("libsparrow.so")}):
    print(path)
""", LD_LIBRARY_PATH=f"{tmp_path}:{os.environ.get('LD_LIBRARY_PATH', '')}")
    assert out[1:] == [sp.library_path()]
    assert "window = -1 must be positive" in out[0]


@pytest.mark.parametrize("prepare", ["import torch; torch.__version__ = torch.torch_version.TorchVersion('1.2.3')",
                                     "import sys; sys.modules['paper_2602_15318_amd._native'] = None"])
def test_a_native_part_that_does_not_fit_is_not_used(prepare):
    """Built for another torch, or not there: the general code takes every call, and the import says so."""
    out, err = _python(prepare + """
import types
import numpy as np, torch
import paper_2602_15318_amd as sp
z, one = torch.zeros(1, 4, 64), np.array([0, 1], np.int32)
try:
    sp.draft_window_attn(z, z, z, one, torch.zeros(1, dtype=torch.int32), one, -1, stream=types.SimpleNamespace(cuda_stream=0))
except sp.SparrowError as e:
    print(e)
""")
    assert "window = -1 must be positive" in out[0]
    assert "RuntimeWarning" in err and "python -m paper_2602_15318_amd.build" in err


def _flat(r):
    if isinstance(r, dict):
        return [x for k in sorted(r) for x in (k, r[k])]
    return list(r) if isinstance(r, tuple) else [r]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("name", NAMES)
def test_both_routes_agree(name, dtype, monkeypatch):
    taken = []

    class Spy:
        def __getattr__(self, n):
            def f(*a):
                r = getattr(native, n)(*a)
                taken.append(r is not NotImplemented)
                return r
            return f

    native = binding._native
    calls = [({}, _calls("cuda", dtype)[name])]
    if name == "verify_attn":
        a = calls[0][1]
        out, lse = torch.empty_like(a[0]), torch.empty(a[0].shape[:2], device="cuda")
        trees = torch.tensor([[-1, 0, 0, 7], [-1, -1, 1, 7]], dtype=torch.int32, device="cuda")[:, :3]
        calls += [({"want_lse": False}, a), ({"out": out, "lse": lse, "scale": 0.5}, a), ({}, [*a[:4], trees, a[5]]),
                  ({}, [*a[:4], None, a[5]]), ({"workspace": torch.empty(1 << 22, dtype=torch.uint8, device="cuda")}, a),
                  ({"stream": torch.cuda.current_stream()}, a)]
    for kw, args in calls:
        results = []
        for part in (Spy(), GENERAL):
            monkeypatch.setattr(binding, "_native", part)
            r = getattr(sp, name)(*args, **kw)
            torch.cuda.synchronize()
            kept = [x.clone() if isinstance(x, torch.Tensor) else x for x in _flat(r)]
            if name == "draft_qkv_append":
                kept += [args[-2].clone(), args[-1].clone()]
            results.append((type(r), kept))
        assert taken[-1] and results[0][0] is results[1][0]
        assert len(results[0][1]) == len(results[1][1])
        for x, y in zip(results[0][1], results[1][1]):
            if isinstance(x, torch.Tensor):
                assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y), (name, kw)
            else:
                assert x == y
    # refusals: the same exception by either route
    base = calls[0][1]
    bad = [[*base[:i], x, *base[i + 1:]] for _, i, x in _odd_forms(name, base) if not isinstance(x, (list, np.integer, Sub))]
    if name == "verify_attn":
        bad.append([*base[:5], 65])                      # the library's own refusal
    if name in ("hsr_fc", "draft_qkv_append"):
        bad.append([torch.zeros(base[0].numel() + 1, dtype=dtype, device="cuda")[1:].view(base[0].shape), *base[1:]])
    for args in bad:
        said = []
        for part in (native, GENERAL):
            monkeypatch.setattr(binding, "_native", part)
            try:
                getattr(sp, name)(*args)
                said.append(None)
            except (ValueError, TypeError, sp.SparrowError) as e:
                said.append((type(e), str(e)))
        torch.cuda.synchronize()
        assert said[0] == said[1], said
