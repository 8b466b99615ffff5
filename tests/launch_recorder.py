"""Which kernels the library launches for a call, found on the CPU: the calls run in a child process against
launch_recorder.c in the place of the HIP runtime, with made-up device addresses that nothing reads.

A call is a dict: {"call": "verify", "dtype", "Hq", "Hkv", "d", "n_q", "lens", "layout", "own"} (dtype: bf16 or f32; lens: rows of each sequence,
draft rows included; layout: "token", "head" or "pair", as kv_strides says; own: a tree per sequence; workspace: its bytes), or
{"call": "accept" | "topk", "dtype", "M", "H", "V"}."""
import ctypes
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2602_15318_amd", "libsparrow.so")
MAX_BATCH = 64


def kv_strides(layout, T, Hkv, d):
    """(stride of a token, of a head) in elements: [T, Hkv, d], [Hkv, T, d] or K and V rows side by side [Hkv, T, 2, d]."""
    return {"token": (Hkv * d, d), "head": (d, T * d), "pair": (2 * d, 2 * T * d)}[layout]


def record(calls, tmp):
    """The launches of every call, in order: {"kernel", "grid", "block", "lds"}; for the partial pass of verification
    on the matrix cores also "splits" and "pieces" (per sequence) and "flat" (bf16), for its combine pass "splits" (of the
    first sequence) and "units" (KV heads x blocks of 64 rows)."""
    shim = os.path.join(str(tmp), "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "launch_recorder.c")], check=True)
    if not os.path.exists(LIB):
        from paper_2602_15318_amd import build
        build.build()
    res = subprocess.run([sys.executable, os.path.abspath(__file__), shim], input=json.dumps(calls), text=True,
                         capture_output=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    return json.loads(res.stdout.splitlines()[-1])


class _Desc(ctypes.Structure):
    _fields_ = [("dtype", ctypes.c_int32), ("n_q_heads", ctypes.c_int32), ("n_kv_heads", ctypes.c_int32),
                ("head_dim", ctypes.c_int32), ("scale", ctypes.c_float), ("kv_stride_token", ctypes.c_int64),
                ("kv_stride_head", ctypes.c_int64), ("parent_stride", ctypes.c_int32)]


def _child(shim):
    rec = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)       # found before the HIP runtime that the library names
    lib = ctypes.CDLL(LIB)
    vp, i32, ws = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t(1 << 40)
    lib.sparrow_last_error.restype = ctypes.c_char_p
    names = {}
    each = ctypes.CFUNCTYPE(None, vp, ctypes.c_char_p)(lambda stub, name: names.__setitem__(stub, name.decode()))
    rec.recorder_kernels(each)
    assert names, "the library did not register its kernels with the recorder"
    plain = subprocess.run(["c++filt"], input="\n".join(names.values()), text=True, capture_output=True, check=True)
    names = {stub: re.sub(r"^void |sparrow::|\(anonymous namespace\)::|\(.*$", "", full.replace("(anonymous namespace)::", ""))
             for stub, full in zip(names, plain.stdout.splitlines())}
    seen = []

    def on_launch(stub, grid, block, lds, args):
        one = {"kernel": names[stub], "grid": list(grid[:3]), "block": list(block[:3]), "lds": lds}
        if one["kernel"].startswith("verify_partial_mfma_kernel"):      # (ten scalars, the last one "shape"; VerifyArgs, SeqTable, PieceTable)
            table = ctypes.cast(args[11], ctypes.POINTER(i32))
            B = next(b for b in range(1, MAX_BATCH + 1) if b == MAX_BATCH or table[b + 1] == 0)
            cu = table[MAX_BATCH + 1:MAX_BATCH + 2 + B]
            one["splits"] = [y - x for x, y in zip(cu, cu[1:])]
            one["pieces"] = ctypes.cast(args[12], ctypes.POINTER(i32))[:B]
            one["flat"] = bool(ctypes.cast(args[9], ctypes.POINTER(i32))[0] & 1)
        if re.match("verify_combine_(tiled|few|long)_kernel", one["kernel"]):     # (four pointers, splits, units, ...)
            one["splits"], one["units"] = (ctypes.cast(args[i], ctypes.POINTER(i32))[0] for i in (4, 5))
        seen.append(one)

    p32 = ctypes.POINTER(ctypes.c_uint32)
    hook = ctypes.CFUNCTYPE(None, vp, p32, p32, ctypes.c_size_t, ctypes.POINTER(vp))(on_launch)
    rec.recorder_on_launch(hook)
    at = vp(1 << 32)                                        # stands for any device address
    out = []
    for c in json.load(sys.stdin):
        del seen[:]
        if c["call"] == "verify":
            B, n_q, lens = len(c["lens"]), c["n_q"], c["lens"]
            st, sh = kv_strides(c.get("layout", "token"), sum(lens), c["Hkv"], c["d"])
            desc = _Desc({"f32": 0, "bf16": 1}[c.get("dtype", "bf16")], c["Hq"], c["Hkv"], c["d"], 0.0, st, sh, n_q if c.get("own") else 0)
            cu = (i32 * (B + 1))(*[sum(lens[:b]) for b in range(B + 1)])
            rc = lib.sparrow_verify_attn(ctypes.byref(desc), at, at, at, cu, at, B, n_q, at, at, at,
                                         ctypes.c_size_t(c["workspace"]) if "workspace" in c else ws, None)
        else:
            code = {"f32": 0, "bf16": 1}[c["dtype"]]
            if c["call"] == "accept":                       # M sequences without draft rows
                rc = lib.sparrow_accept(code, at, at, at, None, c["M"], 0, c["H"], c["V"], at, at, at, at, at, ws, None)
            else:
                rc = lib.sparrow_draft_topk(code, at, at, c["M"], c["H"], c["V"], 4, at, at, at, ws, None)
        assert rc == 0, (c, lib.sparrow_last_error())
        out.append(list(seen))
    print(json.dumps(out))


if __name__ == "__main__":
    _child(sys.argv[1])
