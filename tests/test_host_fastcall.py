"""The binding's native marshaling (csrc/fs_fastcall.c) against ctypes' conversions, on the CPU: its entry points are
callbacks that record what arrives, torch's current device and stream stand-ins; what it does not take, it answers None to."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2509_06261_amd as fs
from paper_2509_06261_amd import _fsfast, binding

vp, i32, i64, u64, f32 = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_uint64, ctypes.c_float
SIGNATURES = [("kv_append", [vp, i32, i32, vp, vp, i32, vp, vp, vp, i32, i64, vp]), ("kv_append_multi", [vp, vp, i32, vp]),
              ("decode_attention", [vp, i32, i32, i32, f32, vp, vp, vp, i32, i32, vp, vp, vp, u64, vp]),
              ("decode_attention_multi", [vp, vp, i32, vp, u64, vp]), ("decode_step_multi", [vp, vp, i32, vp, i32, vp, u64, vp])]
STREAM = 0x5EED0


@pytest.fixture(scope="module")
def got():
    """The recorders take the place of the library's entry points in the whole process, so the binding's own calls keep to
    ctypes meanwhile; afterwards the module forgets them and the binding starts anew."""
    seen = {}
    slow, binding._slow, binding._fast = binding._slow, lambda: None, binding._NotYet

    def recorder(name, types):
        def f(*args):
            seen[name] = list(args)
            for k, t in (("kv_append_multi", {1: binding.fs_append_t}), ("decode_attention_multi", {1: binding.fs_batch_t}),
                         ("decode_step_multi", {1: binding.fs_append_t, 3: binding.fs_batch_t})):
                if k == name:
                    for at, c in t.items():  # (the structures live for the call only)
                        seen[name][at] = ctypes.string_at(args[at], args[at + 1] * ctypes.sizeof(c)) if args[at + 1] else b""
            return 7
        return ctypes.CFUNCTYPE(i32, *types)(f)

    seen["keep"] = [recorder(*x) for x in SIGNATURES]
    _fsfast.init(torch.Tensor, torch.float16, torch.float32, torch.int32, ctypes.c_void_p, binding.fs_batch_t, binding.fs_append_t,
                 lambda: 3, lambda d: STREAM + d, *[ctypes.cast(f, vp).value for f in seen["keep"]])
    yield seen
    _fsfast.init()
    binding._slow = slow


def rows(dt=torch.float16):
    k, v = torch.zeros((5, 2, 8), dtype=dt), torch.zeros((5, 2, 8), dtype=dt)
    return [k, v, torch.zeros(5, dtype=torch.int32), torch.zeros(5, dtype=torch.int32), torch.zeros((3, 4), dtype=torch.int32)]


@pytest.mark.parametrize("dt", [torch.float16, torch.float32])
def test_append(got, dt):
    pool, r = vp(0x1234567890), rows(dt)
    assert _fsfast.kv_append(pool, 1, 2, *r, None) == 7
    k, v, s, p, t = [x.data_ptr() for x in r]
    assert got["kv_append"] == [pool.value, 1, 2, k, v, fs.FS_SRC_FP32 if dt == torch.float32 else fs.FS_SRC_FP16, s, p, t, 4, 5, STREAM + 3]
    appends = [fs.make_append(1, 2, *r), fs.make_append(3, 4, *r)]
    assert _fsfast.kv_append_multi(pool, appends, None) == 7
    assert got["kv_append_multi"] == [pool.value, b"".join(bytes(a) for a in appends), 2, STREAM + 3]


def test_append_leaves_the_unusual_to_ctypes(got):
    r = rows()
    for k, bad in ((0, r[0].double()), (0, r[0].float()), (1, r[1].transpose(1, 2)), (2, r[2].long()), (3, np.zeros(5, np.int32)), (4, r[4].T),
                   (4, torch.zeros(4, dtype=torch.int32)), (2, None), (0, torch.nn.Parameter(r[0]))):
        x = list(r)
        x[k] = bad
        assert _fsfast.kv_append(vp(1), 1, 2, *x, None) is None, k
    assert _fsfast.kv_append(0x1234, 1, 2, *r, None) is None  # (a raw address as the pool, a stream, numpy's integers: ctypes' business)
    assert _fsfast.kv_append(vp(1), np.int32(1), 2, *r, None) is None
    assert _fsfast.kv_append(vp(1), 1 << 40, 2, *r, None) is None
    assert _fsfast.kv_append(vp(1), 1, 2, *r, STREAM) is None
    with pytest.raises(AssertionError):
        fs.fs_kv_append(vp(1), 1, 2, r[0], r[1].float(), *r[2:])


def test_decode(got):
    q, t, n = torch.zeros((3, 4, 64), dtype=torch.float16), torch.zeros((3, 9), dtype=torch.int32), torch.zeros(3, dtype=torch.int32)
    out, lse, ws = torch.zeros_like(q), torch.zeros((3, 4)), torch.zeros(1000, dtype=torch.int32)
    for l in (lse, None):
        assert _fsfast.decode_attention(vp(5), 1, 2, 4, 0.125, q, t, n, out, l, ws, None) == 7
        assert got["decode_attention"] == [5, 1, 2, 4, 0.125, q.data_ptr(), t.data_ptr(), n.data_ptr(), 3, 9, out.data_ptr(),
                                           None if l is None else l.data_ptr(), ws.data_ptr(), 4000, STREAM + 3]
    batches = [fs.make_batch(k, 2, 4, 0.125, q, t, n, out, lse, np.array([1, 2, 3], np.int32)) for k in range(8)]
    assert _fsfast.decode_attention_multi(vp(5), batches, ws, None) == 7
    assert got["decode_attention_multi"] == [5, b"".join(bytes(b) for b in batches), 8, ws.data_ptr(), 4000, STREAM + 3]
    a = [fs.make_append(1, 2, *rows())]
    for appends in (a, []):
        assert _fsfast.decode_step_multi(vp(5), appends, batches[:2], ws, None) == 7
        assert got["decode_step_multi"] == [5, b"".join(bytes(x) for x in appends), len(appends), b"".join(bytes(b) for b in batches[:2]), 2,
                                            ws.data_ptr(), 4000, STREAM + 3]
    assert _fsfast.decode_attention_multi(vp(5), batches + batches[:1], ws, None) is None
    assert _fsfast.decode_attention_multi(vp(5), tuple(batches), ws, None) is None
    assert _fsfast.decode_attention_multi(vp(5), a, ws, None) is None
    assert _fsfast.decode_attention(vp(5), 1, 2, 4, 1, q, t, n, out, lse, ws, None) is None
    assert _fsfast.decode_attention(vp(5), 1, 2, 4, 0.125, q, n, n, out, lse, ws, None) is None


def test_nothing_is_left_behind():
    """After this module's tests no call reaches their recorders (a child process runs them, then calls)."""
    code = """
import ctypes, sys, pytest
assert pytest.main([sys.argv[1], "-q", "-p", "no:cacheprovider", "-k", "append or decode"]) == 0
from paper_2509_06261_amd import _fsfast, binding
import torch
r = [torch.zeros((5, 2, 8), dtype=torch.float16)] * 2 + [torch.zeros(5, dtype=torch.int32)] * 2 + [torch.zeros((3, 4), dtype=torch.int32)]
assert _fsfast.kv_append(ctypes.c_void_p(1), 1, 2, *r, None) is None
assert binding._fast is binding._NotYet and binding._slow.__name__ == "_slow"
"""
    p = subprocess.run([sys.executable, "-c", code, __file__], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-2000:]


def test_package_without_the_module():
    """Not built for the interpreter, the module is done without: every call goes through ctypes."""
    code = """
import ctypes, sys
if sys.argv[1] == "without":
    sys.modules["paper_2509_06261_amd._fsfast"] = None
import paper_2509_06261_amd as fs
from paper_2509_06261_amd import binding
assert (binding._fsfast is None) == (sys.argv[1] == "without")
try:
    fs.fs_kv_append_multi(None, [binding.fs_append_t()], stream=0)
    raise SystemExit("a call without a pool was taken")
except fs.FsError:
    pass
assert binding._fast is binding._NotYet
"""
    for which in ("with", "without"):
        p = subprocess.run([sys.executable, "-c", code, which], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True, timeout=300)
        assert p.returncode == 0, which + p.stdout[-2000:] + p.stderr[-2000:]
