"""The binding's native marshalling on the CPU: a second copy of the module, bound to stand-ins of
the library's functions and to CPU tensors.  A tensor without storage (what a function transform
hands in) is refused before the call, so that the Python path raises its error.  Run in a
process of its own, with a second thread busy, so that a lost thread state shows as a crash."""
import os
import subprocess
import sys

import pytest

from paper_2608_21952_amd import build as libbuild

PROGRAM = r"""
import ctypes, importlib.machinery, importlib.util, shutil, sys, tempfile, threading
import torch

path = shutil.copy(sys.argv[1], tempfile.mkdtemp())
loader = importlib.machinery.ExtensionFileLoader("_binding", path)
native = importlib.util.module_from_spec(importlib.util.spec_from_loader("_binding", loader))
loader.exec_module(native)
calls = []
i64, ptr, i32 = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
quant = ctypes.CFUNCTYPE(i32, ptr, i32, i64, i64, i64, i64, i32, ptr, i32, ptr, ptr)(
    lambda *a: calls.append("quantize") or 0)
size = ctypes.CFUNCTYPE(ctypes.c_size_t, ptr)(lambda d: 64)
scan = ctypes.CFUNCTYPE(i32, ptr, ptr, ptr)(lambda *a: calls.append("scan") or 0)
decode = ctypes.CFUNCTYPE(i32, i64, i64, i64, i64, i64, ptr, ptr)(
    lambda *a: calls.append("decode") or 0)
native.bind(*(ctypes.cast(f, ptr).value for f in (quant, size, scan, decode)), "cpu")

stop = threading.Event()
def spin():
    while not stop.is_set():
        sum(range(100))
other = threading.Thread(target=spin)
other.start()

f = lambda *s: torch.ones(*s)
q = lambda *s: torch.ones(*s, dtype=torch.int8)
B, L, H, G = 2, 256, 3, 1
entries = {
    "quantize": (f(B, L, G, 128), lambda x: native.quantize(x, 1, None, None, 0)),
    "quantize_scale": (f(G), lambda s: native.quantize(f(B, L, G, 128), 1, s, None, 0)),
    "scan": (f(B, L, H, 64), lambda x: native.scan(
        x, f(B, L, H), f(H), q(B, L, G, 128), q(B, L, G, 128), None, None, f(G), f(G), f(H, 64),
        f(H, 64), f(G), None, None, None, None, -1, None, None, 1, 256, 7, 1, 1, 0, 0)),
    "decode": (f(B, H, 64), lambda x: native.decode(
        x, f(B, H), f(H), q(B, G, 128), q(B, G, 128), f(G), f(G), f(H, 64), f(H, 64), f(G),
        q(B, H, 64, 128), None, None, 1, 7, 1, None, -1, 0)),
}
for name, (arg, call) in entries.items():
    print(name, flush=True)
    out = []
    def transformed(t):
        out.append(call(t))
        return t.sum()
    calls.clear()
    if sys.argv[2] == "plain":
        transformed(arg)
        assert out[0] is not None and out[0][0] == 0, out
        assert calls == [name.split("_")[0]], calls
    else:
        if sys.argv[2] == "vmap":
            torch.func.vmap(transformed)(torch.stack([arg, arg]))
        else:
            torch.func.grad(transformed)(arg)
        assert out == [None] and not calls, (out, calls)
stop.set()
other.join()
print("done")
"""


@pytest.mark.parametrize("how", ["plain", "vmap", "grad"])
def test_tensors_without_storage_go_to_the_python_path(how):
    if not os.path.exists(libbuild.BINDING):
        libbuild.build()
    r = subprocess.run([sys.executable, "-c", PROGRAM, libbuild.BINDING, how],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), \
        (r.returncode, r.stdout[-500:], r.stderr[-2000:])
