"""The native short way of the binding over entry points for host memory: what reaches them, and what becomes of tensors that have no
storage and of entry points that raise.  Each in a process of its own, so that one that ends says so."""
import subprocess
import sys
import textwrap

import pytest

from paper_2310_05218_amd import build

pytest.importorskip("torch")

SETUP = """
import ctypes, importlib.util, shutil, tempfile
import torch
from paper_2310_05218_amd import binding

folder = tempfile.mkdtemp()         # a copy of the module: its own bindings
spec = importlib.util.spec_from_file_location("_swnative", shutil.copy({so!r}, folder + "/_swnative.so"))
native = importlib.util.module_from_spec(spec)
shutil.rmtree(folder)
seen = []

@ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * 3, *[ctypes.c_int] * 9, ctypes.c_void_p)
def conv2d(*a):
    seen.append(a)
    return 0

native.bind((ctypes.cast(conv2d, ctypes.c_void_p).value,) * len(binding._NATIVE_ENTRIES), True)
run = lambda x, w: native.run(binding._CONV2D, x, w, None, None, 2, 1)
x, w = torch.randn(2, 8, 12, 14), torch.randn(16, 8, 3, 3)
"""


def child(code):
    r = subprocess.run([sys.executable, "-c", SETUP.format(so=build.BINDING) + textwrap.dedent(code)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"status {r.returncode}\n{r.stdout}\n{r.stderr}"


def test_plain_call():
    child("""
    y = run(x, torch.nn.Parameter(w))
    assert y.shape == (2, 16, 6, 7) and y.dtype == torch.float32 and not y.requires_grad
    assert seen == [(x.data_ptr(), w.data_ptr(), y.data_ptr(), 2, 8, 16, 12, 14, 3, 3, 2, 1, None)]
    assert run(x, w.to("meta")) is None and run(x.double(), w) is None and len(seen) == 1
    """)


def test_tensors_without_storage_are_not_taken():
    """Transformed tensors are plain ones on the same device to every test but that for their memory, which raises."""
    child("""
    got = []
    def f(a, b):
        got.append(run(a, b))
        return a
    torch.vmap(f)(x[None], w[None])
    torch.vmap(f, in_dims=(None, 0))(x, w[None])
    torch.func.vmap(torch.func.vmap(f))(x[None, None], w[None, None])
    torch.func.grad(lambda a: f(a, w).sum())(x)
    torch.func.jvp(f, (x, w), (x, w))
    assert got == [None] * 5 and not seen, got
    assert run(x, w).shape == (2, 16, 6, 7) and len(seen) == 1      # (and the interpreter goes on)
    """)
