"""The argument checks of the Python binding's per-call functions: what they
refuse, with which error, and that buffers passed in are the ones returned."""

import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
dptq = pytest.importorskip("paper_2606_12487_amd")


@pytest.mark.parametrize("call,error,text", [
    (lambda: dptq.rotate_quant(1, 8, 4), TypeError, "x must be a torch.Tensor"),
    (lambda: dptq.rotate_quant(torch.zeros(2, 8), 8, 4), TypeError,
     "x must have dtype torch.float16, got torch.float32"),
    (lambda: dptq.kv_quant(torch.zeros(2, 8).half()), ValueError, "kv must be a GPU tensor"),
    (lambda: dptq.qlinear(torch.zeros(2, 8), None, 5, None, None), ValueError, "bits must be 4 or 8"),
    (lambda: dptq.qlinear(torch.zeros(2, 8), None, 4.5, None, None), ValueError, "bits must be 4 or 8"),
    (lambda: dptq.qlinear_fp6(None, None, None, None, 3, 100, 16), ValueError,
     "no FP6 layout for rows=3, K=100"),
])
def test_refusals(call, error, text):
    dptq.lib()
    with pytest.raises(error, match=text.replace("(", r"\(")):
        call()


# Tensors without storage (function transforms wrap theirs), on fake GPU tensors
# and a fixed stream so that no GPU is needed.  In a process of its own: an
# exception that leaves the native call without the interpreter lock ends it.
_NO_STORAGE = """
import torch, paper_2606_12487_amd as dptq
from torch._subclasses import FakeTensorMode
dptq._binding().init(dptq._check, lambda device: 0)
with FakeTensorMode():
    empty = lambda dtype, *shape: torch.empty(shape, dtype=dtype, device="cuda")
    x, s, w = empty(torch.float16, 3, 128), empty(torch.float32, 3), empty(torch.uint8, 16, 64)
    c, ws, y = empty(torch.uint8, 3, 64), empty(torch.float32, 16), empty(torch.float16, 3, 16)
    a6, w6 = empty(torch.uint8, 3072), empty(torch.uint8, 3072)
    calls = [
        lambda: torch.vmap(lambda r: dptq.rotate_quant(r, 128, 4, c, s))(x[None]),
        lambda: torch.func.vjp(lambda r: dptq.rotate_quant(r, 128, 4)[1], x),
        lambda: torch.func.vjp(lambda r: dptq.rotate_quant_fp6(r, 128)[1], x),
        lambda: torch.func.vjp(lambda r: dptq.rotate_quant_range(r, 128, 8)[1], x),
        lambda: torch.func.vjp(lambda r: dptq.qlinear(c, r, 4, w, ws), s),
        lambda: torch.func.vjp(lambda r: dptq.qlinear_fp6(a6, r, w6, ws, 3, 128, 16, y), s),
        lambda: torch.func.vjp(lambda r: dptq.qlinear_decode_fused(r, 128, 4, w, ws)[0], x),
        lambda: torch.func.vjp(lambda r: dptq.residual_dynamics(x, r, 128)[0], x),
        lambda: torch.func.vjp(lambda r: dptq.kv_quant(r)[1], x),
    ]
    for call in calls:
        try:
            call()
            print("no error")
        except RuntimeError as e:
            print(e)
"""


def test_tensors_without_storage_raise():
    r = subprocess.run([sys.executable, "-c", _NO_STORAGE], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
    lines = [line for line in r.stdout.splitlines() if line]
    assert lines == ["Cannot access data pointer of Tensor that doesn't have storage"] * 9, r.stdout


# Arguments that are no plain integers: what the checks refuse, and what reaches
# the library (which refuses the null pointers of fake tensors: status 1).
_NUMBERS = """
import torch, numpy as np, paper_2606_12487_amd as dptq
from torch._subclasses import FakeTensorMode
dptq._binding().init(dptq._check, lambda device: 0)
with FakeTensorMode():
    empty = lambda dtype, *shape: torch.empty(shape, dtype=dtype, device="cuda")
    x, s, w = empty(torch.float16, 3, 128), empty(torch.float32, 3), empty(torch.uint8, 16, 64)
    c, c8, m = empty(torch.uint8, 3, 64), empty(torch.int8, 3, 128), empty(torch.float32, 3, 1)
    ws, z, y, zw = empty(torch.float32, 16), empty(torch.int32, 3), empty(torch.float16, 3, 16), empty(torch.int32, 16)
    a6, w6 = empty(torch.uint8, 3072), empty(torch.uint8, 3072)
    for call in [
        lambda: dptq.kv_quant(x, 128.5), lambda: dptq.kv_quant(x, "128"), lambda: dptq.kv_quant(x, 128.0),
        lambda: dptq.kv_quant(x, 128.0, c, m, m), lambda: dptq.kv_quant(x, np.int64(128)),
        lambda: dptq.kv_dequant(c, m, m, 128.5), lambda: dptq.kv_dequant(c, m, m, np.float32(128)),
        lambda: dptq.qlinear_fp6(a6, s, w6, ws, 3.0, 128, 16, y),
        lambda: dptq.qlinear_fp6(a6, s, w6, ws, 3, "128", 16, y),
        lambda: dptq.qlinear_range(c, s, z, 4.5, w, ws, zw), lambda: dptq.qlinear_range(c8, s, z, 8.0, w, ws, zw),
        lambda: dptq.rotate_quant_range(x, 128, 4.5, c), lambda: dptq.qlinear_decode_fused(x, 128, None, w, ws, y, c),
        lambda: dptq.rotate_quant(x, 128, 2**70),
        lambda: dptq.residual_dynamics(x, x, 128, 4, "1e-8"),
    ]:
        try:
            call()
            print("no error")
        except Exception as e:
            print(type(e).__name__, getattr(e, "status", ""))
"""


def test_numbers_accepted_and_refused():
    r = subprocess.run([sys.executable, "-c", _NUMBERS], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
    assert [line.strip() for line in r.stdout.splitlines()] == [
        "ValueError", "TypeError", "TypeError", "DptqError 1", "DptqError 1", "ValueError", "DptqError 1",
        "TypeError", "TypeError", "TypeError", "DptqError 1", "TypeError", "TypeError", "ValueError",
        "DptqError 1"], r.stdout


# An allocator that counts the allocations made with the interpreter lock held.
_ALLOCATOR = r"""
#include <sys/types.h>
extern "C" {
int hipMalloc(void**, size_t);
int hipFree(void*);
int PyGILState_Check(void);
int held = 0, calls = 0;
void* counting_malloc(ssize_t size, int, void*) {
  void* p = nullptr;
  ++calls;
  held += PyGILState_Check();
  return hipMalloc(&p, size) == 0 ? p : nullptr;
}
void counting_free(void* p, ssize_t, int, void*) { (void)hipFree(p); }
}
"""
_COUNT = """
import ctypes, sys, torch, paper_2606_12487_amd as dptq
a = torch.cuda.memory.CUDAPluggableAllocator(sys.argv[1], "counting_malloc", "counting_free")
torch.cuda.memory.change_current_allocator(a)
L = ctypes.CDLL(sys.argv[1])
held, calls = (ctypes.c_int.in_dll(L, n) for n in ("held", "calls"))
x = torch.zeros((3, 128), dtype=torch.float16, device="cuda")
w = torch.zeros((16, 64), dtype=torch.uint8, device="cuda")
ws = torch.zeros((16,), device="cuda")
dptq.rotate_quant(x, 128, 4)   # loads the binding
held.value = calls.value = 0
c, s = dptq.rotate_quant(x, 128, 4)
y = dptq.qlinear(c, s, 4, w, ws)
kv = dptq.kv_quant(x)
torch.cuda.synchronize()
print(calls.value, held.value)
"""


@pytest.mark.gpu
def test_outputs_are_allocated_without_the_interpreter_lock(tmp_path):
    src, lib = tmp_path / "alloc.cpp", tmp_path / "alloc.so"
    src.write_text(_ALLOCATOR)
    hip = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", str(lib), "-L" + hip, "-lamdhip64",
                    "-Wl,-rpath," + hip, "-Wl,--unresolved-symbols=ignore-all"], check=True, timeout=60)
    r = subprocess.run([sys.executable, "-c", _COUNT, str(lib)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, (r.stdout, r.stderr[-2000:])
    assert r.stdout.split() == ["6", "0"], r.stdout


@pytest.mark.gpu
def test_buffers_shapes_and_statuses():
    x = torch.randn(3, 256, device="cuda").half()
    codes = torch.empty((3, 128), dtype=torch.uint8, device="cuda")
    scales = torch.empty((3,), device="cuda")
    c, s = dptq.rotate_quant(x, 256, 4, codes, scales)
    assert c is codes and s is scales
    c2, s2 = dptq.rotate_quant(x, had_size=256, bits=4)
    assert torch.equal(c2, codes) and torch.equal(s2, scales)
    with pytest.raises(ValueError, match=r"codes must have shape \(3, 256\), got \(3, 128\)"):
        dptq.rotate_quant(x, 256, 8, codes.view(torch.int8))
    with pytest.raises(ValueError, match=r"scales must have shape \(3,\), got \(4,\)"):
        dptq.rotate_quant(x, 256, 4, codes, torch.empty((4,), device="cuda"))
    with pytest.raises(ValueError, match="x must be contiguous"):
        dptq.rotate_quant(torch.randn(256, 3, device="cuda").half().t(), 256, 4)
    with pytest.raises(ValueError, match="x must be 2-D"):
        dptq.rotate_quant(x[0], 256, 4)
    with pytest.raises(dptq.DptqError) as e:
        dptq.rotate_quant(x, 100, 4)
    assert e.value.status == 1
    # a side stream's work is ordered by that stream
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        c3, s3 = dptq.rotate_quant(x, 256, 4)
    side.synchronize()
    assert torch.equal(c3, codes) and torch.equal(s3, scales)
