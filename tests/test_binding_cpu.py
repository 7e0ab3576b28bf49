"""The binding's native code (csrc/binding.cpp) without a GPU: compiled with
its device check turned to CPU tensors and its stream to none, over stand-ins
for the library's entry points (the three that only compute sizes are the
library's own).

* Ordinary calls are taken (the outputs come back, the entry point ran once),
  any other is left to the Python code (None, nothing ran).
* A daemon thread whose call returns while the interpreter shuts down ends
  quietly, as in a ctypes call, and does not abort the process."""
import ctypes
import importlib.util
import os
import subprocess
import sys

import pytest
import torch

import _cbuild
import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import _build

B1, B128 = fp8q.BLOCK_1x128, fp8q.BLOCK_128x128
SIZES = ("fp8q_scales_count", "fp8q_gemm_splitk_workspace", "fp8q_calibrate_clip_workspace")


def load(path):
    spec = importlib.util.spec_from_file_location("_native", path)
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def bind(m, call):
    address = [ctypes.cast(getattr(fp8q.lib(), n) if n in SIZES else call, ctypes.c_void_p).value
               for n in fp8q._NATIVE_API]
    m.bind(tuple(address))


@pytest.fixture(scope="module")
def path(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("binding"))
    src = open(os.path.join(_build.CSRC, "binding.cpp")).read()
    stream = "return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.device().index()).stream();"
    assert src.count(".is_cuda()") == 2 and src.count(stream) == 1
    with open(os.path.join(out, "binding.cpp"), "w") as f:
        f.write(src.replace(".is_cuda()", ".is_cpu()").replace(stream, "(void)t; return nullptr;"))
    so = os.path.join(out, "_native.so")
    subprocess.check_call(_build.native_command(os.path.join(out, "binding.cpp"), so, "-O0"))
    return so


@pytest.fixture(scope="module")
def stub():
    return _cbuild.helper("binding_stub")


class Sub(torch.Tensor):
    pass


def calls(wrap):
    """(name, arguments, whether outputs are given) of an ordinary call of
    every function, its tensors passed through wrap."""
    def u8(*s):
        return wrap(torch.zeros(s, dtype=torch.uint8))

    def f32(*s):
        return wrap(torch.ones(s, dtype=torch.float32))

    def b16(*s):
        return wrap(torch.zeros(s, dtype=torch.bfloat16))

    x = b16(256, 384)
    a, sa, b, sb = u8(200, 256), f32(400), u8(128, 256), f32(2)
    gemm = (a, sa, B1, b, sb, B128)
    clip = [f32(64) for _ in range(5)] + [0.6, 1.8, 0]
    ws = u8(fp8q.lib().fp8q_calibrate_clip_workspace(64))
    return [
        ("quantize", (x, B1, 0, None, None)),
        ("quantize", (x, B128, fp8q.OUT_TRANSPOSED, u8(384, 256), f32(6))),
        ("quantize_dual", (x, 0, None, None, None, None)),
        ("quantize_dual", (x, fp8q.E5M2, u8(256, 384), f32(768), u8(384, 256), f32(768))),
        ("gemm", gemm + (0, None)),
        ("gemm", gemm + (fp8q.A_E5M2, b16(200, 128))),
        ("gemm_pow2", gemm + (None,)),
        ("gemm_splitk", gemm + (None, u8(16))),
        ("gemm_quantized", gemm + (None, None)),
        ("gemm_quantized", gemm + (u8(200, 128), f32(200))),
        ("gemm_grouped", ([(a, sa, b, sb)] * 3, B1, B128, None)),
        ("gemm_grouped", ([(a, sa, b, sb)] * 2, B1, B128, [b16(200, 128), b16(200, 128)])),
        ("calibrate_clip", tuple(clip) + (None, None, False)),
        ("calibrate_clip", tuple(clip) + (ws, u8(80), True)),
    ]


def test_ordinary_calls_are_taken(path, stub):
    m = load(path)
    bind(m, stub.stub_call)
    count = ctypes.c_int.in_dll(stub, "stub_calls")
    for name, args in calls(lambda t: t):
        count.value = 0
        r = getattr(m, name)(*args)
        assert r is not None and not isinstance(r, int) or r is True, name
        assert count.value == 1, name
        if name not in ("calibrate_clip",):
            outs = list(r) if isinstance(r, (tuple, list)) else [r]
            given = args[-1] if name == "gemm_grouped" else args[{"quantize": 3, "quantize_dual": 2, "gemm": 7,
                                                                  "gemm_pow2": 6, "gemm_splitk": 6,
                                                                  "gemm_quantized": 6}[name]:][:len(outs)]
            for o, g in zip(outs, given or [None] * len(outs)):
                assert g is None or o is g, name


def test_other_calls_are_left(path, stub):
    m = load(path)
    bind(m, stub.stub_call)
    count = ctypes.c_int.in_dll(stub, "stub_calls")
    count.value = 0
    for name, args in calls(lambda t: t.as_subclass(Sub)):
        assert getattr(m, name)(*args) is None, name
    for name, args in calls(lambda t: t):
        first = args[0][0][0] if name == "gemm_grouped" else args[0]
        for bad in (first.double(), first.t() if first.dim() == 2 else first[::2], None, 3):
            wrong = ([(bad,) + args[0][0][1:]] + args[0][1:] if name == "gemm_grouped" else bad,) + args[1:]
            assert getattr(m, name)(*wrong) is None, name
        assert getattr(m, name)(*args[:-1]) is None and getattr(m, name)(*args, None) is None, name
    assert count.value == 0


CHILD = """
import ctypes, sys, threading, time
sys.path[:0] = [%r, %r]
import torch
from test_binding_cpu import bind, load
m = load(%r)
bind(m, ctypes.CDLL(%r).stub_slow_call)
x = torch.zeros(128, 128, dtype=torch.bfloat16)
threading.Thread(target=lambda: m.quantize(x, 3, 0, None, None), daemon=True).start()
time.sleep(0.3)

class Late:                 # the shutdown lasts until the call has returned into it
    def __del__(self, sleep=time.sleep):
        sleep(1.5)

sys.late = Late()
print("shutting down", flush=True)
"""


def test_a_call_may_return_into_the_shutdown(path, stub):
    here = os.path.dirname(os.path.abspath(__file__))
    code = CHILD % (here, os.path.dirname(here), path, stub._name)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.stdout == "shutting down\n" and r.returncode == 0, (r.returncode, r.stderr)
