"""The binding's two routes: ordinary calls go through the native code
(csrc/binding.cpp), any other through the Python code.  Both must make the
same library call: a tensor subclass (which the native code leaves alone)
gives the same bytes as a plain tensor through every entry point, on a stream
of its own too, and both routes report a refused call and a wrong buffer
alike.  The native functions are counted: they take every call of a plain
tensor and none of a subclass."""
import pytest
import torch

import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
B1, B128 = fp8q.BLOCK_1x128, fp8q.BLOCK_128x128


class Sub(torch.Tensor):
    pass


def calls(wrap):
    """Every entry point's outputs, its tensor arguments passed through wrap."""
    x = wrap(synth.activations(200, 512, seed=601, outlier_seed=602, device=DEV))
    w = wrap(synth.weights(256, 512, seed=603, device=DEV))
    d = wrap(synth.grads(256, 512, seed=604, device=DEV))
    out = {}
    for g in (fp8q.TENSOR, fp8q.ROW, fp8q.COL, B1):
        out["quantize", g] = fp8q.quantize(x, g)
    out["transposed"] = fp8q.quantize(w, B128, transposed=True)
    codes = torch.full((200, 640), 9, dtype=torch.uint8, device=DEV)
    out["given"] = fp8q.quantize(x, B1, codes=wrap(codes[:, :512])) + (codes,)
    out["dual"] = fp8q.quantize_dual(d, e5m2=True)
    a, b = [[wrap(t) for t in q] for q in (fp8q.quantize(x, B1), fp8q.quantize(w, B128))]
    out["gemm"] = (fp8q.gemm(*a, B1, *b, B128),)
    buf = torch.full((200, 260), 3.0, dtype=torch.bfloat16, device=DEV)
    fp8q.gemm(*a, B1, *b, B128, out=wrap(buf[:, :256]))
    out["out"] = (buf,)
    out["formats"] = (fp8q.gemm_formats(*a, B1, *b, B128, fp8q.B_E5M2),)
    out["splitk"] = (fp8q.gemm_splitk(*a, B1, *b, B128),)
    ws = torch.zeros(fp8q.gemm_splitk_workspace(200, 256, 512) + 16, dtype=torch.uint8, device=DEV)
    out["splitk ws"] = (fp8q.gemm_splitk(*a, B1, *b, B128, workspace=wrap(ws)),)
    out["quantized"] = fp8q.gemm_quantized(*a, B1, *b, B128)
    out["grouped"] = fp8q.gemm_grouped([(*a, *b), (*a, *b)], B1, B128)
    p, q = [[wrap(t) for t in z] for z in (fp8q.quantize(x, B1, pow2=True), fp8q.quantize(w, B128, pow2=True))]
    out["pow2"] = (fp8q.gemm_pow2(*p, B1, *q, B128),)
    r = {k: wrap(v) for k, v in synth.rl_batch(2, 8, seed=605, device=DEV).items()}
    out["clip"] = fp8q.calibrate_clip(*r.values(), 0.6, 1.8)
    return out


class Counted:
    """The native functions, with the calls that they took and left."""

    def __init__(self, native):
        self.native, self.took, self.left = native, [], []

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.native, name)(*args)
            (self.left if r is None else self.took).append(name)
            return r
        return call


def same(u, v):
    if isinstance(u, dict):
        return list(u) == list(v) and all(type(u[k]) is type(v[k]) and (u[k] == v[k]) for k in u)
    return len(u) == len(v) and all(s.dtype == t.dtype and s.shape == t.shape and
                                    torch.equal(s.as_subclass(torch.Tensor).contiguous().view(torch.uint8),
                                                t.as_subclass(torch.Tensor).contiguous().view(torch.uint8))
                                    for s, t in zip(u, v))


@pytest.mark.parametrize("own_stream", [False, True])
def test_routes_agree(own_stream, monkeypatch):
    counted = [Counted(fp8q._fast()), Counted(fp8q._fast())]
    with torch.cuda.stream(torch.cuda.Stream() if own_stream else torch.cuda.current_stream()):
        monkeypatch.setattr(fp8q, "_calls", counted[0])
        native = calls(lambda t: t)
        monkeypatch.setattr(fp8q, "_calls", counted[1])
        python = calls(lambda t: t.as_subclass(Sub))
        torch.cuda.synchronize()
    names = {"quantize", "quantize_dual", "gemm", "gemm_pow2", "gemm_splitk", "gemm_quantized", "gemm_grouped",
             "calibrate_clip"}
    # (without a workspace gemm_splitk is the Python code's, which makes one)
    assert set(counted[0].took) == names and counted[0].left == ["gemm_splitk"]
    assert set(counted[1].left) == names and not counted[1].took
    assert list(native) == list(python)
    for k in native:
        assert same(native[k], python[k]), k


@pytest.mark.parametrize("wrap", [lambda t: t, lambda t: t.as_subclass(Sub)], ids=["native", "python"])
def test_routes_report_alike(wrap):
    x = wrap(synth.activations(64, 512, seed=611, outlier_seed=612, device=DEV))
    a = [wrap(t) for t in fp8q.quantize(x, B1)]
    b = [wrap(t) for t in fp8q.quantize(wrap(synth.weights(256, 512, seed=613, device=DEV)), B128)]
    with pytest.raises(fp8q.Fp8qError) as e:                       # K not a multiple of 128
        fp8q.gemm(a[0][:, :96], a[1], B1, b[0][:, :96], b[1], B1)
    assert e.value.status == -2
    with pytest.raises(fp8q.Fp8qError) as e:                       # misaligned columns
        fp8q.quantize(x[:, 1:129], B1)
    assert e.value.status == -3
    with pytest.raises(ValueError, match="unsupported|invalid|shape|holds"):
        fp8q.quantize(x, B1, scales=wrap(torch.empty(7, dtype=torch.float32, device=DEV)))
    with pytest.raises(ValueError, match="contraction sizes differ"):
        fp8q.gemm(a[0], a[1], B1, b[0][:, :256], b[1], B128)
    with pytest.raises(ValueError, match="out must have shape"):
        fp8q.gemm(*a, B1, *b, B128, out=wrap(torch.empty((64, 255), dtype=torch.bfloat16, device=DEV)))
