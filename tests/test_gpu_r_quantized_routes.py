"""fp8q_gemm_quantized gives the bytes of fp8q_quantize on fp8q_gemm's output
wherever fp8q_gemm sums its K blocks in another order than one after another
(the thin tiles are held to it beside their other tests).

* Two K groups: ragged rows, an even and an odd 1024-column band (the second
  walks K backwards), the fewest K blocks and several rounds of the ring.
* A bf16 output of 2 GiB, which fp8q_gemm cuts so that its last 256 rows take
  another kernel than the rest."""
import pytest
import torch

import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

from _routes import route

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
B1, B128 = fp8q.BLOCK_1x128, fp8q.BLOCK_128x128


def check(M, K, N, seed):
    A, sA = fp8q.quantize(synth.activations(M, K, seed=seed, outlier_seed=seed + 1, device=DEV), B1)
    B, sB = fp8q.quantize(synth.weights(N, K, seed=seed + 2, device=DEV), B128)
    codes, scales = fp8q.gemm_quantized(A, sA, B1, B, sB, B128)
    want, ws = fp8q.quantize(fp8q.gemm(A, sA, B1, B, sB, B128), B1)
    assert torch.equal(codes, want) and torch.equal(scales, ws)


@pytest.mark.parametrize("shape", [(64, 4096, 12288), (128, 4096, 6144), (190, 5120, 5120), (256, 4096, 4096)])
def test_where_gemm_takes_k_groups(shape):
    print("quantized output, K groups", shape, flush=True)
    assert route("block", *shape) == "two K groups"
    check(*shape, seed=1201)


def test_where_gemm_cuts_its_output():
    M, K, N = 1 << 18, 256, 4096
    print("quantized output, output cut at 2 GiB", flush=True)
    assert route("block", 256, K, N) == "two K groups" and route("block", M - 256, K, N) in ("large", "mid")
    check(M, K, N, seed=1211)
