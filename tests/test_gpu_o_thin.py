"""Thin GEMM tiles: problems too small for the tile kernels, where every wave
takes K blocks of its own through LDS of its own and the eight waves' partial
tiles are added in wave order.  Every tile size at its edges (one row, ragged
rows and columns, fewer K blocks than waves and a remainder of them) against
the oracle, for every pair; the backward formats; the grouped launch bit for
bit against single calls; and the split-K kernel at sizes where it is still
chosen over these tiles, every split count (the elementwise bound counts the
K blocks' roundings one after another, KB of them; here a wave has KB / 8 and
at most 7 additions follow, fewer for every KB)."""
import numpy as np
import pytest
import torch

import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

from _routes import route
from test_gpu_b_gemm import PAIRS, run_pair
from test_gpu_h_grouped import check_group
from test_gpu_l_splitk import splits_of

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
B1, B128 = fp8q.BLOCK_1x128, fp8q.BLOCK_128x128
# (M, K, N): 16 x 16, 16 x 16 with one K block, 16 x 32, 32 x 32 (odd blocks), 32 x 64, 64 x 64 (K from 8192 on)
SHAPES = [(1, 1152, 512), (13, 128, 384), (30, 1024, 4096), (61, 1920, 4096), (121, 1024, 4096), (250, 8320, 4096)]


@pytest.mark.parametrize("pair", list(PAIRS))
@pytest.mark.parametrize("shape", SHAPES)
def test_thin_against_oracle(pair, shape):
    ga, gb = PAIRS[pair]
    M, K, N = shape
    if gb != B128:
        N -= 6                                   # ragged columns where the pair allows them
    assert route(pair, M, K, N) == "thin"
    a = synth.activations(M, K, seed=801, outlier_seed=802, device=DEV)
    b = synth.weights(N, K, seed=803, device=DEV)
    run_pair(a, b, ga, gb, rows=np.unique(np.append(np.arange(0, M, 1 + M // 40), M - 1)), label="thin %s" % pair,
             pad=-N % 4 or 4)


@pytest.mark.parametrize("shape", SHAPES)
def test_thin_pow2_and_formats(shape):
    """Power-of-two scales: the fp32-scale kernel on the same operands gives
    the same products (each scale product exact), so results agree to the
    roundings of the sums; E5M2 codes in A, B or both: equal to E4M3 codes
    of the same values where both formats hold them."""
    M, K, N = shape
    assert all(route(f, M, K, N) == "thin" for f in ("pow2", "block", "blockk"))
    a = synth.activations(M, K, seed=811, outlier_seed=812, device=DEV)
    b = synth.weights(N, K, seed=813, device=DEV)
    A, sA = fp8q.quantize(a, B1, pow2=True)
    B, sB = fp8q.quantize(b, B128, pow2=True)
    got, ref = fp8q.gemm_pow2(A, sA, B1, B, sB, B128).float(), fp8q.gemm(A, sA, B1, B, sB, B128).float()
    # one bf16 unit (2^-8) of the value, or of the fp32 error of cancelling sums
    assert torch.all((got - ref).abs() <= 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().amax())
    # powers of two in E4M3 and E5M2: exponent fields 1 .. 7 above each bias
    g = torch.Generator(device=DEV).manual_seed(814)
    e = torch.randint(0, 4, (M + N, K), generator=g, device=DEV, dtype=torch.uint8)
    sign = torch.randint(0, 2, (M + N, K), generator=g, device=DEV, dtype=torch.uint8) * 0x80
    e4, e5 = (0x38 + e * 8) | sign, (0x3C + e * 4) | sign
    for pair, gb in (("block", B128), ("blockk", B1)):
        sb = torch.ones(fp8q.scales_count(N, K, gb), dtype=torch.float32, device=DEV)
        sa = torch.ones(fp8q.scales_count(M, K, B1), dtype=torch.float32, device=DEV)
        want = fp8q.gemm(e4[:M], sa, B1, e4[M:], sb, gb)
        for fmt in (1, 2, 3):
            x = (e5 if fmt & 1 else e4)[:M]
            y = (e5 if fmt & 2 else e4)[M:]
            assert torch.equal(fp8q.gemm_formats(x, sa, B1, y, sb, gb, fmt), want), (pair, fmt)


@pytest.mark.parametrize("shape", SHAPES)
def test_thin_quantized_output(shape):
    """The quantized output is the quantizer's on the plain call's output,
    bit for bit (both sum in the thin tiles' order)."""
    M, K, N = shape
    assert route("quantized", M, K, N) == "thin"
    A, sA = fp8q.quantize(synth.activations(M, K, seed=841, outlier_seed=842, device=DEV), B1)
    B, sB = fp8q.quantize(synth.weights(N, K, seed=843, device=DEV), B128)
    codes = torch.full((M, N + 128), 0x55, dtype=torch.uint8, device=DEV)
    _, scales = fp8q.gemm_quantized(A, sA, B1, B, sB, B128, codes=codes[:, :N])
    want, ws = fp8q.quantize(fp8q.gemm(A, sA, B1, B, sB, B128), B1)
    assert torch.equal(codes[:, :N], want) and torch.equal(scales, ws)
    assert torch.all(codes[:, N:] == 0x55), "columns past N were written"


@pytest.mark.parametrize("M,K", [(8, 2048), (40, 384), (100, 1024)])
def test_thin_grouped(M, K):
    """Problems of different widths share one thin launch whatever tile a
    single call gives each; a large one beside them takes its own."""
    x = synth.activations(M, K, seed=821, outlier_seed=822, device=DEV)
    ws = [synth.weights(n, K, seed=823 + i, device=DEV) for i, n in enumerate((4096, 1024, 128, 12288))]
    check_group([x] * 4, ws, B1, B128, label="thin grouped")


@pytest.mark.parametrize("shape", [(2, 250, 7168, 5120), (4, 200, 16384, 4096), (8, 43, 32768, 3072)])
@pytest.mark.parametrize("pair", ["block", "row"])
def test_split_still_chosen(pair, shape):
    splits, M, K, N = shape
    ga, gb = PAIRS[pair]
    assert splits_of(M, N, K) == splits and route("splitk " + pair, M, K, N) == "split-K"
    a = synth.activations(M, K, seed=831, outlier_seed=832, device=DEV)
    b = synth.weights(N, K, seed=833, device=DEV)
    run_pair(a, b, ga, gb, rows=np.arange(3, M, 23), label="split-K S=%d %s" % (splits, pair), gemm=fp8q.gemm_splitk,
             adds=splits - 1)
