"""The last round of a large GEMM launch: 256 x 256 tiles run one per CU,
256 at a time, and a last round of up to 64 tiles is cut into four 128 x 128
parts each, of up to 128 into two 128 x 256 parts, while a fuller one keeps
whole tiles.  Shapes at both sides of each limit, ragged in M and (where the
pair allows it) in N, every form that runs these tiles (long K: at short K
such grids take 128 x 128 tiles).  Every tile shape
sums an output's K blocks in one order, so the result must equal, bit for
bit, the same product computed in strips of rows that take the smaller
tiles; the strips' kernels and sampled rows here are held to the oracle."""
import numpy as np
import pytest
import torch

import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

from _routes import route
from test_gpu_b_gemm import PAIRS, run_pair

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
K = 4224                               # odd number of K blocks: no K groups in the strips
# (tile rows, tile columns): a last round of 2, 64 (quarters), 72, 128 (halves), 148 (whole)
GRIDS = [(77, 10), (36, 16), (42, 20), (56, 16), (33, 20)]
FORMS = ["tensor", "row", "block", "blockk", "pow2", "e5m2", "quantized", "grouped"]


def call(form, a, sa, b, sb, strip=False):
    ga, gb = PAIRS[form] if form in PAIRS else PAIRS["block"]
    if form == "pow2":
        return [fp8q.gemm_pow2(a, sa, ga, b, sb, gb)]
    if form == "e5m2":
        return [fp8q.gemm_formats(a, sa, ga, b, sb, gb, fp8q.A_E5M2)]
    if form == "quantized":
        return list(fp8q.gemm_quantized(a, sa, ga, b, sb, gb))
    if form == "grouped":   # two problems whose tiles together make the grid
        cut = b.shape[0] // 256 * 128
        parts = [(a, sa, b[:cut], sb[:cut // 128 * (K // 128)].clone()),
                 (a, sa, b[cut:], sb[cut // 128 * (K // 128):].clone())] if cut else [(a, sa, b, sb)]
        # (a problem's K direction goes by its own columns)
        return [torch.cat([fp8q.gemm(p[0], p[1], ga, p[2], p[3], gb) for p in parts] if strip
                          else fp8q.gemm_grouped(parts, ga, gb), dim=1)]
    return [fp8q.gemm(a, sa, ga, b, sb, gb)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("form", FORMS)
def test_last_round_equals_strips(form, grid):
    tm, tn = grid
    M, N = 256 * tm - 71, 256 * tn - (60 if form in ("tensor", "row", "blockk") else 128)
    ga, gb = PAIRS[form] if form in PAIRS else PAIRS["block"]
    x = synth.activations(M, K, seed=501, outlier_seed=502, device=DEV)
    w = synth.weights(N, K, seed=503, device=DEV)
    print("last round", form, M, K, N, flush=True)
    assert form == "grouped" or route("block" if form == "e5m2" else form, M, K, N) == "large"
    a, sa = fp8q.quantize(x, ga, pow2=form == "pow2", e5m2=form == "e5m2")
    b, sb = fp8q.quantize(w, gb, pow2=form == "pow2")
    got = call(form, a, sa, b, sb)
    narrow = N // 256 * 128 if form == "grouped" and N >= 256 else N
    strip = -(-256 // -(-narrow // 128)) * 128   # 256 tiles of 128 x 128 or a few more
    assert route(form if form in PAIRS else "block", strip, K, narrow) in ("mid", "eight waves")
    for r in list(range(0, M - strip, strip)) + [M - strip]:
        e = r + strip
        s = sa if ga == fp8q.TENSOR else sa[r:e] if ga == fp8q.ROW else sa.view(K // 128, M)[:, r:e].reshape(-1)
        want = call(form, a[r:e], s.contiguous(), b, sb, strip=True)
        assert torch.equal(got[0][r:e].view(torch.uint8), want[0].view(torch.uint8)), "rows %d .. %d" % (r, e)
        if form == "quantized":
            assert torch.equal(got[1].view(N // 128, M)[:, r:e], want[1].view(N // 128, e - r))


@pytest.mark.parametrize("pair", ["block", "blockk"])
@pytest.mark.parametrize("grid", GRIDS[1:4])
def test_last_round_against_oracle(pair, grid):
    """(blockk: its 256 x 256 tiles too, with their column scales)"""
    M, N = 256 * grid[0] - 71, 256 * grid[1] - (128 if pair == "block" else 60)
    assert route(pair, M, K, N) == "large"
    a = synth.activations(M, K, seed=511, outlier_seed=512, device=DEV)
    b = synth.weights(N, K, seed=513, device=DEV)
    rows = np.unique(np.concatenate([np.arange(0, M, 509), np.arange(M - 12, M)]))
    run_pair(a, b, *PAIRS[pair], rows=rows, label="%s last round %dx%d" % (pair, *grid))
