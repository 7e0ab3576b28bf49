"""Tensorwise quantization of small tensors (up to 131072 elements in one
kernel, whose workgroups each take the whole tensor's amax) against the
oracle, byte for byte: the smallest tensor, pieces that do not fill a
workgroup, both sides of the limit, padded rows in and out, and amaxes of
zero, of the smallest and largest bf16 values."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("pow2,e5m2", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("rows,cols", [(1, 16), (17, 48), (129, 336), (128, 1024), (8193, 16)])
def test_small_tensor(rows, cols, pow2, e5m2):
    base = synth.activations(rows, cols, seed=901, outlier_seed=902)
    for scale in (0.0, 2.0 ** -133, 2.0 ** -100, 1.0, 2.0 ** 120):
        x = (base.float() * scale).clamp(-3.3e38, 3.3e38).to(torch.bfloat16)
        want, ws = oracle.quantize(synth.bf16_bits(x), oracle.TENSOR, False, pow2, e5m2)
        padded = torch.zeros((rows, cols + 24), dtype=torch.bfloat16, device=DEV)
        padded[:, :cols] = x.to(DEV)
        for src, pad in ((x.to(DEV), 0), (padded[:, :cols], 32)):
            codes = torch.full((rows, cols + pad), 0xA5, dtype=torch.uint8, device=DEV)
            _, s = fp8q.quantize(src, fp8q.TENSOR, codes=codes[:, :cols], pow2=pow2, e5m2=e5m2)
            assert np.array_equal(codes[:, :cols].cpu().numpy(), want), (scale, pad)
            assert np.array_equal(s.cpu().numpy(), ws), (scale, pad)
            assert torch.all(codes[:, cols:] == 0xA5)
