"""The 1x128 quantizer's kernel for few elements against the oracle, byte for
byte: one row, rows that do not fill a workgroup's eight, columns that do not
fill its 512, padded rows in and out, both formats and scale rules, amaxes of
zero and of tiny values; and sizes just past its lines, which take the other
kernel."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_22870_amd as fp8q
from paper_2609_22870_amd import synth

from _routes import few_rows

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("pow2,e5m2", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("rows,cols", [(1, 128), (7, 640), (9, 512), (33, 1152), (256, 4096), (8192, 128), (8193, 128),
                                       (65537, 512)])
def test_few_rows(rows, cols, pow2, e5m2):
    assert few_rows(rows, cols) == (rows not in (8193, 65537))
    x = synth.activations(rows, cols, seed=951, outlier_seed=952)
    x[0, :64] = 0.0
    if rows > 5:
        x[3] = 0.0
        x[5] *= 2.0 ** -110
    want, ws = oracle.quantize(synth.bf16_bits(x), oracle.BLOCK_1x128, False, pow2, e5m2)
    padded = torch.zeros((rows, cols + 24), dtype=torch.bfloat16, device=DEV)
    padded[:, :cols] = x.to(DEV)
    codes = torch.full((rows, cols + 32), 0xA5, dtype=torch.uint8, device=DEV)
    _, s = fp8q.quantize(padded[:, :cols], fp8q.BLOCK_1x128, codes=codes[:, :cols], pow2=pow2, e5m2=e5m2)
    assert np.array_equal(codes[:, :cols].cpu().numpy(), want)
    assert np.array_equal(s.cpu().numpy(), ws)
    assert torch.all(codes[:, cols:] == 0xA5)
