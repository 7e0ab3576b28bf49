"""The rule that chooses a GEMM's kernel (csrc/dispatch.h), on the host."""
import random

import pytest

from _routes import FORMS, route


@pytest.mark.parametrize("form", list(FORMS))
def test_every_size_has_a_route(form):
    """Sizes over the whole range: each entry point names a kernel that it
    has (quantized output no plain 64 x 64 tile, split-K its own only for
    itself)."""
    rng = random.Random(5)
    seen = set()
    for _ in range(4000):
        M, K, N = int(2 ** rng.uniform(0, 17)), 128 * int(2 ** rng.uniform(0, 8)), 128 * int(2 ** rng.uniform(0, 9))
        seen.add(route(form, M, K, N))
    want = {"large", "mid", "eight waves", "thin", "two K groups"}
    if form != "quantized":
        want |= {"small"}
    if form == "splitk":
        want |= {"split-K"}
    assert seen == want
