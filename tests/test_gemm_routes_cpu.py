"""The rules that choose a call's kernel (csrc/dispatch.h), on the host."""
import random

import pytest

from _routes import FORMS, few_rows, route


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
    if form.startswith("splitk"):
        want |= {"split-K"}
    assert seen == want


@pytest.mark.parametrize("form", ["tensor", "row", "block", "blockk", "pow2", "quantized"])
def test_short_k_stays_off_large_tiles(form):
    """Grids of a few hundred 256 x 256 tiles at one K block, which take 3 to
    29% longer on them than on 128 x 128 tiles; and long K, where it is the
    other way."""
    for M, N in ((3000, 8192), (1500, 12288), (5000, 5120)):
        assert route(form, M, 128, N) == "mid", (M, N)
    for M, N in ((3001, 17408), (4096, 17408), (16384, 12288)):
        assert route(form, M, 5120, N) == "large", (M, N)
    if form == "blockk":
        for M, N in ((8192, 4096), (16384, 6144), (16384, 12288), (4096, 17408)):
            assert [route(form, M, K, N) for K in (128, 512, 16384)] == ["mid", "mid", "large"], (M, N)
        assert route(form, 6528, 1280, 16384) == route(form, 4096, 1280, 17408) == "large"  # on mid 6% longer
    if form == "quantized":
        assert route(form, 2500, 2048, 8192) == "large"  # on mid 6% longer


def test_quantized_output_sums_as_the_plain_call():
    """The thin tiles and the two K groups have sum orders of their own: both
    calls take them at the same sizes, everywhere."""
    rng = random.Random(6)
    for _ in range(20000):
        M, K, N = int(2 ** rng.uniform(0, 11)), 128 * int(2 ** rng.uniform(0, 8)), 128 * int(2 ** rng.uniform(0, 8))
        plain, quantized = route("block", M, K, N), route("quantized", M, K, N)
        own = ("thin", "two K groups")
        assert (plain if plain in own else None) == (quantized if quantized in own else None), (M, K, N)


@pytest.mark.parametrize("form", ["tensor", "row", "block", "blockk", "pow2"])
def test_short_k_stays_off_thin_tiles(form):
    """A hundred or two rows, a wide output and a few K blocks: 40 to 85%
    longer on thin tiles than on 64 x 64 or eight-wave 128 x 128 ones; and
    the problems that thin tiles are for."""
    for M, K, N in ((192, 128, 8192), (160, 256, 8192), (192, 512, 8192), (8, 128, 25600)):
        assert route(form, M, K, N) != "thin", (M, K, N)
    for M, K, N in ((8, 4096, 6144), (16, 12288, 4096), (64, 12288, 4096), (256, 1024, 1024), (256, 12288, 2048)):
        assert route(form, M, K, N) == "thin", (M, K, N)


@pytest.mark.parametrize("form", ["splitk tensor", "splitk row", "splitk block", "splitk blockk"])
def test_split_where_it_takes_less_time(form):
    """Few rows against weights too large for the cache stay split (thin tiles
    10 to 19% longer); the decode down-projection and shorter K do not."""
    for M, K, N in ((33, 17408, 5120), (33, 25600, 5120), (64, 17408, 5120), (64, 25600, 5120), (64, 25600, 6144),
                    (250, 16384, 4096)):
        assert route(form, M, K, N) == "split-K", (M, K, N)
    for M, K, N in ((256, 12288, 4096), (200, 4096, 384), (8, 25600, 5120), (320, 3072, 5120)):
        assert route(form, M, K, N) == "thin", (M, K, N)


def test_many_short_rows_are_quantized_eight_a_thread():
    """Two rows a thread are 3 to 14% slower there, and faster on the rest."""
    for rows, cols in ((131072, 128), (131072, 256), (40000, 128), (131072, 512), (131073, 128), (16384, 17408)):
        assert not few_rows(rows, cols)
    for rows, cols in ((1, 128), (8192, 128), (8192, 256), (40000, 512), (16384, 4096), (3001, 5120), (256, 12288)):
        assert few_rows(rows, cols)
