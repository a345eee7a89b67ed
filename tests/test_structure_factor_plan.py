"""Launch shapes of the context-free structure factor (host code only): what every
plan has to keep, and that counts of k tiles just past a block's 16 waves do not
leave most of a second group's waves idle."""
import os

import numpy as np
import pytest

from paper_2205_13824_amd import build as B
from paper_2205_13824_amd import rbsog as R

SIZES = [1, 63, 64, 65, 1000, 10002, 200_000, 1_999_998, 2 ** 31 - 1]
VECTORS = [1, 64, 65, 1000, 1024, 1025, 1100, 1500, 2047, 2049, 4000, 65537, 2 ** 20, 65535 * 256]


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(R.LIB_PATH):
        B.build()
    return R.lib()


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
@pytest.mark.parametrize("n_k", VECTORS)
def test_plans_cover_the_work(prec, n_k):
    tiles = -(-n_k // 64)
    for n in SIZES:
        p = R.rbsog_debug_structure_factor_plan(n, n_k, prec)
        assert 1 <= p["tiles"] <= 16 and p["streams"] == 16 // p["tiles"]
        assert (p["groups"] - 1) * p["tiles"] < tiles <= p["groups"] * p["tiles"]
        assert p["groups"] <= 65535  # blocks of a launch's second dimension
        assert 1 <= p["chunks"] <= max(1, min(512 // p["groups"], 2 ** 20 // n_k, n))


@pytest.mark.parametrize("n_k", [v for v in VECTORS if v > 1024] + list(range(1025, 3000, 64)))
def test_several_groups_fill_their_waves(n_k):
    """The waves that a SIMD runs of every group, over the particle streams, against
    the tiles there are: within 1.35 of it (17 tiles in groups of 16: 1.88)."""
    p = R.rbsog_debug_structure_factor_plan(1_999_998, n_k, R.RBSOG_FP32C)
    waves = p["tiles"] * p["streams"]
    assert p["groups"] * (-(-waves // 4) * 4) / p["streams"] <= 1.35 * -(-n_k // 64)


def test_arguments_are_checked():
    out = np.zeros(4, dtype=np.int64)
    f = R.lib().rbsog_debug_structure_factor_plan
    for n, n_k, prec, ptr in ((0, 1, 0, R._ptr(out)), (1, 0, 0, R._ptr(out)), (1, 1, 7, R._ptr(out)), (1, 1, 0, None)):
        assert f(n, n_k, prec, ptr) == -1
