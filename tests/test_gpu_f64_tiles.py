"""FP64 products on both tile edges against the oracle: edge 32 (few tiles) at
the dimensions where tiles begin, end and divide, edge 64 (more than 1536
tiles of 64) with padded dimensions that are and are not multiples of 64."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system, water_system  # noqa: E402


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
@pytest.mark.parametrize("n", [1, 2, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 129])
def test_small_dimensions(oracle_lib, n, iteration):
    sizes = [min(13, n - q) for q in range(0, n, 13)]
    s = random_block_system(200 + n, sizes, density=0.7, coupling=0.04, groups="all", mu=0.01)
    ctx = smx.Context(0).load(s).configure(precision="fp64", iteration=iteration)
    r = ctx.evaluate()
    ctx.close()
    ref = oracle_lib.submatrix(s)
    assert np.abs(r.d_values - ref.d_values).max() <= 1e-10
    assert abs(r.n_elec - ref.n_elec) <= 1e-9


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
def test_many_tiles(oracle_lib, iteration):
    s = water_system(200, 18.13, 4.6, 33)
    ctx = smx.Context(0).load(s).configure(precision="fp64", iteration=iteration)
    r = ctx.evaluate()
    n = ctx.group_info()["n"]
    ctx.close()
    nt = -(-n // 64)
    assert (nt * (nt + 1) // 2).sum() > 1536
    odd = (-(-n // 32)) % 2 == 1
    assert odd.any() and (~odd).any()
    pick = sorted({int(np.argmin(n)), int(np.argmax(n)), int(np.nonzero(odd)[0][0]), int(np.nonzero(~odd)[0][0])})
    ref = oracle_lib.submatrix(s, which=np.array(pick), nthreads=8)
    ok = ~np.isnan(ref.d_values)
    assert ok.any() and np.abs(r.d_values[ok] - ref.d_values[ok]).max() <= 1e-10
