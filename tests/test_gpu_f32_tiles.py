"""FP32 bulk products on both tile edges: edge 32 at the dimensions where tiles
begin, end and divide, edge 64 (more than 1536 tiles of 64), Newton-Schulz and
Pade steps, against the oracle at the bound of the reduced-precision modes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system, water_system  # noqa: E402


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
@pytest.mark.parametrize("n", [1, 16, 17, 31, 32, 33, 63, 64, 65, 97, 129])
def test_small_dimensions(oracle_lib, n, iteration):
    sizes = [min(13, n - q) for q in range(0, n, 13)]
    s = random_block_system(500 + n, sizes, density=0.7, coupling=0.04, groups="all", mu=0.01)
    ctx = smx.Context(0).load(s).configure(precision="fp32", iteration=iteration)
    r = ctx.evaluate()
    ctx.close()
    assert np.abs(r.d_values - oracle_lib.submatrix(s).d_values).max() <= 1e-6


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
def test_many_tiles(oracle_lib, iteration):
    s = water_system(200, 18.13, 4.6, 33)
    ctx = smx.Context(0).load(s).configure(precision="fp32", iteration=iteration)
    r = ctx.evaluate()
    n = ctx.group_info()["n"]
    ctx.close()
    assert ((-(-n // 64)) * (-(-n // 64) + 1) // 2).sum() > 1536
    pick = np.array(sorted({int(np.argmin(n)), int(np.argmax(n)), 100}))
    ref = oracle_lib.submatrix(s, which=pick, nthreads=8)
    ok = ~np.isnan(ref.d_values)
    assert np.abs(r.d_values[ok] - ref.d_values[ok]).max() <= 1e-6
