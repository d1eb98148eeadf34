"""Word products on the 32 x 32 tiles of small batches: bitwise the 128 x 128
tiles (which a chosen operand stream keeps), at the dimensions where tiles and K
steps begin and end, every word format and both iterations; and within 1e-6 of
the oracle in the multi-word formats."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402


def run(s, precision, iteration, variant):
    ctx = smx.Context(0).load(s).configure(precision=precision, iteration=iteration)
    smx.smx_set_kernel_variant(ctx.handle, variant)
    r = ctx.evaluate(allow_not_converged=precision == "bf16")
    h = smx.smx_get_history(ctx.handle)
    x = ctx.submatrix(0, 1)
    ctx.close()
    return r, h, x


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "bf16"])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 129, 200])
def test_bitwise_the_128_tiles(oracle_lib, n, precision, iteration):
    sizes = [min(13, n - q) for q in range(0, n, 13)]
    s = random_block_system(700 + n, sizes, density=0.7, coupling=0.04, groups="all", mu=0.01)
    a, ha, xa = run(s, precision, iteration, 0)
    b, hb, xb = run(s, precision, iteration, 1)       # the register-prefetch stream: 128 x 128 tiles
    assert np.array_equal(a.d_values, b.d_values) and np.array_equal(xa, xb)
    assert a.n_elec == b.n_elec and a.status == b.status
    for q in ("resid", "tau", "nsteps"):
        assert np.array_equal(ha[q], hb[q], equal_nan=True)
    if precision != "bf16":
        assert np.abs(a.d_values - oracle_lib.submatrix(s).d_values).max() <= 1e-6
