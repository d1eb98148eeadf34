"""smx_evaluate_static against smx_evaluate, bitwise: every edge of the products' tiles,
both tile orders, several waves; and a problem at the limit of the array, whose FP64 and
FP32 products take the quarters of 128 x 128 tiles because no room is left for lists."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import dense_to_bsc, random_block_system, water_config  # noqa: E402


def check(s, precision, order, **cfg):
    ctx = smx.Context(0).load(s).configure(precision=precision, **cfg)
    smx.smx_set_tile_order(ctx.handle, order)
    r = ctx.evaluate(allow_not_converged=precision == "bf16")
    smx.smx_evaluate_static(ctx.handle)
    try:
        smx.smx_wait(ctx.handle)
        status = smx.SMX_OK
    except smx.SmxError as e:
        status = e.code
    d = np.empty(ctx.nvalues)
    smx.smx_get_d(ctx.handle, d)
    assert status == r.status and np.array_equal(d, r.d_values)
    assert smx.smx_trace(ctx.handle) == r.n_elec and smx.smx_energy(ctx.handle) == r.energy
    ctx.close()


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16x2", "bf16x3", "bf16"])
@pytest.mark.parametrize("n", [1, 32, 33, 64, 65, 97, 128, 129, 161, 257, 390])
def test_small(n, precision, iteration):
    sizes = [min(13, n - q) for q in range(0, n, 13)]
    s = random_block_system(900 + n, sizes, density=0.6, coupling=0.03, groups="pairs", mu=0.01)
    for order in (0, 1):
        check(s, precision, order, iteration=iteration)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16x2"])
def test_large_batch(precision):
    check(water_config("water256"), precision, 0)


@pytest.mark.parametrize("n,m", [(4000, 2282), (3990, 2282)])
def test_quarters_at_the_limit(n, m):
    """Two groups; n_pad = 4000: the last 128 x 128 tiles reach 96 rows beyond it, quarters wholly."""
    sizes = [500] * (m // 500) + [m % 500]
    first = len(sizes)
    sizes += [500] * ((n - m) // 500) + [(n - m) % 500]
    k = np.zeros((n, n))
    hop = np.where(np.arange(n - 1) % 2 == 0, -1.0, -0.6)
    k[np.arange(n - 1), np.arange(1, n)] = hop
    k[np.arange(1, n), np.arange(n - 1)] = hop
    s = dense_to_bsc(k, sizes, np.ones((len(sizes),) * 2, dtype=bool),
                     groups=[list(range(first)), list(range(first, len(sizes)))], mu=0.0)
    for precision in ("fp64", "fp32"):
        check(s, precision, 0)
