"""The 128 x 128 word products that load straight into LDS, on small batches.  Those take
32 x 32 tiles by default; a size bucket that no group reaches keeps every group on the
128 x 128 kernel of large batches (tests/test_host_tiles.py shows which kernel each
setting launches).  Bitwise against the 32 x 32 tiles, the other operand streams and the
256 x 256 tiles, at remainders of every kind; and under the debug checks, whose guard
regions then lie behind the 128 x 128 kernel's writes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

NO_GROUP = 1 << 20


def run(s, precision, shape, variant=0, debug=False, **cfg):
    ctx = smx.Context(0).load(s).configure(precision=precision, **cfg)
    smx.smx_set_tile_shape(ctx.handle, shape)
    smx.smx_set_kernel_variant(ctx.handle, variant)
    smx.smx_set_debug_checks(ctx.handle, debug)
    r = ctx.evaluate(allow_not_converged=precision == "bf16")
    h = smx.smx_get_history(ctx.handle)
    ctx.close()
    return r, h


def same(a, b):
    (r, h), (q, g) = a, b
    return (np.array_equal(r.d_values, q.d_values) and r.n_elec == q.n_elec and r.energy == q.energy
            and r.status == q.status and all(np.array_equal(h[k], g[k], equal_nan=True) for k in ("resid", "tau", "nsteps")))


@pytest.mark.parametrize("iteration", ["ns2", "pade3"])
@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "bf16"])
@pytest.mark.parametrize("n", [1, 31, 33, 65, 97, 127, 128, 129, 160, 193, 255, 257, 290, 385])
def test_bitwise_the_other_tiles(n, precision, iteration):
    sizes = [min(13, n - q) for q in range(0, n, 13)]
    s = random_block_system(1100 + n, sizes, density=0.7, coupling=0.03, groups="all", mu=0.01)
    a = run(s, precision, NO_GROUP, iteration=iteration)
    assert same(a, run(s, precision, 0, iteration=iteration))               # 32 x 32
    assert same(a, run(s, precision, NO_GROUP, 1, iteration=iteration))     # register prefetch
    assert same(a, run(s, precision, NO_GROUP, 2, iteration=iteration))     # persistent
    assert same(a, run(s, precision, 32, iteration=iteration))              # 256 x 256 (not three words)


@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "bf16"])
def test_debug_checks(precision):
    s = random_block_system(61, [13, 5, 5, 17, 9, 31, 22, 13, 27, 11, 5, 25] * 2, density=0.45, coupling=0.02,
                            groups="pairs", mu=0.0)
    assert same(run(s, precision, NO_GROUP), run(s, precision, NO_GROUP, debug=True))
