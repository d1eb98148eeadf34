"""The gather in pieces of columns: the bound s_g is bitwise the row sum in
column order of the submatrix that the walk by block columns gives
(smx_get_submatrix), over one-element and ragged blocks, unstored blocks, and
row counts at and around the pieces of 16, 64 and 256."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

SIZES = {
    "one_element": [1] * 70,
    "ragged": [13, 5, 5, 17, 9, 31, 1, 2, 27, 1, 5, 25],
    "n1": [1], "n16": [16], "n17": [16, 1], "n32": [31, 1], "n64": [40, 24], "n65": [64, 1],
    "n256": [128, 128], "n257": [200, 57], "n321": [13] * 24 + [9],
}


@pytest.mark.parametrize("precision", ["fp64", "fp16x2", "fp32", "bf16x3"])
@pytest.mark.parametrize("name", sorted(SIZES))
def test_bounds_and_density(oracle_lib, name, precision):
    s = random_block_system(600, SIZES[name], density=0.5, coupling=0.03, groups="pairs" if len(SIZES[name]) > 2 else "all",
                            mu=0.013)
    ctx = smx.Context(0).load(s).configure(precision=precision)
    r = ctx.evaluate()
    scale = ctx.group_info()["scale"]
    for g in range(min(s.ngroups, 8)):
        a = np.abs(ctx.submatrix(g, 0))
        assert scale[g] == np.add.accumulate(a, axis=1)[:, -1].max()
    ctx.close()
    err = np.abs(r.d_values - oracle_lib.submatrix(s).d_values).max()
    assert err <= (1e-10 if precision == "fp64" else 1e-6)
