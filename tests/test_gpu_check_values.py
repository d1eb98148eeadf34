"""The validation of K's values finds a planted asymmetry or NaN wherever it
sits, for every lane split of the kernel (mean block of 1, 4..511, 512 and more elements)
and for more blocks than one sweep of its grid covers."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

CASES = {
    "one_element_blocks": dict(blk_sizes=[1] * 600, density=0.9),     # 324,000 blocks: two sweeps
    "small_blocks": dict(blk_sizes=[3, 2, 4, 1] * 60, density=0.8),   # 46,000 blocks of 8 lanes: two sweeps
    "one_block": dict(blk_sizes=[37], density=1.0),
    "mixed_blocks": dict(blk_sizes=[13, 5, 5, 31, 1] * 18, density=0.6),
    "large_blocks": dict(blk_sizes=[23, 25] * 35, density=1.0),       # 64 lanes: two sweeps
}




@pytest.mark.parametrize("name", sorted(CASES))
def test_planted_values_are_found(name):
    s = random_block_system(5, **CASES[name])
    ctx = smx.Context(0).load(s)
    n = len(s.values)
    big = np.abs(s.values).max()
    off = s.val_off()
    diag = np.repeat(np.arange(s.nblk), np.diff(s.col_ptr)) == s.row_idx
    rng = np.random.default_rng(3)
    for q in sorted({0, n - 1, *rng.integers(0, n, 6).tolist()}):
        p = int(np.searchsorted(off, q, side="right")) - 1
        if diag[p] and s.blk_size[s.row_idx[p]] == 1:
            continue                                     # its own mirror
        v = s.values.copy()
        r, c = divmod(q - int(off[p]), int(s.blk_size[s.row_idx[p]]))
        if diag[p] and r == c:
            continue
        v[q] += 4e-12 * big
        with pytest.raises(smx.SmxError) as e:
            smx.smx_update_values(ctx.handle, v)
        assert e.value.code == smx.SMX_E_NOT_SYMMETRIC
        ctx.load(s)
        v = s.values.copy()
        v[q] += 0.25e-12 * big
        smx.smx_update_values(ctx.handle, v)
    for q in (0, n // 2, n - 1):
        for bad in (np.nan, np.inf, -np.inf):
            v = s.values.copy()
            v[q] = bad
            with pytest.raises(smx.SmxError) as e:
                smx.smx_update_values(ctx.handle, v)
            assert e.value.code == smx.SMX_E_NONFINITE
            ctx.load(s)
    ctx.close()
