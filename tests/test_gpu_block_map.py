"""The groups' block maps, built on the device: the gathered submatrix is
bitwise the principal submatrix of K over the group's rows (unstored blocks zero)
less mu on the diagonal, for row counts at and around the 16 columns of a
workgroup and the 64 rows of a wave, sparse and full patterns, groups in any
order, and again after another pattern on the same context."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402


def check(ctx, s):
    dense = np.zeros((s.n, s.n))
    first = np.concatenate([[0], np.cumsum(s.blk_size)]).astype(int)
    off = s.val_off()
    rows = []
    for j in range(s.nblk):
        rows.append(s.row_idx[s.col_ptr[j]:s.col_ptr[j + 1]])
        for p in range(s.col_ptr[j], s.col_ptr[j + 1]):
            i = s.row_idx[p]
            blk = s.values[off[p]:off[p + 1]].reshape(s.blk_size[i], s.blk_size[j], order="F")
            dense[first[i]:first[i + 1], first[j]:first[j + 1]] = blk
    ctx.load(s).configure(precision="fp64")
    ctx.evaluate()
    for g in range(s.ngroups):
        blocks = np.unique(np.concatenate([rows[j] for j in s.grp_blocks[s.grp_ptr[g]:s.grp_ptr[g + 1]]]))
        at = np.concatenate([np.arange(first[i], first[i + 1]) for i in blocks])
        a = dense[np.ix_(at, at)] - s.mu * np.eye(len(at))
        assert np.array_equal(ctx.submatrix(g, 0), a), g


@pytest.mark.parametrize("m", [1, 15, 16, 17, 63, 64, 65, 130])
def test_submatrix_of_k(m):
    sizes = [1 + (7 * i) % 3 for i in range(m)]
    ctx = smx.Context(0)
    every = list(range(m))
    check(ctx, random_block_system(700 + m, sizes, density=1.0, coupling=0.02, groups=[every], mu=0.01))
    check(ctx, random_block_system(701 + m, sizes, density=0.15, coupling=0.02,
                                   groups=[every[1::2][::-1], every[0::2]] if m > 1 else [[0]], mu=-0.02))
    check(ctx, random_block_system(702 + m, sizes, density=0.05, coupling=0.02, groups="column"))
    ctx.close()
