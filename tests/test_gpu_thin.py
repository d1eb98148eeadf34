"""The thin products of the own-column polish, against the dense sign: rows and
K at and around the 64 rows of a workgroup, the 32 of a K step and the 64 of a
stage; own columns at and around a block of 16; few workgroups (one column block
each) and enough for two; and a K that is its own sign at step 0."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402


def worst(sizes, precision, coupling=0.03):
    """max |D - D_ref| with every block stored, so that each group's submatrix is K."""
    s = random_block_system(800 + sum(sizes), sizes, density=1.1, coupling=coupling / np.sqrt(max(sum(sizes), 64) / 64))
    ctx = smx.Context(0).load(s).configure(precision=precision)
    d = ctx.evaluate(allow_not_converged=precision == "bf16").d_values
    ctx.close()
    first = np.concatenate([[0], np.cumsum(s.blk_size)]).astype(int)
    off = s.val_off()
    k, got = np.zeros((s.n, s.n)), np.zeros((s.n, s.n))
    for j in range(s.nblk):
        for p in range(s.col_ptr[j], s.col_ptr[j + 1]):
            i = s.row_idx[p]
            at = np.ix_(range(first[i], first[i + 1]), range(first[j], first[j + 1]))
            shape = (s.blk_size[i], s.blk_size[j])
            k[at] = s.values[off[p]:off[p + 1]].reshape(shape, order="F")
            got[at] = d[off[p]:off[p + 1]].reshape(shape, order="F")
    w, v = np.linalg.eigh(k - s.mu * np.eye(s.n))
    return np.abs(got - (v * (w < 0)) @ v.T).max()


@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "fp32", "bf16"])
@pytest.mark.parametrize("sizes", [[1], [15, 16], [16, 17], [33, 30], [31, 33, 1], [17, 48, 1], [63, 33, 1],
                                   [65, 64], [100, 93, 17], [130, 1, 126]])
def test_few_workgroups(sizes, precision):
    # one BF16 word holds X to 2^-9 an element: 2e-2 bounds its D after the polish
    assert worst(sizes, precision) <= (2e-2 if precision == "bf16" else 1e-6)


@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "fp32"])
@pytest.mark.parametrize("blk", [16, 33])
def test_many_workgroups(blk, precision):
    # 64 groups of n = 64 blk: 1024 and 2112 workgroups of 64 rows
    assert worst([blk] * 64, precision) <= 1e-6


@pytest.mark.parametrize("precision", ["fp16x2", "bf16x3", "fp32"])
def test_sign_at_step_0(precision):
    assert worst([40, 31], precision, coupling=0.0) <= 1e-12
