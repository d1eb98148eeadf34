"""The blocked reflectors at the dimensions where their blocks of 16 end, where
the rows held in registers change (n_pad 1024 / 1536 / more), and with more own
columns than one block of 16 takes: the diagonalisation path against LAPACK.
Bounds as for the reduction: 64 n u ||A|| on eigenvalues, times sqrt(n) / (4 kT)
on D."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

KT = 0.05


@pytest.mark.parametrize("n,own", [(3, 1), (18, 16), (19, 17), (35, 33), (50, 1), (1024, 17), (1025, 17), (1536, 40),
                                   (1537, 5), (1570, 33)])
def test_own_columns_against_lapack(n, own):
    sizes = [own] + [min(31, n - q) for q in range(own, n, 31)]
    s = random_block_system(400 + n, sizes, density=1.0, coupling=0.05, groups=[[0], list(range(1, len(sizes)))], mu=0.03)
    ctx = smx.Context(0).load(s).configure(precision="fp64", kT=KT)
    d = s.with_values(ctx.evaluate().d_values).to_dense()
    ctx.close()
    ref, q = np.linalg.eigh(s.to_dense())
    f = 0.5 * (1.0 - np.tanh((ref - s.mu) / (2 * KT)))
    u = 2.0 ** -53
    bound = 64 * n * u * np.abs(ref).max() * np.sqrt(n) / (4 * KT) + 8 * n * u
    assert np.abs(d - (q * f) @ q.T).max() <= bound
