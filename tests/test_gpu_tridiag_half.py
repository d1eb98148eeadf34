"""The diagonalisation path at the dimensions where the Householder reduction's
panels, 16-column strips and 64-row pieces begin and end, and where it changes
from the lower triangle to the full block (n = 1280 / 1281), against LAPACK.

Bounds: a backward stable reduction and eigensolver leave eigenvalues within a
modest multiple of n u ||A|| (64 n u ||A|| here), and D = f(A) within the same
times the Lipschitz constant 1 / (4 kT) of the Fermi function, times another
sqrt(n) for the elementwise sum over eigenvectors."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

KT = 0.05


@pytest.mark.parametrize("n", [1, 2, 3, 4, 16, 17, 18, 19, 33, 34, 63, 64, 65, 66, 81, 130, 257, 513, 514, 1025,
                               1279, 1280, 1281])
def test_against_lapack(n):
    sizes = [min(31, n - q) for q in range(0, n, 31)]
    s = random_block_system(300 + n, sizes, density=1.0, coupling=0.05, groups="all", mu=0.03)
    ctx = smx.Context(0).load(s).configure(precision="fp64", kT=KT)
    r = ctx.evaluate()
    lam, w = smx.smx_get_spectrum(ctx.handle)
    ctx.close()
    k = s.to_dense()
    ref, q = np.linalg.eigh(k)
    u = 2.0 ** -53
    bound = 64 * n * u * np.abs(ref).max()
    assert np.abs(np.sort(lam) - ref).max() <= bound
    assert abs(w.sum() - n) <= 64 * n * n * u
    f = 0.5 * (1.0 - np.tanh((ref - s.mu) / (2 * KT)))
    dense = (q * f) @ q.T
    d = s.with_values(r.d_values).to_dense()
    assert np.abs(d - dense).max() <= bound * np.sqrt(n) / (4 * KT) + 8 * n * u
    assert abs(r.n_elec - f.sum()) <= n * bound / (4 * KT) + 8 * n * n * u
