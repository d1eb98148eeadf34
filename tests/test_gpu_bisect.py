"""Eigenvalues of tridiagonal forms that strain the Sturm counts: scales far
from 1, exact zeros on the diagonal (leading minors vanish at 0), multiple
eigenvalues, blocks that split, couplings near the splitting threshold.
Against LAPACK, within 64 n u ||A||."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import dense_to_bsc, tb_chain  # noqa: E402


def spectrum(k, scale):
    n = len(k)
    sizes = [min(16, n - q) for q in range(0, n, 16)]
    s = dense_to_bsc(k * scale, sizes, np.ones((len(sizes), len(sizes)), bool), groups=[list(range(len(sizes)))])
    ctx = smx.Context(0).load(s).configure(precision="fp64", kT=0.1 * scale)
    ctx.evaluate()
    lam, _ = smx.smx_get_spectrum(ctx.handle)
    ctx.close()
    return np.sort(lam)


def matrices(n):
    rng = np.random.default_rng(n)
    g = rng.normal(size=(n, n)) * 0.1
    yield "random", g + g.T
    yield "chain", tb_chain(n - n % 2, 2).to_dense()                      # zero diagonal
    yield "ring", tb_chain(n - n % 2, 2, periodic=True).to_dense()        # pairs of equal eigenvalues
    yield "identity", np.eye(n)
    yield "two_blocks", np.kron(np.eye(2), (g + g.T)[:n // 2 + 1, :n // 2 + 1])
    for c in (1e-7, 1e-15, 1e-17):
        d = np.diag(np.where(np.arange(n) % 2 == 0, 1.0, -1.0))
        yield f"coupling_{c:g}", d + c * (np.eye(n, k=1) + np.eye(n, k=-1))


@pytest.mark.parametrize("scale", [1.0, 1e-140, 1e140, 3.7e-9])
@pytest.mark.parametrize("n", [2, 9, 10, 17, 25, 130])
def test_spectrum(n, scale):
    for name, k in matrices(n):
        ref = np.linalg.eigvalsh(k)
        err = np.abs(spectrum(k, scale) / scale - ref).max()
        assert err <= 64 * len(k) * 2.0 ** -53 * max(np.abs(ref).max(), 1e-300), (name, err)
