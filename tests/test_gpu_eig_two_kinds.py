"""Submatrices on both sides of the dimension where the Householder reduction changes
from the lower triangle to the full block, in one evaluation: spectra and D against
LAPACK's of each cluster, and D bitwise that of each cluster evaluated alone.  Bounds as
for one submatrix (64 n u ||A|| on eigenvalues, times 1 / (4 kT) and sqrt(n) on D)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import dense_to_bsc  # noqa: E402

KT, MU = 0.05, 0.03


def clusters(ns, seed=5):
    """Uncoupled dense clusters of the given dimensions, two groups each."""
    rng = np.random.default_rng(seed)
    parts = []
    for n in ns:
        g = rng.normal(0.0, 0.02, (n, n))
        parts.append((g + g.T) / 2 + np.diag(np.where(rng.uniform(size=n) < 0.5, -0.5, 0.5)))
    return parts


def system(parts):
    sizes, groups, owner = [], [], []
    for c, k in enumerate(parts):
        n, first = len(k), len(sizes)
        blk = min(47, n // 3)
        b = [min(blk, n - q) for q in range(0, n, blk)]
        sizes += b
        owner += [c] * len(b)
        half = first + len(b) // 3
        groups += [list(range(first, half)), list(range(half, first + len(b)))]
    kd = np.zeros((sum(sizes),) * 2)
    o = 0
    for k in parts:
        kd[o:o + len(k), o:o + len(k)] = k
        o += len(k)
    owner = np.array(owner)
    return dense_to_bsc(kd, sizes, owner[:, None] == owner[None, :], groups=groups, mu=MU)


def evaluate(s):
    ctx = smx.Context(0).load(s).configure(precision="fp64", kT=KT)
    r = ctx.evaluate()
    lam, w = smx.smx_get_spectrum(ctx.handle)
    n = ctx.group_info()["n"]
    ctx.close()
    return s.with_values(r.d_values).to_dense(), lam, n


@pytest.mark.parametrize("ns", [(1280, 1281), (1281, 1280), (33, 1312, 1248, 1300), (1600, 100)])
def test_both_kinds_in_one_launch(ns):
    parts = clusters(ns)
    d, lam, n_g = evaluate(system(parts))
    assert list(n_g) == [n for n in ns for _ in (0, 1)]
    u = 2.0 ** -53
    o = q = 0
    for n, k in zip(ns, parts):
        ref, v = np.linalg.eigh(k)
        bound = 64 * n * u * np.abs(ref).max()
        for _ in (0, 1):
            assert np.abs(np.sort(lam[q:q + n]) - ref).max() <= bound
            q += n
        f = 0.5 * (1.0 - np.tanh((ref - MU) / (2 * KT)))
        own = d[o:o + n, o:o + n]
        assert np.abs(own - (v * f) @ v.T).max() <= bound * np.sqrt(n) / (4 * KT) + 8 * n * u
        assert np.array_equal(own, evaluate(system([k]))[0])
        o += n
