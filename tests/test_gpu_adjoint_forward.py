"""The adjoint carried forward with the iterates, against the oracle's
Daleckii-Krein gradient where its rounding grows (small gaps at mu, many
steps) and where groups leave at different steps (step 0 among them).

Bound: a step's products round by n u relative to their operands, six products
a step, and the direction grows to at most s / gap times the seed on the way,
so the error of dL/dA_g = Xb / s_g is at most 6 K n u ||seed||_F / gap; the
oracle's divided differences are allowed the same."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402


def compare(oracle_lib, s, mu, gap):
    rng = np.random.default_rng(11)
    gd = rng.normal(size=s.values.shape)
    ctx = smx.Context(0).load(s).configure(precision="fp64", mu=mu)
    ctx.evaluate()
    info = ctx.group_info()
    dk, dmu = ctx.backward(1.0, 0.5, gd)
    dk2, dmu2 = ctx.backward(1.0, 0.5, gd)
    ctx.close()
    assert np.array_equal(dk, dk2) and dmu == dmu2
    ref = oracle_lib.frozen_gradient(s, info["iters"], info["scale"], mu, 1.0, 0.5, gd)
    seed = 0.5 * np.sqrt((gd ** 2).sum() + 0.25 * s.n) + 0.5 * np.sqrt((s.values ** 2).sum())
    k, n = int(info["iters"].max()), int(info["n"].max())
    tol = 12.0 * max(k, 1) * n * 2.0 ** -53 * seed / gap
    a, b = oracle_lib.symmetric_part(s, dk), oracle_lib.symmetric_part(s, ref["dk"])
    err = np.abs(a - b).max()
    print(f"gap {gap:.1e}: max|sym dK - oracle| = {err:.2e} (bound {tol:.2e}, max|dK| {np.abs(b).max():.2e}), "
          f"k {info['iters'].min()}-{k}, n up to {n}")
    assert err <= tol
    assert abs(dmu - ref["dmu"]) <= tol * np.sqrt(n * s.ngroups)
    return info


@pytest.mark.parametrize("gap", [1e-2, 1e-3, 1e-4])
def test_small_gap(oracle_lib, gap):
    s = random_block_system(31, [13, 5, 5, 17, 9, 31, 22, 13, 27, 11, 5, 25], density=0.45, coupling=0.02,
                            groups="pairs", mu=0.0)
    lam = np.concatenate([oracle_lib.group_eig(s, g, mu=0.0)[1] for g in range(s.ngroups)])
    compare(oracle_lib, s, float(lam[lam < 0].max()) + gap, gap)


def test_groups_that_leave_at_different_steps(oracle_lib):
    s = random_block_system(8, [1, 7, 1, 5, 9, 1, 3], density=0.3, coupling=0.05, groups="column", mu=0.0)
    lam = np.concatenate([oracle_lib.group_eig(s, g, mu=0.0)[1] for g in range(s.ngroups)])
    info = compare(oracle_lib, s, 0.0, float(np.abs(lam).min()))
    assert info["iters"].min() == 0 and len(set(info["iters"] % 2)) == 2
