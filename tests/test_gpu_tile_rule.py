"""One context, every precision in turn, where the modes take tiles of different edges
(FP64 32, FP32 64, words 128 or 32): the FP32 products on their own tile list, in one
wave and in several, in the caller's order of tiles, and from the fixed device array.
Against LAPACK's sign of the dense matrix (one group: D is the full density matrix), to
the modes' usual 1e-10 and 1e-6, and bitwise among themselves."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import random_block_system  # noqa: E402

TOL = {"fp64": 1e-10, "fp32": 1e-6, "fp16x2": 1e-6, "bf16x3": 1e-6}


@pytest.mark.parametrize("n,groups", [(1024, 1), (1025, 1), (1057, 2), (1100, 3)])
def test_every_precision(n, groups):
    sizes = [min(25, n - q) for q in range(0, n, 25)]
    cut = [len(sizes) * g // groups for g in range(groups + 1)]
    s = random_block_system(n, sizes, density=1.0, coupling=0.01, mu=0.01,
                            groups=[list(range(a, b)) for a, b in zip(cut[:-1], cut[1:])])
    lam, q = np.linalg.eigh(s.to_dense())
    d = q[:, lam < s.mu] @ q[:, lam < s.mu].T
    ctx = smx.Context(0).load(s)
    first = {}
    for order, limit in ((0, 0), (1, 0), (0, 120 << 20)):
        smx.smx_set_tile_order(ctx.handle, order)
        for precision in ("fp64", "fp32", "fp16x2", "bf16x3", "fp64", "fp32"):
            r = ctx.configure(precision=precision, workspace_limit=limit).evaluate()
            assert np.abs(s.with_values(r.d_values).to_dense() - d).max() <= TOL[precision]
            ref = first.setdefault(precision, r)
            assert np.array_equal(r.d_values, ref.d_values) and r.n_elec == ref.n_elec and r.energy == ref.energy
    assert groups == 1 or ctx.stats()["nwaves"] > 1
    smx.smx_set_tile_order(ctx.handle, 0)
    for precision, ref in first.items():
        ctx.configure(precision=precision, workspace_limit=0)
        smx.smx_evaluate_static(ctx.handle)
        smx.smx_wait(ctx.handle)
        out = np.empty(ctx.nvalues)
        smx.smx_get_d(ctx.handle, out)
        assert np.array_equal(out, ref.d_values) and smx.smx_trace(ctx.handle) == ref.n_elec
    ctx.close()
