"""What the fixed device array of smx_evaluate_static takes, on the CPU over a stub of the
HIP runtime: the largest groups of a dense matrix that fit beside the tables and the
state (m own columns; one wave per group).  The numbers are those of the first form of
the array's layout: tables that grow push problems out that used to fit."""

import os

import pytest

import hipstub

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


@pytest.mark.parametrize("n,m", [(4000, 2282), (5000, 1151), (6000, 294)])
def test_largest_groups_that_fit(tmp_path, n, m):
    out = hipstub.run(hipstub.build(tmp_path), f"""
from waterbox import BlockSparse


def fits(n, m, precision):
    sizes, groups = [], []
    for c0 in range(0, n, m):                  # groups of m columns, in blocks of up to 1000
        own = min(m, n - c0)
        blocks = [min(1000, own - q) for q in range(0, own, 1000)]
        groups.append(list(range(len(sizes), len(sizes) + len(blocks))))
        sizes += blocks
    nb = len(sizes)
    s = BlockSparse(np.array(sizes, np.int32), np.arange(nb + 1, dtype=np.int64) * nb,
                    np.tile(np.arange(nb, dtype=np.int32), nb), np.zeros(n * n),
                    np.cumsum([0] + [len(g) for g in groups]).astype(np.int32),
                    np.concatenate(groups).astype(np.int32))
    ctx = smx.Context(0).load(s).configure(precision=precision)
    launches()
    try:
        smx.smx_evaluate_static(ctx.handle)
        return True
    except smx.SmxError as e:
        assert e.code == smx.SMX_E_NOMEM, e
        return False
    finally:
        ctx.close()


for precision in ("fp64", "fp32", "fp16x2"):
    print(fits({n}, {m}, precision), *sorted(set(launches("ns_"))), sep=";")
    print(fits({n}, {m} + 1, precision))
""")
    rows = [r.split(";") for r in out.splitlines()]
    assert [r[0] for r in rows] == ["True", "False"] * 3
    # no room for lists of 64 x 64 tiles: the quarters of the 128 x 128 ones (8 slots a
    # tile, with one group to a wave)
    nt = -(-n // 128)
    slots = 8 * nt * (nt + 1) // 2
    assert rows[0][1:] == [f"('ns_f64_kernel<{m}, 2, true>', {4 * slots})" for m in (0, 1)]
    assert rows[2][1:] == [f"('ns_f32_kernel<{m}, 2, true>', {4 * slots})" for m in (0, 1)]
    assert rows[4][1:] == [f"('ns_words_kernel<0, 2, {m}, 0>', {slots})" for m in (0, 1)]
