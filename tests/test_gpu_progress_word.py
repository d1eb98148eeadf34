"""The host follows the iteration by a progress word in host memory.  It must not
take an earlier evaluation's or wave's word for the current one's: evaluations
enqueued behind one another without a wait, polling switched on and off, several
waves, two threads with a context and stream each.  Bitwise against evaluations
that are waited for one by one."""

import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import water_config  # noqa: E402


def reference(s, precision, mus):
    out = []
    for mu in mus:
        ctx = smx.Context(0).load(s).configure(precision=precision, mu=mu)
        r = ctx.evaluate()
        out.append((r.d_values.copy(), r.n_elec, r.energy, ctx.group_info()["iters"]))
        ctx.close()
    return out


def check(ctx, ref):
    d = np.empty(ctx.nvalues)
    smx.smx_get_d(ctx.handle, d)
    assert np.array_equal(d, ref[0])
    assert smx.smx_trace(ctx.handle) == ref[1] and smx.smx_energy(ctx.handle) == ref[2]
    assert np.array_equal(ctx.group_info()["iters"], ref[3])


@pytest.mark.parametrize("waves", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp16x2", "fp32"])
def test_evaluations_behind_one_another(precision, waves):
    s = water_config("water16")
    mus = [0.0, 0.02, -0.02]
    ref = reference(s, precision, mus)
    ctx = smx.Context(0).load(s).configure(precision=precision, workspace_limit=12 << 20 if waves else 0)
    for poll in (1, 0, 1, 1):
        smx.smx_set_host_poll(ctx.handle, poll)
        for mu, r in zip(mus, ref):
            smx.smx_set_mu(ctx.handle, mu)
            smx.smx_evaluate(ctx.handle)           # not waited for before the next one
        smx.smx_wait(ctx.handle)
        check(ctx, ref[-1])
        smx.smx_set_mu(ctx.handle, mus[0])
        smx.smx_evaluate(ctx.handle)
        smx.smx_wait(ctx.handle)
        check(ctx, ref[0])
    assert not waves or ctx.stats()["nwaves"] > 1
    ctx.close()


def test_two_threads():
    torch = pytest.importorskip("torch")
    s = water_config("water16")
    mus = [0.0, 0.02, -0.02]
    ref = reference(s, "fp64", mus)
    failed = []

    def work(first):
        try:
            ctx = smx.Context(0, stream=torch.cuda.Stream().cuda_stream).load(s).configure(precision="fp64")
            for k in range(12):
                q = (first + k) % 3
                smx.smx_set_mu(ctx.handle, mus[q])
                smx.smx_evaluate(ctx.handle)
                smx.smx_wait(ctx.handle)
                check(ctx, ref[q])
            ctx.close()
        except Exception as e:       # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=work, args=(q,)) for q in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
