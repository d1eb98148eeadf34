"""N, E and the status are those of the last evaluation also where the context's
stream is another one by the time they are read: evaluations behind work that keeps
their stream busy, read through another stream; and a captured evaluation replayed on
the default stream.  Bitwise against evaluations waited for one by one."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2004_10811_amd as smx  # noqa: E402
from waterbox import water_config  # noqa: E402

MUS = (0.0, 0.4)        # different N and E


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


@pytest.fixture(scope="module")
def system():
    return water_config("water16")


def results(s, mu, **cfg):
    ctx = smx.Context(0).load(s).configure(mu=mu, **cfg)
    r = ctx.evaluate()
    ctx.close()
    return r.n_elec, r.energy, r.d_values


def busy(torch):
    a = torch.full((8192, 8192), 1e-4, device="cuda")
    for _ in range(30):                     # about 0.2 s on the current stream
        a = a @ a
    return a


@pytest.mark.parametrize("cfg", [dict(precision="fp64"), dict(precision="fp16x2"), dict(precision="fp64", kT=0.01)])
@pytest.mark.parametrize("first", ["default", "side"])
def test_read_through_another_stream(torch, system, first, cfg):
    ref = [results(system, mu, **cfg) for mu in MUS]
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    on = torch.cuda.default_stream() if first == "default" else side
    ctx = smx.Context(0, stream=on.cuda_stream).load(system).configure(**cfg)
    smx.smx_set_host_poll(ctx.handle, 0)
    for q in (0, 1, 0):
        smx.smx_set_stream(ctx.handle, on.cuda_stream)
        smx.smx_set_mu(ctx.handle, MUS[q])
        torch.cuda.synchronize()
        with torch.cuda.stream(on):
            keep = busy(torch)
        smx.smx_evaluate(ctx.handle)
        smx.smx_set_stream(ctx.handle, other.cuda_stream)
        n, e = smx.smx_trace(ctx.handle), smx.smx_energy(ctx.handle)
        smx.smx_wait(ctx.handle)
        d = np.empty(ctx.nvalues)
        smx.smx_get_d(ctx.handle, d)
        assert n == ref[q][0] and e == ref[q][1] and np.array_equal(d, ref[q][2])
        del keep
    ctx.close()


def test_replay_on_the_default_stream(torch, system):
    ref = [results(system, mu, precision="fp64") for mu in MUS]
    side = torch.cuda.Stream()
    ctx = smx.Context(0, stream=side.cuda_stream).load(system).configure(precision="fp64", mu=MUS[1])
    smx.smx_evaluate_static(ctx.handle)     # tables in place before the capture
    smx.smx_wait(ctx.handle)
    graph = torch.cuda.CUDAGraph()
    smx.smx_set_mu(ctx.handle, MUS[0])
    with torch.cuda.graph(graph, stream=side):
        smx.smx_evaluate_static(ctx.handle)
    for _ in range(3):
        smx.smx_set_mu(ctx.handle, MUS[1])
        smx.smx_evaluate_static(ctx.handle)
        smx.smx_wait(ctx.handle)
        assert smx.smx_trace(ctx.handle) == ref[1][0]
        keep = busy(torch)
        graph.replay()                      # the current stream: the default one
        assert smx.smx_trace(ctx.handle) == ref[0][0] and smx.smx_energy(ctx.handle) == ref[0][1]
        smx.smx_wait(ctx.handle)
        del keep
    ctx.close()
