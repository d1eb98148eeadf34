"""The host's side of the progress word, on the CPU: an evaluation that ends in an error
inside the step loop leaves words of its steps behind, and none of them may pass for
a step of the next evaluation."""

import os

import pytest

import hipstub

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hipstub.build(tmp_path_factory.mktemp("hipstub"))


@pytest.mark.parametrize("precision,kernel", [("fp64", "ns_f64_kernel<0,"), ("fp16x2", "ns_words32_kernel<0, 2, 0>")])
def test_tags_after_an_error(stub, precision, kernel):
    """Every group finishes in step 2; then again, in a context whose first evaluation
    ended where the event of one of its launches could not be created."""
    hipstub.run(stub, f"""
s = water_config("water16")


def context():
    return smx.Context(0).load(s).configure(precision={precision!r})


ctx = context()
stub.stub_set(2, NEVER)
smx.smx_evaluate(ctx.handle)
events, steps = stub.stub_events(), len(launches({kernel!r}))
assert 3 <= steps <= 6, steps
ctx.close()
for back in range(1, 2 * steps):              # the last events created are those of the launches
    ctx = context()
    stub.stub_set(2, events - back)
    try:
        smx.smx_evaluate(ctx.handle)
        assert False, "no error"
    except smx.SmxError as e:
        assert e.code == smx.SMX_E_NOMEM
    launches()
    smx.smx_update_values(ctx.handle, s.values)   # waits: the words of the steps before the error are written
    stub.stub_set(2, NEVER)
    smx.smx_evaluate(ctx.handle)
    n = len(launches({kernel!r}))
    assert n == steps, (back, n, steps)
    ctx.close()
""")
