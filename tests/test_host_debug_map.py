"""The debug checks look at the block maps that the gathers read, not only at the host's
copy: over a stub of the HIP runtime, where no kernel runs and the device's maps stay
zero, an evaluation with the checks on is refused and names the table."""

import os

import pytest

import hipstub

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


@pytest.mark.parametrize("precision", ["fp64", "fp16x2"])
def test_device_map_is_checked(tmp_path, precision):
    hipstub.run(hipstub.build(tmp_path), f"""
ctx = smx.Context(0).load(water_config("water16")).configure(precision={precision!r})
stub.stub_set(2, NEVER)
smx.smx_evaluate(ctx.handle)
smx.smx_set_debug_checks(ctx.handle, True)
try:
    smx.smx_evaluate(ctx.handle)
    assert False, "the zero map was accepted"
except smx.SmxError as e:
    assert e.code == smx.SMX_E_INVALID and "block map" in str(e), e
""")
