"""Which tiles the products of a batch take, on the CPU: the launches of an evaluation
over a stub of the HIP runtime.  Few tiles on every XCD: 32 x 32; a few large groups,
whose tiles share an XCD each: not the word products (128 x 128) and not the FP32 ones
(64 x 64); large batches: the large tiles."""

import os

import pytest

import hipstub

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")

F64 = {32: "ns_f64_kernel<{m}, 1, false>", 64: "ns_f64_kernel<{m}, 2, false>"}
F32 = {32: "ns_f32_kernel<{m}, 1, false>", 64: "ns_f32_kernel<{m}, 2, false>"}
FORMAT = {"fp16x2": "0, 2", "bf16x3": "1, 3", "bf16": "1, 1"}


def word(precision, edge):
    f = FORMAT[precision]
    return f"ns_words32_kernel<{f}, {{m}}>" if edge == 32 else f"ns_words_kernel<{f}, {{m}}, 0>"


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hipstub.build(tmp_path_factory.mktemp("hipstub"))


# n of a group, groups, edges of FP64, FP32, two, three and one words
CASES = [
    (100, 16, 32, 32, 32, 32, 32),
    (300, 30, 32, 32, 32, 32, 32),          # 220 tiles of 32 on an XCD
    (300, 40, 32, 32, 32, 32, 32),          # 275
    (500, 16, 32, 32, 32, 32, 128),         # 272
    (600, 8, 32, 32, 32, 32, 32),           # 190
    (700, 8, 32, 32, 32, 32, 128),          # 253
    (850, 8, 32, 32, 32, 128, 128),         # 378
    (700, 20, 32, 32, 128, 128, 128),       # 759
    (1000, 1, 32, 32, 128, 128, 128),       # 528
    (1025, 1, 32, 64, 128, 128, 128),
    (3000, 1, 32, 64, 128, 128, 128),
    (2000, 4, 64, 64, 128, 128, 128),       # 2112 tiles of 64
]


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("n,groups,e64,e32,e2,e3,e1", CASES)
def test_tiles_of_a_batch(stub, n, groups, e64, e32, e2, e3, e1, static):
    want = {"fp64": F64[e64], "fp32": F32[e32], "fp16x2": word("fp16x2", e2), "bf16x3": word("bf16x3", e3),
            "bf16": word("bf16", e1)}
    out = hipstub.run(stub, f"""
n, groups = {n}, {groups}
blk = max(1, min(25, n // groups))
sizes = [min(blk, n - q) for q in range(0, n, blk)]
cut = [len(sizes) * g // groups for g in range(groups + 1)]
s = random_block_system(3, sizes, density=1.0, groups=[list(range(a, b)) for a, b in zip(cut[:-1], cut[1:])])
ctx = smx.Context(0).load(s)
for precision in {list(want)!r}:
    ctx.configure(precision=precision)
    stub.stub_set(1, NEVER)
    launches()
    (smx.smx_evaluate_static if {static} else smx.smx_evaluate)(ctx.handle)
    print(precision, "|".join(sorted(set(k for k, g in launches("ns_")))), sep=":")
""")
    got = dict(line.split(":") for line in out.splitlines())
    for precision, names in got.items():
        assert set(names.split("|")) == {want[precision].format(m=m) for m in (0, 1)}, (precision, names)
    assert set(got) == set(want)


@pytest.mark.parametrize("shape,variant,names", [
    (0, 0, {"fp16x2": "ns_words32_kernel<0, 2, {m}>", "bf16x3": "ns_words32_kernel<1, 3, {m}>",
            "bf16": "ns_words32_kernel<1, 1, {m}>"}),
    (1 << 20, 0, {"fp16x2": "ns_words_kernel<0, 2, {m}, 0>", "bf16x3": "ns_words_kernel<1, 3, {m}, 0>",
                  "bf16": "ns_words_kernel<1, 1, {m}, 0>"}),
    (32, 0, {"fp16x2": "ns_words256_kernel<0, 2, {m}>", "bf16x3": "ns_words_kernel<1, 3, {m}, 0>",
             "bf16": "ns_words256_kernel<1, 1, {m}>"}),
    (1 << 20, 1, {"fp16x2": "ns_words_kernel<0, 2, {m}, 1>", "bf16": "ns_words_kernel<1, 1, {m}, 1>"}),
    (1 << 20, 2, {"fp16x2": "ns_words_persistent<0, 2, {m}>", "bf16": "ns_words_persistent<1, 1, {m}>"}),
])
def test_tiles_the_caller_chose(stub, shape, variant, names):
    """A size bucket that no group reaches keeps a small batch on the 128 x 128 tiles."""
    out = hipstub.run(stub, f"""
ctx = smx.Context(0).load(water_config("water16"))
smx.smx_set_tile_shape(ctx.handle, {shape})
smx.smx_set_kernel_variant(ctx.handle, {variant})
for precision in {list(names)!r}:
    ctx.configure(precision=precision)
    stub.stub_set(1, NEVER)
    launches()
    smx.smx_evaluate(ctx.handle)
    print(precision, "|".join(sorted(set(k for k, g in launches("ns_")))), sep=":")
""")
    for line in out.splitlines():
        precision, got = line.split(":")
        assert set(got.split("|")) == {names[precision].format(m=m) for m in (0, 1)}, line
