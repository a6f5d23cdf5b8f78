"""Planning of products, steps and adjoints at every accepted order of magnitude
(CPU, on a runtime that launches nothing): no overflow, no division by zero, and
above the workspace cap the kernels that need little of it."""
import pytest

import stub_util

pytestmark = pytest.mark.slow


@pytest.fixture(scope="module")
def stub():
    return stub_util.build()


# powers of two (whole blocks, the largest even block counts), their neighbours
# and the last 64 sizes below 2^25
SIZES = sorted({(1 << k) + d for k in range(16, 31) for d in (-129, -63, -1, 0, 1, 63, 129)
                if (1 << k) + d <= 1 << 30} | {(1 << 25) - d for d in range(64)} | {3 << 28})


@pytest.mark.parametrize("call,kernel", [
    ("apply(n, F64)", "k_pair_f64"), ("step(n, F64)", "k_pair_f64"),
    ("adjoint(n, F64)", "k_adjoint_f64"), ("adjoint(n, KAHAN)", "k_adjoint_f32"),
    ("apply(n, KAHAN)", "k_pair_f32"), ("apply(n, PLAIN)", "k_pair_f32")])
def test_large_sizes(stub, call, kernel):
    out = stub_util.child(stub, """
for n in %r:
    st = %s
    print(n, st, " ".join(launches()), flush=True)
""" % (SIZES, call))
    lines = out.split("\n")[:-1]
    assert len(lines) == len(SIZES)
    for n, line in zip(SIZES, lines):
        f = line.split(" ")
        assert f[:2] == [str(n), "0"], line
        if n >= 1 << 20:
            assert kernel in line, line
