"""A tuning run that fails leaves the shape that an earlier run installed (CPU, on a
runtime that launches nothing and can refuse a kernel)."""
import pytest

import stub_util

pytestmark = pytest.mark.slow


@pytest.mark.parametrize("n,prec,kernel", [(333, "KAHAN", "k_row_f32"), (333, "F64", "k_row_f64"),
                                           (6007, "KAHAN", "k_wave_f32"),
                                           (6007, "F64", "k_wave_f64")])
def test_tuned_shape_survives_a_failed_run(n, prec, kernel):
    """The automatic choice is timed last, and the runtime's clock makes later
    candidates slower: the first run installs another shape, the second ends with
    the failure of the automatic choice's kernel."""
    out = stub_util.child(stub_util.build(), """
n, prec = %d, %s
def shape():
    c = SdKernelConfig()
    assert L.sd_get_kernel_config(prec, i64(n), C.byref(c)) == OK
    return [getattr(c, f[0]) for f in c._fields_]
def tune():
    st = L.sd_autotune(p, i64(n), prec, None, None, i64(0))
    return st, launches()
before = shape()
st, ran = tune()
assert st == OK and any(%r in k for k in ran), (st, ran[-5:])
tuned = shape()
assert tuned != before
L.stub_fail_kernel(%r.encode(), C.c_long(0))
st, ran = tune()
assert st == EDEVICE, st
assert shape() == tuned, (before, tuned, shape())
L.stub_fail_kernel(b"", C.c_long(0))
apply(n, prec)
assert not any(%r in k for k in launches())
print("held")
""" % (n, prec, kernel, kernel, kernel))
    assert "held" in out
