"""sd_kernel_name names the pair kernel that mobility_apply launches (CPU, on a
runtime that records launches), for the automatic choice on either side of its
lines and for forced shapes."""
import pytest

import stub_util

pytestmark = pytest.mark.slow


def test_named_kernel_is_the_launched_one():
    out = stub_util.child(stub_util.build(), """
L.sd_kernel_name.restype = C.c_char_p
def name(n, prec):
    s = L.sd_kernel_name(prec, i64(n))
    return s and s.decode()
seen = set()
def check(n, prec):
    assert apply(n, prec) == OK
    k = launches()[0].split("<")[0]
    assert name(n, prec) == k, (n, prec, name(n, prec), k)
    seen.add(k)
for n in (1, 64, 333, 1300, 3999, 4000, 5899, 5900, 16383, 16384, 65536, 100000, 120000, 400000):
    for prec in (KAHAN, F64, PLAIN):
        check(n, prec)
for prec, cfg in ((KAHAN, (0, 256, 4, 1, 8)), (KAHAN, (1, 128, 4, 1, 4)),
                  (KAHAN, (2, 256, 4, 1, 8)), (KAHAN, (2, 256, 4, 2, 16)), (F64, (0, 64, 2, 1, 0))):
    c = SdKernelConfig(*cfg)
    assert L.sd_set_kernel_config(prec, C.byref(c)) == OK
    check(5000, prec)
    assert L.sd_set_kernel_config(prec, None) == OK
assert name(0, KAHAN) is None and name(5, 7) is None
print(len(seen), sorted(seen))
""")
    assert out.startswith("9 "), out
