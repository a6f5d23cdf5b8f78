"""What a call does when device memory for its workspace cannot be had (CPU, on a
runtime that launches nothing and can refuse allocations)."""
import pytest

import stub_util

pytestmark = pytest.mark.slow


@pytest.fixture(scope="module")
def stub():
    return stub_util.build()


@pytest.mark.parametrize("call,wave,general", [
    ("apply(60000, F64)", "k_wave_f64", "k_pair_f64_lds"),
    ("step(60000, F64)", "k_wave_f64", "k_pair_f64_lds"),
    ("run(60000, F64, 3)", "k_wave_f64", "k_pair_f64_lds"),
    ("adjoint(40000, F64)", "k_wave_adjoint", "k_adjoint_f64"),
    ("adjoint(40000, KAHAN)", "k_wave_adjoint", "k_adjoint_f32"),
    ("run_adjoint(40000, KAHAN, 5, 2)", "k_wave_adjoint", "k_adjoint_f32")])
def test_general_kernels_without_the_wave_workspace(stub, call, wave, general):
    """The kernels that need tens of MiB run where hundreds are refused; once
    the memory is there, the others run again."""
    out = stub_util.child(stub, """
alloc_limit(100 << 20)
print(%(c)s, " ".join(launches()))
alloc_limit(1 << 40)
print(%(c)s, " ".join(launches()))
""" % dict(c=call)).split("\n")
    assert out[0].startswith("0 ") and general in out[0] and wave not in out[0]
    assert out[1].startswith("0 ") and wave in out[1] and general not in out[1]


def test_no_memory_at_all_is_reported(stub):
    out = stub_util.child(stub, """
alloc_limit(1 << 10)
for st in (apply(60000, F64), apply(6007, KAHAN), adjoint(3001, F64), step(300, KAHAN)):
    print(st == ENOMEM, launches(), L.sd_last_error().decode())
""").split("\n")[:-1]
    assert len(out) == 4
    for line in out:
        assert line.startswith("True [] workspace allocation"), line


@pytest.mark.parametrize("prec", ["KAHAN", "F64"])
def test_long_segments_hold_frames_only(stub, prec):
    """A trajectory gradient with one long checkpoint segment allocates its frames
    and, beside them, less than another half: 2000 steps of 8192 particles."""
    out = stub_util.child(stub, """
n, steps = 8192, 2000
alloc_limit(1 << 40)
st = run_adjoint(n, %s, steps, steps)
L.stub_total.restype = C.c_size_t
print(st, L.stub_total() / (24.0 * n * steps))
""" % prec).split("\n")
    st, ratio = out[0].split(" ")
    assert st == "0" and float(ratio) < 1.5, out[0]
