"""The library's host code against a HIP runtime that launches nothing
(host_stub.cpp), for CPU tests of what a call plans, allocates and launches.
Undefined behaviour of the host code traps."""
import concurrent.futures as cf
import functools
import glob
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r"""
import ctypes as C
class SdParams(C.Structure):         # as in sd.h
    _fields_ = [("a", C.c_double), ("eta", C.c_double), ("tensor", C.c_int32),
                ("overlap", C.c_int32), ("box", C.c_double * 3)]
class SdKernelConfig(C.Structure):
    _fields_ = [(k, C.c_int32) for k in ("variant", "block", "splits", "ilp", "kahan_block")]
L = C.CDLL(%r)
L.stub_log.restype = C.c_char_p
L.stub_largest.restype = C.c_size_t
L.sd_last_error.restype = C.c_char_p
KAHAN, F64, PLAIN = 0, 1, 2
OK, EINVAL, EALIGN, ENOMEM, EDEVICE, EUNSUPPORTED = range(6)
P = SdParams(1.0, 1.0, 0, 0)
p = C.byref(P)
A = C.c_void_p(1 << 30)          # a device array (nothing reads it)
i64, dbl = C.c_int64, C.c_double
def launches():
    # names of the kernels launched since the last call, without arguments
    out = []
    for line in L.stub_log().decode().splitlines():
        out.append(line.split("(")[0].replace("void ", "").replace("sd::", ""))
    return out
def largest():
    return L.stub_largest()
def alloc_limit(b):
    L.stub_alloc_limit(C.c_size_t(b))
def apply(n, prec):
    return L.mobility_apply(p, i64(n), A, A, A, prec, None)
def adjoint(n, prec):
    return L.mobility_adjoint(p, i64(n), A, A, A, A, A, prec, None)
def step(n, prec):
    return L.sd_step(p, i64(n), A, A, None, None, dbl(0.1), i64(0), 0, prec, None)
def run(n, prec, steps):
    return L.sd_run(p, i64(n), A, A, None, dbl(0.1), i64(steps), i64(0), 0, prec, None, i64(0), None)
def run_adjoint(n, prec, steps, every, ck=None):
    return L.sd_run_adjoint(p, i64(n), A, A, dbl(0.1), i64(steps), prec, ck, i64(every), A, A, A,
                            None)
"""


@functools.lru_cache(maxsize=None)
def build() -> str:
    """Path of libsd_stub.so, built anew once in a test session (20 seconds)."""
    sys.path.insert(0, ROOT)
    from paper_1205_6333_amd import build as B
    out_dir = os.path.join(B.BUILD, "stub")
    os.makedirs(out_dir, exist_ok=True)
    empty = os.path.join(out_dir, "empty.bin")     # the device code: none
    open(empty, "w").close()
    flags = [B.hipcc(), "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-fPIC",
             "-Xclang", "-fcuda-include-gpubinary", "-Xclang", empty,
             "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined",
             "-I" + os.path.join(ROOT, "include"), "-I" + B.CSRC]
    srcs = sorted(glob.glob(os.path.join(B.CSRC, "*.hip")) + glob.glob(os.path.join(B.CSRC, "*.cpp")))
    srcs.append(os.path.join(ROOT, "tests", "host_stub.cpp"))

    def one(src):
        obj = os.path.join(out_dir, os.path.basename(src) + ".o")
        r = subprocess.run(flags + ["-c", src, "-o", obj], stdout=subprocess.PIPE,
                           stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout
        return obj

    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(one, srcs))
    lib = os.path.join(out_dir, "libsd_stub.so")
    # (its own runtime functions before those of a runtime that is loaded already)
    r = subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", lib] + objs,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return lib


def child(lib, script) -> str:
    """Runs script after PRELUDE in a child process; returns what it printed."""
    r = subprocess.run([sys.executable, "-c", PRELUDE % lib + script],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, "exit status %d\n%s" % (r.returncode, r.stdout[-3000:])
    return r.stdout
