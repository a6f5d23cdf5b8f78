"""Adjoints above the size where the symmetric pass's workspace ends (1 GiB, n =
53250): the one-sided kernels and their merge, a single pass against the oracle
and the Euler loop (which packs the cotangent for every pass there) against the
composition of single passes."""
import functools

import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3, to_dev4

pytestmark = pytest.mark.gpu

N = 53505       # one particle in the last work-group
FORMS = {"rpy": dict(), "overlap": dict(overlap=True), "oseen": dict(tensor=1)}


@functools.lru_cache(maxsize=None)
def _inputs(close):
    x = W.random_suspension(N, seed=N)
    if close:   # pairs of every class, in one work-group and far apart
        rng = np.random.default_rng(N)
        for a in (0, N // 2, N - 8):
            x[a + 1] = x[a] + [1.3, 0.2, 0.0]
            x[a + 2] = x[a] + [0.0, 2.0005, 0.0]
            x[(a + N // 3) % N] = x[a] + rng.uniform(0.2, 0.5, 3)
    return tuple(W.round_to_f32(v) for v in
                 (x, W.gaussian_forces(N, seed=1), W.gaussian_forces(N, seed=2)))


@pytest.mark.parametrize("form", list(FORMS))
def test_large_adjoint(orc, form):
    """Tolerances of the smaller adjoints: 1e-11 in FP64, 1e-6 in FP32."""
    import torch
    import paper_1205_6333_amd as sd
    x, f, lam = _inputs(form == "overlap")
    po = orc.params(**FORMS[form])
    rx, rf = orc.mobility_vjp_x(po, x, f, lam), orc.mobility_transpose(po, x, lam)
    for prec, dt, tol in ((1, torch.float64, 1e-11), (0, torch.float32, 1e-6)):
        gx, gf = sd.mobility_adjoint(*[to_dev4(v, dt) for v in (x, f, lam)],
                                     params=sd.params(**FORMS[form]), precision=prec)
        assert rel2(gx.cpu().numpy(), rx) <= tol and rel2(gf.cpu().numpy(), rf) <= tol


@pytest.mark.parametrize("prec,tol", [(1, 1e-12), (0, 1e-6)])
def test_large_trajectory_gradient(prec, tol):
    """Three steps, a checkpoint every two, overlapping pairs; the reference takes
    the states from sd_run and the passes from mobility_adjoint, in FP64."""
    import torch
    import paper_1205_6333_amd as sd
    x, f, g = _inputs(True)
    p, dt, steps = sd.params(overlap=True), 0.01, 3
    f64 = to_dev4(f, torch.float64)
    states, xd = [to_dev3(x)], to_dev3(x)
    for k in range(steps - 1):
        sd.sd_run(xd, f64, dt, 1, step0=k, precision=sd.SD_FP64, params=p)
        states.append(xd.clone())
    lam, gf = to_dev3(g), torch.zeros((N, 3), dtype=torch.float64, device=xd.device)
    for xk in reversed(states):
        a, b = sd.mobility_adjoint(sd.sd_pack(xk, sd.SD_FP64), f64, sd.sd_pack(lam, sd.SD_FP64),
                                   params=p, precision=sd.SD_FP64)
        gf, lam = gf + dt * b, lam + dt * a
    hx, hf = sd.sd_run_adjoint(to_dev3(x), to_dev4(f, torch.float64 if prec == 1 else torch.float32),
                               dt, steps, to_dev3(g), checkpoint_every=2, precision=prec, params=p)
    assert rel2(hx.cpu().numpy(), lam.cpu().numpy()) <= tol
    assert rel2(hf.cpu().numpy(), gf.cpu().numpy()) <= tol
