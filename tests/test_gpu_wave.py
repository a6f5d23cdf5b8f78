"""The kernels of the automatic choice for small and middle suspensions (whole
rows in one launch; each pair of particles once in wave-symmetric blocks)
against the oracle at the sizes where their schedules change: single
work-groups, remainders of the rounds of 256 particles, the first sizes with two
particles per work-group and of the wave-symmetric kernels, odd and even block
counts, ragged last blocks, near, overlapping and coincident pairs."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, rowerr, to_dev3, to_dev4

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1205_6333_amd as sd
    sd.lib()
    return sd


def _positions(n, box, close):
    """Random positions: a suspension, or (close) with pairs of every class,
    two of them coincident, in the first, a middle and the last block."""
    x = W.periodic_suspension(n, seed=n)[0] if box else W.random_suspension(n, seed=n)
    if close:
        rng = np.random.default_rng(n)
        for a in (0, n // 2, n - 8):
            x[a + 1] = x[a] + [1.3, 0.2, 0.0]
            x[a + 2] = x[a] + [0.0, 2.0005, 0.0]
            x[(a + n // 3) % n] = x[a] + rng.uniform(-0.5, 0.5, 3)
        x[n - 1] = x[0]
        x[n - 2] = x[n // 2]
    return x, W.box_side(n, 0.05)


@pytest.mark.parametrize("n", [9, 255, 257, 513, 1025, 1299, 1300, 1301, 3999, 4000, 4096, 4097,
                               4225])
@pytest.mark.parametrize("form", ["rpy", "overlap", "oseen", "box"])
def test_f64_product(sd, orc, n, form):
    """Velocities and premise counts of the FP64 product (1e-12: the sum of n
    FP64 terms of either order is within a few hundred eps of the other's)."""
    import torch
    x, L = _positions(n, form == "box", form != "oseen")
    f = W.gaussian_forces(n, seed=n + 1)
    kw = dict(overlap=form != "rpy", tensor=1 if form == "oseen" else 0,
              box=L if form == "box" else None)
    sd.sd_premise_counts(reset=True)
    v = sd.mobility_apply(to_dev4(x, torch.float64), to_dev4(f, torch.float64),
                          params=sd.params(**kw), precision=sd.SD_FP64)
    counts = sd.sd_premise_counts(reset=True)
    po = orc.params(**kw)
    ref = orc.mobility(po, x, f)
    assert rel2(v.cpu().numpy(), ref) <= 1e-12 and rowerr(v.cpu().numpy(), ref) <= 1e-11
    assert counts == tuple(orc.premise_counts(po, x))


@pytest.mark.parametrize("n", [9, 255, 257, 512, 513, 768, 769, 1024, 1025, 1299, 1300, 1301, 2047,
                               5899, 5900, 6016, 6017, 6145])
@pytest.mark.parametrize("prec", [0, 2])
@pytest.mark.parametrize("form", ["rpy", "overlap", "oseen", "box"])
def test_f32_product(sd, orc, n, prec, form):
    """The same for the FP32 products (tolerances of the one-sided kernels'
    tests: 1e-6 compensated, 1e-5 plain)."""
    import torch
    x, L = _positions(n, form == "box", form != "oseen")
    x, f = W.round_to_f32(x), W.round_to_f32(W.gaussian_forces(n, seed=n + 1))
    kw = dict(overlap=form != "rpy", tensor=1 if form == "oseen" else 0,
              box=L if form == "box" else None)
    sd.sd_premise_counts(reset=True)
    v = sd.mobility_apply(to_dev4(x, torch.float32), to_dev4(f, torch.float32),
                          params=sd.params(**kw), precision=prec)
    counts = sd.sd_premise_counts(reset=True)
    po = orc.params(**kw)
    ref = orc.mobility(po, x, f)
    tol = 1e-6 if prec == 0 else 1e-5
    assert rel2(v.cpu().numpy(), ref) <= tol and rowerr(v.cpu().numpy(), ref) <= 10 * tol
    assert counts == tuple(orc.premise_counts(po, x))


@pytest.mark.parametrize("n,prec,tol", [(300, 1, 1e-12), (300, 0, 1e-6), (1301, 0, 1e-6),
                                        (4100, 1, 1e-12), (6000, 0, 1e-6)])
@pytest.mark.parametrize("integ", [0, 1])
@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("steps", [1, 2, 3, 40])
def test_time_steps(sd, orc, n, prec, tol, integ, box, steps):
    """The kernels that also take the time step, eager (odd and even counts) and
    with graph replays (40), against the oracle: displacements within tol."""
    import torch
    if steps == 40 and n > 2000:
        steps = 35   # two replays and three eager steps
    x, L = _positions(n, box, False)
    f, dt = W.gravity_forces(n) + 0.2 * W.gaussian_forces(n, seed=5), 0.002
    if prec != 1:
        f = W.round_to_f32(f)
    xd, vp = to_dev3(x), to_dev3(np.zeros_like(x))
    sd.sd_set_graph_mode(2 if steps >= 35 else 1)
    try:
        sd.sd_run(xd, to_dev4(f, torch.float64 if prec == 1 else torch.float32), dt, steps,
                  v_prev=vp, integrator=integ, precision=prec,
                  params=sd.params(box=L if box else None))
    finally:
        sd.sd_set_graph_mode(1)
    ref, vl, _ = orc.run(orc.params(box=L if box else None), x, f, dt, steps, integrator=integ)
    assert rel2(xd.cpu().numpy() - x, ref - x) <= tol
    if integ:
        assert rel2(vp.cpu().numpy(), vl) <= tol


@pytest.mark.parametrize("n", [100, 1400])
def test_steps_with_near_pairs_and_checkpoints(sd, orc, n):
    """Overlapping spheres (their FP64 positions are read by other work-groups
    during a step) and checkpoints at odd and even steps; sd_step continues."""
    import torch
    x, _ = _positions(n, False, True)
    f, dt = W.round_to_f32(W.gaussian_forces(n, seed=8)), 0.001
    po = orc.params(overlap=True)
    for prec, tol in ((1, 1e-11), (0, 1e-6)):
        fd = to_dev4(f, torch.float64 if prec == 1 else torch.float32)
        ps = sd.params(overlap=True)
        xd, ck = to_dev3(x), to_dev3(np.zeros((3 * n, 3)))
        sd.sd_run(xd, fd, dt, 5, checkpoints=ck, checkpoint_every=2, precision=prec, params=ps)
        sd.sd_step(xd, fd, dt, 5, precision=prec, params=ps)
        ref = orc.run(po, x, f, dt, 6, stride=2)
        got = ck.cpu().numpy().reshape(3, n, 3)
        assert np.array_equal(got[0], x)
        for k in (1, 2):
            assert rel2(got[k] - x, ref[2][k] - x) <= tol
        assert rel2(xd.cpu().numpy() - x, ref[0] - x) <= tol


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 193, 1000])
@pytest.mark.parametrize("prec,tol", [(0, 1e-6), (1, 1e-11)])
@pytest.mark.parametrize("form", ["rpy", "overlap", "oseen"])
def test_adjoint(sd, orc, n, prec, tol, form):
    """Both gradients, tolerances of the one-sided kernel's tests."""
    import torch
    x, _ = _positions(n, False, n >= 63 and form != "oseen")
    f, lam = W.gaussian_forces(n, seed=n + 1), W.gaussian_forces(n, seed=n + 2)
    if prec != 1:
        x, f, lam = W.round_to_f32(x), W.round_to_f32(f), W.round_to_f32(lam)
    dt = torch.float64 if prec == 1 else torch.float32
    kw = dict(overlap=form == "overlap", tensor=1 if form == "oseen" else 0)
    gx, gf = sd.mobility_adjoint(to_dev4(x, dt), to_dev4(f, dt), to_dev4(lam, dt),
                                 params=sd.params(**kw), precision=prec)
    po = orc.params(**kw)
    ref = orc.mobility_vjp_x(po, x, f, lam)
    if n > 1:
        assert rel2(gx.cpu().numpy(), ref) <= tol
    else:
        assert np.all(gx.cpu().numpy() == 0.0)
    assert rel2(gf.cpu().numpy(), orc.mobility_transpose(po, x, lam)) <= tol


def test_trajectory_gradient(sd, orc):
    """The Euler adjoint (each pass leaves the next cotangent record) against
    the oracle's: 7 steps with a checkpoint every 3."""
    import torch
    n, steps, every, dt = 200, 7, 3, 0.01
    x, _ = _positions(n, False, False)
    f = W.gravity_forces(n) + 0.1 * W.gaussian_forces(n, seed=6)
    g = W.gaussian_forces(n, seed=7)
    for prec, tol in ((1, 1e-11), (0, 1e-6)):
        fr = f if prec == 1 else W.round_to_f32(f)
        rt = torch.float64 if prec == 1 else torch.float32
        gx, gf = sd.sd_run_adjoint(to_dev3(x), to_dev4(fr, rt), dt, steps, to_dev3(g),
                                   checkpoint_every=every, precision=prec)
        rx, rf = orc.run_adjoint_euler(orc.params(), x, fr, dt, steps, g)
        assert rel2(gx.cpu().numpy(), rx) <= tol and rel2(gf.cpu().numpy(), rf) <= tol
