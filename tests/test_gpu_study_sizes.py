"""The precision study's kernel at every group width (16 lanes per sphere down
to one) and at one and several rounds of pairs, against the oracle's Euler loop,
with overlapping and coincident spheres where the near branch acts."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import to_dev3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("form", ["rpy", "overlap", "oseen"])
def test_cluster_sizes(orc, n, form):
    """FP64 throughout 1e-12 of the displacement, compensated FP32 sums with
    FP64 or double-single positions 1e-6 (FP32 terms, a few dozen steps), plain
    FP32 positions 1e-3, as in the four-sphere tests."""
    import torch
    import paper_1205_6333_amd as sd
    rng = np.random.default_rng(n)
    if form == "overlap":
        x = rng.normal(0.0, 1.5, size=(n, 3))
        if n >= 5:
            x[n - 1] = x[1]
    else:
        x = W.clusters(1, n, n, min_dist=2.6, seed=n)[1]
    f = W.gravity_forces(n) + 0.2 * W.gaussian_forces(n, seed=n)
    f = W.round_to_f32(f)
    kw = dict(overlap=form == "overlap", tensor=1 if form == "oseen" else 0)
    steps, dt = 40, 0.01
    ref, _, tr = orc.run(orc.params(**kw), x, f, dt, steps, stride=20)
    tol = {(3, 2): 1e-12, (1, 2): 1e-6, (2, 1): 1e-6, (0, 2): 1e-5, (3, 1): 1e-11, (0, 0): 1e-3}
    specs = [dict(acc=a, pos=p, dt=dt, steps=steps, stride=20) for a, p in tol]
    state = torch.zeros((len(specs), 2, n, 3), dtype=torch.float64, device="cuda")
    state[:, 0] = to_dev3(x)
    traj = sd.sd_cluster_run(state, to_dev3(f), specs, params=sd.params(**kw))
    got, traj = state.cpu().numpy().sum(1), traj.cpu().numpy().reshape(len(specs), 2, n, 3)
    disp = np.abs(ref - x).max()
    for k, t in enumerate(tol.values()):
        assert np.abs(got[k] - ref).max() <= t * disp, (specs[k], np.abs(got[k] - ref).max() / disp)
        assert np.abs(traj[k, 0] - tr[1]).max() <= t * disp
