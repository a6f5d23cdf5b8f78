"""The end of the block-symmetric kernel's launches (split rows, j side, near
pairs, then velocities or the time step) where four waves share a run: candidate
lists that fill several times, blocks with and without an antipode, odd and even
numbers of steps (the positions end in the caller's array either way)."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3

pytestmark = pytest.mark.gpu

CFG = {"variant": 2, "block": 128, "splits": 2, "ilp": 1, "kahan_block": 8}
ONE_SIDED = {"variant": 0, "block": 256, "splits": 2, "ilp": 1, "kahan_block": 8}


@pytest.mark.parametrize("integ", [0, 1])
@pytest.mark.parametrize("steps", [1, 4, 5])
@pytest.mark.parametrize("n,side", [(130, 6.0), (513, 9.0), (2000, 60.0)])
def test_steps_match_the_one_sided_kernel(n, side, steps, integ):
    """Velocities of FP32 sums agree to 1e-6 (the other product tests); the
    displacement of a few short steps is their sum."""
    import torch
    import paper_1205_6333_amd as sd
    rng = np.random.default_rng(n + steps)
    x0 = rng.uniform(0.0, side, size=(n, 3))     # crowded: every run near every other
    p = sd.params(overlap=True)
    frc = sd.sd_pack(to_dev3(W.gaussian_forces(n, seed=4)))
    dt, out, vel = 1e-3, [], []
    try:
        for cfg in (CFG, ONE_SIDED):
            sd.sd_set_kernel_config(sd.SD_FP32_KAHAN, cfg)
            x = to_dev3(x0)
            vp = torch.zeros_like(x)
            sd.sd_premise_counts(reset=True)
            vel.append(sd.mobility_apply(sd.sd_pack(x), frc, params=p).cpu().numpy())
            counts = sd.sd_premise_counts(reset=True)
            if integ:
                sd.sd_run(x, frc, dt, steps, v_prev=vp, integrator=sd.SD_AB2, params=p)
                vel.append(vp.cpu().numpy())
            else:
                sd.sd_run(x, frc, dt, steps, params=p)
            out.append((x.cpu().numpy() - x0, counts))
    finally:
        sd.sd_set_kernel_config(sd.SD_FP32_KAHAN, None)
    assert out[0][1] == out[1][1] and out[0][1][0] > 0
    assert rel2(out[0][0], out[1][0]) <= 1e-6
    half = len(vel) // 2
    for a, b in zip(vel[:half], vel[half:]):
        assert rel2(a, b) <= 1e-6
