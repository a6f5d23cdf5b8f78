"""Lubrication forces of a suspension far from the origin: the same as those at the
origin of the same (rounded) differences, in about the same time."""
import time

import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [2.0 ** 31, 1.0e10, -3.0e12])
def test_far_suspension(orc, offset):
    """Differences of far positions are exact in FP64, so the forces meet the
    lubrication tests' 1e-12; the ratio of times is about 1 (and 1000 where the
    suspension shares one cell)."""
    import torch
    import paper_1205_6333_amd as sd
    n = 4000
    x = W.random_suspension(n, phi=0.3, min_dist=2.02, seed=3)
    far = x + [offset, -offset, offset]
    v = W.gaussian_forces(n, seed=4)
    vd, p, lb = to_dev3(v), sd.params(), sd.lub(1.0, 1e-3)

    def timed(pos):
        xd = to_dev3(pos)
        out = sd.lubrication_forces(xd, vd, params=p, lub_params=lb)
        torch.cuda.synchronize()
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            sd.lubrication_forces(xd, vd, f_out=out, params=p, lub_params=lb)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return out.cpu().numpy(), min(t)

    (_, t_near), (got, t_far) = timed(x), timed(far)
    ref = orc.lubrication_force(orc.params(), orc.lub(1.0, 1e-3), far, v)
    assert rel2(got, ref) <= 1e-12
    assert t_far <= 10.0 * t_near, (t_far, t_near)
