"""Trajectory gradients whose checkpoint segments are too long to keep their
records (sd_run_adjoint stages each state again): the same states and passes, so
the same bits as with shorter segments, whose records are kept."""
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import to_dev3, to_dev4

pytestmark = pytest.mark.gpu


# rows, the wave-symmetric and the block-symmetric kernel; more than 64 MiB of
# records (32 or 16 bytes per particle and step) in one segment
@pytest.mark.parametrize("n,prec,steps", [(3000, 1, 701), (8192, 1, 258), (8192, 0, 515),
                                          (16384, 0, 258)])
def test_staged_again_or_kept(n, prec, steps):
    import torch
    import paper_1205_6333_amd as sd
    x = W.random_suspension(n, seed=n)
    f = to_dev4(W.gravity_forces(n) + 0.1 * W.gaussian_forces(n, seed=1),
                torch.float64 if prec == 1 else torch.float32)
    g = to_dev3(W.gaussian_forces(n, seed=2))
    a = sd.sd_run_adjoint(to_dev3(x), f, 1e-3, steps, g, checkpoint_every=steps, precision=prec)
    b = sd.sd_run_adjoint(to_dev3(x), f, 1e-3, steps, g, checkpoint_every=100, precision=prec)
    for u, v in zip(a, b):
        assert torch.isfinite(u).all() and torch.equal(u, v)
