"""Lubrication forces where cells hold more particles than one walk of a chain
takes (a multiple of them, one fewer, one more), against the oracle."""
import numpy as np
import pytest

from gpu_util import rel2, to_dev3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 8, 9, 10, 16, 17, 18, 25, 64, 300])
def test_one_crowded_cell(orc, n):
    """FP64 sums of n overlapping pairs: 1e-11, as in the other crowded form; two
    calls give the same bits."""
    import torch
    import paper_1205_6333_amd as sd
    rng = np.random.default_rng(n)
    x, v = rng.uniform(0.1, 2.6, size=(n, 3)), rng.normal(size=(n, 3))
    p, lb = sd.params(), sd.lub(1.0, 1e-3)
    f = sd.lubrication_forces(to_dev3(x), to_dev3(v), params=p, lub_params=lb)
    assert torch.equal(f, sd.lubrication_forces(to_dev3(x), to_dev3(v), params=p, lub_params=lb))
    ref = orc.lubrication_force(orc.params(), orc.lub(1.0, 1e-3), x, v)
    assert rel2(f.cpu().numpy(), ref) <= 1e-11
