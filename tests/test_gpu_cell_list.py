"""The hashed cell list of the lubrication forces where its chains are not the
ordinary ones: many close particles in one cell (more than a pass of the chain
takes), coordinates far from the origin, boxes of one to three cells."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["dense", "far", "one cell", "two cells", "three cells"])
def test_cell_list_forms(orc, form):
    """FP64 sums of at most some hundred terms: 1e-11 (the tolerance of the
    other lubrication tests); the order is fixed, so a repeat is bitwise."""
    import torch
    import paper_1205_6333_amd as sd
    rng = np.random.default_rng(11)
    n, box = 300, None
    if form == "dense":
        x = rng.uniform(0.0, 6.0, size=(n, 3))
    elif form == "far":
        x = W.random_suspension(n, phi=0.3, min_dist=2.02, seed=5) + [3.0e7, -2.0e7, 12345.5]
        x[:3] = [[1e250, 0, 0], [-1e250, 0, 0], [0, 1e30, -1e30]]
    else:
        box = {"one cell": 5.0, "two cells": 7.5, "three cells": 9.5}[form]
        n = 20
        x = rng.uniform(-box, 2 * box, size=(n, 3))
    v = rng.normal(size=(n, 3))
    p, lb = sd.params(box=box), sd.lub(1.0, 1e-3)
    f = sd.lubrication_forces(to_dev3(x), to_dev3(v), params=p, lub_params=lb)
    for _ in range(3):
        assert torch.equal(f, sd.lubrication_forces(to_dev3(x), to_dev3(v), params=p,
                                                    lub_params=lb))
    ref = orc.lubrication_force(orc.params(box=box), orc.lub(1.0, 1e-3), x, v)
    assert np.abs(ref).max() > 0.0
    assert rel2(f.cpu().numpy(), ref) <= 1e-11
