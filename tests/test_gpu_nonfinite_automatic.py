"""Non-finite inputs in the kernels of the automatic choice and in the adjoints:
they propagate to every row that sums a term of them, count as no pair below 2a,
and leave nothing behind; in the products a pair whose r^2 overflows contributes
nothing (in the adjoints, products of two projections overflow with it)."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev4

pytestmark = pytest.mark.gpu

NAMES = {(300, 0): "k_row_f32", (1500, 0): "k_row_f32", (6000, 0): "k_wave_f32",
         (16500, 0): "k_pair_f32_sym_asm", (300, 1): "k_row_f64", (1500, 1): "k_row_f64",
         (4100, 1): "k_wave_f64"}


def _t(prec):
    import torch
    return torch.float64 if prec == 1 else torch.float32


@pytest.mark.parametrize("n,prec", list(NAMES))
def test_products(n, prec):
    import torch
    import paper_1205_6333_amd as sd
    assert sd.sd_kernel_name(prec, n) == NAMES[n, prec]
    x, f = W.random_suspension(n, seed=61), W.gaussian_forces(n, seed=62)
    p = sd.params(overlap=True)

    def apply(a, b):
        return sd.mobility_apply(to_dev4(a, _t(prec)), to_dev4(b, _t(prec)), params=p, precision=prec)

    clean = apply(x, f)
    assert torch.isfinite(clean).all()
    sd.sd_premise_counts(reset=True)
    for i in (0, n // 2, n - 1):
        for bad in ([0.0, np.nan, 0.0], [np.inf, -np.inf, 0.0]):
            y = x.copy()
            y[i] = bad
            assert not torch.isfinite(apply(y, f)).any()
        h = f.copy()
        h[i, 2] = np.inf
        assert not torch.isfinite(apply(x, h)).any()
    assert sd.sd_premise_counts(reset=True) == (0, 0)
    assert torch.equal(apply(x, f), clean)
    # r^2 beyond the range: as a particle so far away that its terms vanish
    y, z = x.copy(), x.copy()
    y[7, 0], z[7, 0] = (1e200, 1e15) if prec == 1 else (1e25, 1e15)
    got, ref = apply(y, f), apply(z, f)
    assert rel2(got.cpu().numpy(), ref.cpu().numpy()) <= (1e-12 if prec == 1 else 1e-6)


@pytest.mark.parametrize("n,prec", [(300, 0), (1500, 0), (300, 1), (1500, 1)])
def test_adjoints(n, prec):
    """The position gradient holds products of every force and cotangent with the
    row's, M lam only the cotangents."""
    import torch
    import paper_1205_6333_amd as sd
    v = [W.random_suspension(n, seed=61), W.gaussian_forces(n, seed=62), W.gaussian_forces(n, seed=63)]

    def adjoint(*a):
        return sd.mobility_adjoint(*[to_dev4(u, _t(prec)) for u in a], precision=prec)

    clean = adjoint(*v)
    assert all(torch.isfinite(u).all() for u in clean)
    for i in (0, n // 2, n - 1):
        for k, bad in ((0, np.nan), (0, np.inf), (1, np.inf), (2, -np.inf)):
            w = [u.copy() for u in v]
            w[k][i, 1] = bad
            gx, gf = adjoint(*w)
            assert not torch.isfinite(gx).all(dim=1).any()
            if k == 1:
                assert torch.equal(gf, clean[1])
            else:
                assert not torch.isfinite(gf).all(dim=1).any()
        assert all(torch.equal(a, b) for a, b in zip(adjoint(*v), clean))
