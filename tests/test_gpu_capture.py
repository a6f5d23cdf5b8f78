"""Calls captured into the caller's own HIP graph (after a first call, which
allocates the library's workspace): every replay on new inputs equals the eager
call, with eager work on other inputs between the replays."""
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import to_dev3, to_dev4

pytestmark = pytest.mark.gpu


def _replays(call, inputs, others, outputs):
    """inputs: the captured call's buffers; others: sets of values for them."""
    import torch
    for buf, val in zip(inputs, others[0]):
        buf.copy_(val)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    for buf, val in zip(inputs, others[0]):
        buf.copy_(val)
    with torch.cuda.graph(g):
        call()
    for vals in others + others[::-1]:
        for buf, val in zip(inputs, vals):
            buf.copy_(val)
        call()
        want = [o.clone() for o in outputs]
        for o in outputs:
            o.zero_()
        for buf, val in zip(inputs, vals):
            buf.copy_(val)
        g.replay()
        torch.cuda.synchronize()
        for o, w in zip(outputs, want):
            assert torch.isfinite(w).all() and torch.equal(o, w)


@pytest.mark.parametrize("n,prec", [(200, 0), (200, 1), (1400, 0), (6000, 0), (4100, 1), (16500, 0),
                                    (3000, 2)])
@pytest.mark.parametrize("box", [False, True])
def test_product(n, prec, box):
    import torch
    import paper_1205_6333_amd as sd
    dt = torch.float64 if prec == 1 else torch.float32
    L = W.box_side(n, 0.05)
    p = sd.params(overlap=True, box=L if box else None)
    sets = [[to_dev4(W.random_suspension(n, seed=s), dt), to_dev4(W.gaussian_forces(n, seed=s), dt)]
            for s in (1, 2)]
    bufs = [torch.empty_like(v) for v in sets[0]]
    vel = torch.zeros((n, 3), dtype=torch.float64, device=bufs[0].device)
    _replays(lambda: sd.mobility_apply(*bufs, vel, params=p, precision=prec), bufs, sets, [vel])


@pytest.mark.parametrize("n,prec", [(200, 0), (1100, 0), (1100, 1)])
def test_adjoint(n, prec):
    import torch
    import paper_1205_6333_amd as sd
    dt = torch.float64 if prec == 1 else torch.float32
    sets = [[to_dev4(v, dt) for v in (W.random_suspension(n, seed=s), W.gaussian_forces(n, seed=s),
                                      W.gaussian_forces(n, seed=s + 5))] for s in (1, 2)]
    bufs = [torch.empty_like(v) for v in sets[0]]
    gx = torch.zeros((n, 3), dtype=torch.float64, device=bufs[0].device)
    gf = torch.zeros_like(gx)
    _replays(lambda: sd.mobility_adjoint(*bufs, gx, gf, precision=prec), bufs, sets, [gx, gf])


@pytest.mark.parametrize("n,prec", [(200, 0), (6000, 0), (4100, 1), (16500, 0)])
@pytest.mark.parametrize("lub", [False, True])
def test_steps(n, prec, lub):
    """Five Euler steps, with and without lubrication."""
    import torch
    import paper_1205_6333_amd as sd
    f = W.gaussian_forces(n, seed=9)
    frc = to_dev3(f) if lub else to_dev4(f, torch.float64 if prec == 1 else torch.float32)
    sets = [[to_dev3(W.random_suspension(n, min_dist=2.3, seed=s)),
             to_dev3(0.1 * W.gaussian_forces(n, seed=s))] for s in (1, 2)]
    x, v = [torch.empty_like(t) for t in sets[0]]
    if lub:
        call = lambda: sd.sd_run_lub(x, frc, v, 1e-3, 5, precision=prec)
    else:
        call = lambda: sd.sd_run(x, frc, 1e-3, 5, precision=prec)
    _replays(call, [x, v], sets, [x])
