"""FP32 adjoint on either side of the size where its sums are compensated with
every term, and where a block or a chunk of the schedule is partly filled."""
import numpy as np
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("n", [1, 2, 15, 17, 63, 65, 129, 1023, 1024])
def test_fp32_adjoint_sizes(n, overlap):
    """Against the FP64 pass on the same FP32 inputs: 1e-6, as the products (a
    term carries about 2e-7, the sums less)."""
    import torch
    import paper_1205_6333_amd as sd
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, 5.0 * n ** (1.0 / 3.0), size=(n, 3)).astype(np.float32)
    p = sd.params(overlap=overlap)
    dev = [to_dev3(v.astype(np.float64)) for v in
           (x, rng.normal(size=(n, 3)).astype(np.float32), rng.normal(size=(n, 3)).astype(np.float32))]
    a = sd.mobility_adjoint(*[sd.sd_pack(v) for v in dev], params=p)
    b = sd.mobility_adjoint(*[sd.sd_pack(v, sd.SD_FP64) for v in dev], params=p)
    for u, v in zip(a, b):
        if n == 1 and not v.any():
            assert not u.any()
        else:
            assert rel2(u.cpu().numpy(), v.cpu().numpy()) <= 1e-6
    again = sd.mobility_adjoint(*[sd.sd_pack(v) for v in dev], params=p)
    assert all(torch.equal(u, v) for u, v in zip(a, again))
