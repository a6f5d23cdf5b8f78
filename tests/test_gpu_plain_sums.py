"""SD_FP32_PLAIN means plain FP32 sums at every size: its automatic choice runs the
configuration that it names, bit for bit, in products and in steps, and differs
from the compensated sums."""
import pytest

from paper_1205_6333_amd import workloads as W

from gpu_util import rel2, to_dev3, to_dev4

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 333, 3000, 6007, 16383, 16384, 19999])
def test_plain_sums_are_plain(n):
    import torch
    import paper_1205_6333_amd as sd
    x, f = W.random_suspension(n, seed=n), W.gaussian_forces(n, seed=n + 1)
    pos, frc = to_dev4(x, torch.float32), to_dev4(f, torch.float32)
    pos64 = to_dev4(W.round_to_f32(x), torch.float64)
    frc64 = to_dev4(W.round_to_f32(f), torch.float64)
    plain, kahan = sd.SD_FP32_PLAIN, sd.SD_FP32_KAHAN

    def both():
        xd = to_dev3(x)
        sd.sd_run(xd, frc, 1e-2, 3, precision=plain)
        return sd.mobility_apply(pos, frc, precision=plain), xd

    auto = both()
    sd.sd_set_kernel_config(plain, sd.sd_get_kernel_config(plain, n))
    try:
        forced = both()
    finally:
        sd.sd_set_kernel_config(plain, None)
    assert all(torch.equal(a, b) for a, b in zip(auto, forced))
    comp = sd.mobility_apply(pos, frc, precision=kahan)
    ref = sd.mobility_apply(pos64, frc64, precision=sd.SD_FP64).cpu().numpy()
    assert not torch.equal(auto[0], comp)
    # 1e-5 plain, 1e-6 compensated: the tolerances of the other products' tests
    assert rel2(auto[0].cpu().numpy(), ref) <= 1e-5 and rel2(comp.cpu().numpy(), ref) <= 1e-6
