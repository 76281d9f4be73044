"""Results are read from a context whose device is not the current one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_spectrum_while_another_device_is_current():
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    from paper_1209_0461_amd import PMNu
    with torch.cuda.device(0):
        ctx = PMNu(16, 1000, 100.0, 8, 8, [0.3])
        ctx.set_history(0, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)),
                                pnu_half=np.ones((1, 8)), pnu_half_init=np.ones(8),
                                theta_over_delta_init=np.zeros(8)))
        pos = torch.rand((1000, 3), device="cuda") * 100.0
        acc = torch.zeros_like(pos)
        ctx.step(pos, acc, 0.2)
        torch.cuda.synchronize()
        want = ctx.spectrum(0)
    with torch.cuda.device(1):
        got = ctx.spectrum(0)
        assert torch.cuda.current_device() == 1
    with torch.cuda.device(0):
        ctx.close()
    for k in want:
        assert np.array_equal(got[k], want[k])
