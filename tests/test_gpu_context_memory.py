"""Device memory that a context holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _held(make):
    """What make() returns and the bytes it left allocated."""
    import torch
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    made = make()
    torch.cuda.synchronize()
    return made, before - torch.cuda.mem_get_info()[0]


def test_a_loaded_network_holds_no_training_workspace():
    import torch
    from paper_1209_0461_amd import binding
    from test_gpu_surrogate import _ctx, _data
    ctxs = [_ctx() for _ in range(9)]
    x, y = (torch.from_numpy(v).cuda() for v in _data(512, 3))
    binding.pm_nu_surrogate_init(ctxs[0].h, x, y, 4)
    blob = binding.pm_nu_surrogate_save(ctxs[0].h)
    out = torch.empty_like(y)

    def load():
        for c in ctxs[1:]:
            binding.pm_nu_surrogate_load(c.h, blob)
            binding.pm_nu_surrogate_predict(c.h, x, out)
    # weights, moments and the weight image are 0.6 MB; buffers go in pieces of 2 MB
    assert _held(load)[1] <= 8 * 4 * MB
    binding.pm_nu_surrogate_grad(ctxs[1].h, x, y, torch.empty(35329, device="cuda"))
    for c in ctxs:
        c.close()
