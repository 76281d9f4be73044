"""The deposit a new context uses, on both sides of the rule's lines: the modes it leads to equal
those of the other deposit bit for bit (exact sums of the same fixed-point weights)."""
import json

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,n_boxes,n_part,default", [
    (32, 1, 40000, 4), (64, 1, 256 * 4096, 4), (64, 1, 256 * 4096 + 1, 6), (64, 2, 128 * 4096, 4),
    (64, 3, 21 * 4096, 4), (64, 3, 22 * 4096, 6), (64, 9, 4096, 6), (128, 1, 16 * 4096, 4),
    (128, 1, 16 * 4096 + 1, 6), (128, 2, 4096, 6), (256, 1, 4096, 6)])
def test_default_deposit(n_mesh, n_boxes, n_part, default):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    rng = np.random.default_rng(n_part)
    pos = torch.from_numpy((rng.random((n_boxes, n_part, 3)) * 100.0).astype(np.float32)).cuda()
    ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3] * n_boxes)
    assert json.loads(binding.pm_nu_tuning(ctx.h))["deposit_mode"] == default
    out = [torch.empty((n_mesh, n_mesh, n_mesh // 2 + 1, 2), device="cuda") for _ in range(2)]
    ctx.deposit(pos)
    binding.pm_nu_copy_modes(ctx.h, n_boxes - 1, out[0])
    binding.pm_nu_set_launch(ctx.h, 10 - default, 256, 1, 256)
    ctx.deposit(pos)
    binding.pm_nu_copy_modes(ctx.h, n_boxes - 1, out[1])
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(out[0], out[1])
