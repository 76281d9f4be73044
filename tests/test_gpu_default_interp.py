"""The interpolation a new context uses, on both sides of the rule's lines: the same accelerations
bit for bit as the other one gives (the same products in the same order)."""
import json

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,n_boxes,n_part,mode,block", [
    (8, 1, 1, 0, 256), (64, 1, 131072, 0, 256), (64, 1, 131073, 0, 512), (32, 2, 1 << 20, 0, 512),
    (32, 2, (1 << 20) + 1, 1, 512), (128, 3, 1 << 20, 0, 256), (128, 3, (1 << 20) + 1, 1, 512)])
def test_default_interpolation(n_mesh, n_boxes, n_part, mode, block):
    from paper_1209_0461_amd import PMNu, binding
    rng = np.random.default_rng(n_part)
    pos = rng.random((n_boxes, n_part, 3)) * 100.0
    pos[:, :n_part // 2] = np.sort(pos[:, :n_part // 2], axis=1)     # compact chunks and others
    pos = torch.from_numpy(pos.astype(np.float32)).cuda()
    ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3] * n_boxes)
    for b in range(n_boxes):
        ctx.set_history(b, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)),
                                pnu_half=np.ones((1, 8)), pnu_half_init=np.ones(8),
                                theta_over_delta_init=np.zeros(8)))
    tuning = json.loads(binding.pm_nu_tuning(ctx.h))
    assert (tuning["interp_mode"], tuning["interp_block"]) == (mode, block)
    acc = [torch.zeros_like(pos) for _ in range(2)]
    ctx.step(pos, acc[0], 0.2)
    binding.pm_nu_set_launch(ctx.h, tuning["deposit_mode"], 256, 1 - mode, 512)
    ctx.step(pos, acc[1], 0.2)
    torch.cuda.synchronize()
    ctx.close()
    assert acc[0].abs().max() > 0 or n_part == 1
    assert torch.equal(acc[0], acc[1])
