"""Every deposit mode adds the same fixed-point weights: a set of particles on which a fraction
from a fused multiply-subtract moved a weight by one unit and, through it, 1843 modes by an ulp."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_modes_agree(mode):
    from paper_1209_0461_amd import PMNu, binding
    n_mesh, n_part = 64, 196608
    rng = np.random.default_rng(n_part)
    pos = rng.random((2, n_part, 3)) * 100.0
    for b in range(2):
        cell = np.floor(pos[b] / 100.0 * 8).astype(int)
        pos[b] = pos[b][np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    pos = torch.from_numpy(pos.astype(np.float32)).cuda()
    got = []
    for m in (0, mode):
        ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3] * 2)
        binding.pm_nu_set_launch(ctx.h, m, 256, 1, 256)
        out = torch.empty((n_mesh, n_mesh, n_mesh // 2 + 1, 2), device="cuda")
        ctx.deposit(pos)
        binding.pm_nu_copy_modes(ctx.h, 1, out)
        torch.cuda.synchronize()
        ctx.close()
        got.append(out)
    assert torch.equal(got[0], got[1])
