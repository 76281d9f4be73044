"""Small meshes with many particles: the deposit's chunk size on both sides of the rule's lines sums
the same fixed-point weights as one thread per particle, bit for bit, and the default
interpolation gives the same accelerations as the other one."""
import json

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _positions(n_boxes, n_part, compact):
    rng = np.random.default_rng(n_part)
    pos = rng.random((n_part, 3)) * 100.0
    if compact:                       # sorted by coarse cell: chunks that fit their LDS tile
        cell = np.floor(pos / 12.5).astype(int)
        pos = pos[np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    pos = torch.from_numpy(pos.astype(np.float32)).cuda()
    out = pos[None].repeat(n_boxes, 1, 1)
    out[-1] = torch.roll(pos, 37, 0)                       # the last box has chunks of its own
    return out.contiguous()


def _context(n_mesh, pos):
    from paper_1209_0461_amd import PMNu
    ctx = PMNu(n_mesh, pos.shape[1], 100.0, 8, 8, [0.3] * len(pos))
    for b in range(len(pos)):
        ctx.set_history(b, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)),
                                pnu_half=np.ones((1, 8)), pnu_half_init=np.ones(8),
                                theta_over_delta_init=np.zeros(8)))
    return ctx


# 256 chunks of 4096, a box of 512 particles, and four particles a node at 32^3
@pytest.mark.parametrize("n_mesh,n_boxes,n_part", [
    (8, 1, 255 * 4096), (8, 1, 255 * 4096 + 1), (16, 1, 255 * 4096), (16, 1, 255 * 4096 + 1),
    (16, 300, 512), (16, 300, 513), (32, 8, 4 * 32 ** 3 - 1), (32, 8, 4 * 32 ** 3),
    (32, 7, 4 * 32 ** 3)])
@pytest.mark.parametrize("compact", [True, False])
def test_mode_4_sums_exactly(n_mesh, n_boxes, n_part, compact):
    from paper_1209_0461_amd import binding
    pos = _positions(n_boxes, n_part, compact)
    ctx = _context(n_mesh, pos)
    got = []
    for mode in (0, 4):
        binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
        got.append(torch.empty((n_mesh,) * 3, device="cuda"))
        ctx.deposit(pos)
        binding.pm_nu_copy_density(ctx.h, n_boxes - 1, got[-1])
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("n_mesh,mode", [(8, 0), (16, 0), (32, 1)])
def test_default_interpolation_of_many_particles(n_mesh, mode):
    from paper_1209_0461_amd import binding
    pos = _positions(1, (1 << 21) + 77, True)
    ctx = _context(n_mesh, pos)
    tuning = json.loads(binding.pm_nu_tuning(ctx.h))
    assert (tuning["deposit_mode"], tuning["interp_mode"], tuning["interp_block"]) == (4, mode, 512)
    acc = [torch.zeros_like(pos) for _ in range(2)]
    ctx.step(pos, acc[0], 0.2)
    binding.pm_nu_set_launch(ctx.h, 4, 256, 1 - mode, 512)
    ctx.step(pos, acc[1], 0.2)
    torch.cuda.synchronize()
    ctx.close()
    assert acc[0].abs().max() > 0 and torch.equal(acc[0], acc[1])
