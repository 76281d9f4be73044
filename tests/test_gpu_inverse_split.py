"""The last inverse passes of small meshes: a box by itself (one workgroup per plane and
component) and the same box in a batch of more than 256 planes (one per plane) give the same
accelerations bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _force(pos, n_mesh):
    from paper_1209_0461_amd import PMNu
    n_boxes = pos.shape[0]
    ctx = PMNu(n_mesh, pos.shape[1], 100.0, 8, 8, [0.3] * n_boxes)
    for b in range(n_boxes):
        ctx.set_history(b, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)),
                                pnu_half=np.ones((1, 8)), pnu_half_init=np.ones(8),
                                theta_over_delta_init=np.zeros(8)))
    acc = torch.zeros_like(pos)
    ctx.step(pos, acc, 0.2)
    grids = [torch.empty(n_mesh ** 3, device="cuda") for _ in range(3)]
    from paper_1209_0461_amd import binding
    for axis in range(3):
        binding.pm_nu_copy_force_grid(ctx.h, n_boxes - 1, axis, grids[axis])
    torch.cuda.synchronize()
    ctx.close()
    return acc[-1], torch.stack(grids)


@pytest.mark.parametrize("n_mesh,n_boxes", [(8, 33), (16, 17), (32, 9), (64, 5)])
def test_one_component_a_workgroup(n_mesh, n_boxes):
    rng = np.random.default_rng(n_mesh)
    pos = torch.from_numpy((rng.random((n_boxes, 1000, 3)) * 100.0).astype(np.float32)).cuda()
    batch, alone = _force(pos, n_mesh), _force(pos[-1:].contiguous(), n_mesh)
    assert batch[1].abs().max() > 0
    for b, a in zip(batch, alone):
        assert torch.equal(b, a)
