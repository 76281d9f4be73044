"""Deposit variants chosen by the number of particles: every chunk size sums the same 64-bit
fixed-point weights, so the density equals that of one thread per particle bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _density(pos, n_mesh, box, mode):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(n_mesh, pos.shape[0], box, 8, 8, [0.3])
    binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
    ctx.deposit(torch.from_numpy(pos).cuda())
    out = torch.empty((n_mesh,) * 3, dtype=torch.float32, device="cuda")
    binding.pm_nu_copy_density(ctx.h, 0, out)
    torch.cuda.synchronize()
    ctx.close()
    return out.cpu().numpy()


# one chunk of 512 and its neighbours; a mesh above 32^3; the last particle count that takes
# the small chunks on a larger mesh and the first that does not
@pytest.mark.parametrize("n_mesh,n_part", [(8, 1), (32, 511), (32, 512), (32, 513), (32, 40000),
                                           (64, 100003), (64, 511 * 4096), (64, 511 * 4096 + 1)])
@pytest.mark.parametrize("compact", [True, False])
def test_mode_4_chunks_sum_exactly(n_mesh, n_part, compact):
    rng = np.random.default_rng(n_part)
    box = 100.0
    pos = rng.random((n_part, 3)) * box
    if compact:                       # sorted by coarse cell: chunks that fit their LDS tile
        cell = np.floor(pos / box * 8).astype(int)
        pos = pos[np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    pos = pos.astype(np.float32)
    assert np.array_equal(_density(pos, n_mesh, box, 4), _density(pos, n_mesh, box, 0))
