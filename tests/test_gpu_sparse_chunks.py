"""The patch deposit's chunk sizes for sparse particles, at the lines between them and at chunks
that are not full: the modes equal those of one thread per particle bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _modes(pos, n_mesh, mode):
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(n_mesh, pos.shape[1], 100.0, 8, 8, [0.3] * pos.shape[0])
    binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
    out = torch.empty((n_mesh, n_mesh, n_mesh // 2 + 1, 2), device="cuda")
    for _ in range(2):                       # the registry and the side grid are used again
        ctx.deposit(pos)
    binding.pm_nu_copy_modes(ctx.h, pos.shape[0] - 1, out)
    torch.cuda.synchronize()
    ctx.close()
    return out


@pytest.mark.parametrize("n_mesh,n_part", [
    (64, 1), (64, 1023), (64, 1025), (64, 98304), (64, 98305), (64, 196608), (64, 196609),
    (32, 12288), (32, 12289), (128, 300001)])
@pytest.mark.parametrize("mode", [6, 7, 8])
@pytest.mark.parametrize("compact", [True, False])
def test_sparse_chunks_sum_exactly(n_mesh, n_part, mode, compact):
    rng = np.random.default_rng(n_part)
    pos = rng.random((2, n_part, 3)) * 100.0
    if compact:                              # sorted by coarse cell: chunks that fit a patch
        for b in range(2):
            cell = np.floor(pos[b] / 100.0 * 8).astype(int)
            pos[b] = pos[b][np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2],
                                       kind="stable")]
    pos = torch.from_numpy(pos.astype(np.float32)).cuda()
    assert torch.equal(_modes(pos, n_mesh, mode), _modes(pos, n_mesh, 0))
