"""The fixed-point mesh of deposit modes 0..5 is left cleared by the first pass that reads it:
later deposits, other modes in between, replays of a captured step and eager steps between them
all see a zero mesh, and the density stays readable."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _pos(n, seed):
    return torch.from_numpy((np.random.default_rng(seed).random((n, 3)) * 100.0)
                            .astype(np.float32)).cuda()


def _context(n_mesh, n_part, stream=None):
    from paper_1209_0461_amd import PMNu
    ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3], stream=stream)
    ctx.set_history(0, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)), pnu_half=np.ones((1, 8)),
                            pnu_half_init=np.ones(8), theta_over_delta_init=np.zeros(8)))
    return ctx


def _density(ctx, n_mesh):
    from paper_1209_0461_amd import binding
    out = torch.empty((n_mesh,) * 3, device="cuda")
    binding.pm_nu_copy_density(ctx.h, 0, out)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n_mesh,fused", [(8, 1), (32, 1), (64, 1), (64, 0), (128, 1), (256, 0)])
def test_deposits_in_turn(n_mesh, fused):
    from paper_1209_0461_amd import binding
    n = 5000
    sets = [_pos(n, s) for s in range(3)]
    alone = []
    for p in sets:
        ctx = _context(n_mesh, n)
        binding.pm_nu_set_launch(ctx.h, 4, 256, 1, 256)
        ctx.deposit(p)
        alone.append(_density(ctx, n_mesh))
        ctx.close()
        assert abs(alone[-1].double().sum().item() / n - 1.0) < 1e-6
    ctx = _context(n_mesh, n)
    binding.pm_nu_set_forward_zy(ctx.h, fused)
    for mode, i in ((4, 0), (0, 1), (6, 2), (1, 2), (4, 0), (4, 1)):
        binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
        ctx.deposit(sets[i])
        got = _density(ctx, n_mesh)
        if mode < 6:
            assert torch.equal(got, alone[i]), (mode, i)
    ctx.close()


def test_replays_and_eager_steps_between_them():
    from paper_1209_0461_amd import binding
    n, n_mesh = 5000, 32
    stream = torch.cuda.Stream()
    pos, acc = _pos(n, 5), torch.zeros((n, 3), device="cuda")
    torch.cuda.synchronize()
    ctx = _context(n_mesh, n, stream.cuda_stream)
    binding.pm_nu_graph_capture(ctx.h, pos, acc, 0.2)
    want = []
    for turn in range(4):
        acc.zero_()
        torch.cuda.synchronize()
        if turn % 2:
            ctx.step(pos, acc, 0.2)
        for _ in range(3):
            binding.pm_nu_graph_launch(ctx.h)
        torch.cuda.synchronize()
        want.append((acc.clone(), _density(ctx, n_mesh)))
    ctx.close()
    assert want[0][0].abs().max() > 0
    for a, d in want[1:]:
        assert torch.equal(a, want[0][0]) and torch.equal(d, want[0][1])
