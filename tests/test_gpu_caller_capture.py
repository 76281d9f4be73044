"""A caller's own capture of pm_nu_deposit as the first deposit of a context: the captured work has
not run when the next eager deposit comes, which must find a cleared mesh all the same, and so
must every replay."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _density(ctx, n_mesh):
    from paper_1209_0461_amd import binding
    out = torch.empty((n_mesh,) * 3, device="cuda")
    binding.pm_nu_copy_density(ctx.h, 0, out)
    torch.cuda.synchronize()
    return out


def _leave_used_memory(n_mesh, n):
    """Contexts whose freed buffers, which a new one may be given, hold no zeros."""
    from paper_1209_0461_amd import PMNu
    pos = torch.rand((n, 3), device="cuda") * 100.0
    ctxs = [PMNu(m, n, 100.0, 8, 8, [0.3]) for m in (n_mesh, 2 * n_mesh, n_mesh)]
    for c in ctxs:
        c.set_history(0, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)), pnu_half=np.ones((1, 8)),
                              pnu_half_init=np.ones(8), theta_over_delta_init=np.zeros(8)))
        c.step(pos, torch.zeros_like(pos), 0.2)
    torch.cuda.synchronize()
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("n_mesh", [16, 32])
@pytest.mark.parametrize("mode", [0, 4])
def test_captured_deposit_before_any_other(n_mesh, mode):
    from paper_1209_0461_amd import PMNu, binding
    n = 5000
    pos = [torch.from_numpy((np.random.default_rng(s).random((n, 3)) * 100.0)
                            .astype(np.float32)).cuda() for s in range(2)]
    want = []
    for p in pos:
        ctx = PMNu(n_mesh, n, 100.0, 8, 8, [0.3])
        binding.pm_nu_set_launch(ctx.h, mode, 256, 0, 256)
        ctx.deposit(p)
        want.append(_density(ctx, n_mesh))
        ctx.close()
        assert abs(want[-1].double().sum().item() / n - 1.0) <= 2.0 ** -24
    _leave_used_memory(n_mesh, n)
    stream = torch.cuda.Stream()
    ctx = PMNu(n_mesh, n, 100.0, 8, 8, [0.3], stream=stream.cuda_stream)
    binding.pm_nu_set_launch(ctx.h, mode, 256, 0, 256)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.deposit(pos[0])
    for turn in range(3):
        ctx.deposit(pos[1])
        torch.cuda.synchronize()
        assert torch.equal(_density(ctx, n_mesh), want[1]), turn
        for _ in range(2):
            with torch.cuda.stream(stream):
                graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(_density(ctx, n_mesh), want[0]), turn
    ctx.close()
