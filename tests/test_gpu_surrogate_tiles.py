"""The surrogate network's kernels at the edges of their tiles: 32 rows a tile, at most 256
workgroups in a gradient and 512 in a prediction, each walking several tiles beyond that."""
import numpy as np
import pytest

from test_gpu_surrogate import NPARAM, _ctx, _data, _std_inputs, _unpack

pytestmark = pytest.mark.gpu


# tolerances: the layer inputs' 16-bit significand is 1.5e-5 per layer, so 1e-4 of the target
# scale covers three layers; dZ rounded to bfloat16 (2^-9 per value and layer) bounds the
# gradient's relative error by three times that, 6e-3
@pytest.mark.parametrize("n", [1, 31, 32, 33, 256 * 32 - 1, 256 * 32 + 1, 512 * 32 + 33])
def test_predict_and_gradient_at_tile_edges(n):
    import torch
    from paper_1209_0461_amd import binding
    from oracle import mlp
    ctx = _ctx()
    x0, y0 = _data(512, 3)
    binding.pm_nu_surrogate_init(ctx.h, torch.from_numpy(x0).cuda(), torch.from_numpy(y0).cuda(), 4)
    params, mu, sg, ymu, ysg = _unpack(binding.pm_nu_surrogate_save(ctx.h))
    x, y = _data(n, 1000 + n)
    y[3::50] = np.nan                          # rows without a target count for nothing
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    xs = _std_inputs(x, mu, sg)
    out = torch.full((n + 5,), 7.0, device="cuda")
    binding.pm_nu_surrogate_predict(ctx.h, xd, out[:n])
    ref, _ = mlp.forward(params, xs, bf16=True)
    got = out.cpu().numpy()
    assert np.abs(got[:n] - (ref[:, 0] * ysg + ymu)).max() <= 1e-4 * ysg
    assert np.all(got[n:] == 7.0)
    g = torch.full((NPARAM,), np.nan, device="cuda")
    loss = binding.pm_nu_surrogate_grad(ctx.h, xd, yd, g)
    ok = np.isfinite(y)
    m = int(ok.sum())
    ref_loss, ref_g = mlp.mse_loss_and_grads(params, xs[ok], (y[ok].astype(np.float64) - ymu) / ysg,
                                             bf16=True)
    assert loss == pytest.approx(ref_loss * m / n, rel=1e-4)
    flat = np.concatenate([a.reshape(-1) for pair in ref_g for a in pair]) * m / n
    assert np.linalg.norm(g.cpu().numpy() - flat) <= 6e-3 * np.linalg.norm(flat)
    # the same sums in the same order every time
    g2 = torch.empty_like(g)
    binding.pm_nu_surrogate_grad(ctx.h, xd, yd, g2)
    assert torch.equal(g, g2)
    ctx.close()
