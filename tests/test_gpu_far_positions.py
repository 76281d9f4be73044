"""Finite coordinates far outside the box (wrapped, like any outside [0, L)), from a few boxes out to
beyond 2^51 cells, where a coordinate's index no longer fits an FP64 mantissa: every deposit adds
the same fixed-point weights as one thread per particle, bit for bit and with no mass lost, and
every interpolation gives the accelerations of the direct gather."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FAR = [3e9, -4e9, 7e12, -2.3e15, 3e15, -7e17, 1.1e19, 9e24, -2e30, 3.4e38]


def _positions(n_mesh, where):
    """Compact chunks with a far particle every 700; a wave of them; chunks of nothing else."""
    n = 5 * 4096 + 77
    rng = np.random.default_rng(n_mesh)
    pos = rng.random((n, 3)) * 100.0
    cell = np.floor(pos / 100.0 * 8).astype(int)
    pos = pos[np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    pos = pos.astype(np.float32)
    far = np.asarray(FAR, np.float32) * rng.uniform(0.5, 1.0, (n, len(FAR))).astype(np.float32)
    at = {"alone": np.arange(0, n, 700), "wave": np.arange(4096, 4160),
          "chunk": np.arange(8192, 16384)}[where]
    for axis in range(3):
        take = at if axis == 0 else at[rng.random(len(at)) < 0.5]
        pos[take, axis] = far[take, rng.integers(0, len(FAR), len(take))]
    return torch.from_numpy(pos).cuda()


def _step(pos, n_mesh, deposit, interp):
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(n_mesh, len(pos), 100.0, 8, 8, [0.3])
    ctx.set_history(0, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)), pnu_half=np.ones((1, 8)),
                            pnu_half_init=np.ones(8), theta_over_delta_init=np.zeros(8)))
    binding.pm_nu_set_launch(ctx.h, deposit, 256, interp, 256)
    binding.pm_nu_set_keep_density(ctx.h, 1)
    rho, acc = torch.empty((n_mesh,) * 3, device="cuda"), torch.zeros_like(pos)
    ctx.step(pos, acc, 0.2)
    binding.pm_nu_copy_density(ctx.h, 0, rho)
    torch.cuda.synchronize()
    ctx.close()
    return rho, acc


@pytest.mark.parametrize("n_mesh", [16, 64, 256])
@pytest.mark.parametrize("where", ["alone", "wave", "chunk"])
def test_far_coordinates(n_mesh, where):
    pos = _positions(n_mesh, where)
    rho, acc = _step(pos, n_mesh, 0, 0)
    # FP32 nodes, each within half an ulp of the exact sums
    assert abs(rho.double().sum().item() / len(pos) - 1.0) <= 2.0 ** -24
    assert torch.isfinite(acc).all()
    delta = None
    for mode in range(1, 10):
        if mode >= 8 and n_mesh < 32:
            continue
        got, a = _step(pos, n_mesh, mode, (mode - 1) % 3 + 1)
        # forces: the same modes and the same products in the same order
        assert torch.equal(a, acc), (mode, (a - acc).abs().max().item())
        if mode < 6:
            assert torch.equal(got, rho), mode
        else:                         # read back from delta = rho / rho_bar - 1 in FP32
            delta = got if delta is None else delta
            assert torch.equal(got, delta), mode
            bar = len(pos) / n_mesh ** 3
            assert (got.double() - rho.double()).abs().max() <= 2.0 ** -21 * (rho.max() + bar)


@pytest.mark.parametrize("n_mesh", [16, 64])
@pytest.mark.parametrize("hide", [np.nan, np.inf, -np.inf])
def test_far_coordinates_beside_skipped_particles(n_mesh, hide):
    """Particles that are skipped must not hide a far one of their wave or chunk."""
    pos = _positions(n_mesh, "alone")
    n = len(pos)
    for start, count, axis in ((0, 1, 0), (640, 128, 1), (4096, 64, 2), (4199, 3, 0), (8192, 4096, 1)):
        keep = pos[start:start + count:5].clone()
        pos[start:start + count, axis] = float(hide)
        pos[start:start + count:5] = keep
    bad = ~torch.isfinite(pos).all(dim=1)
    assert 0 < int(bad.sum()) < n and (pos[~bad].abs() > 1e9).any()
    rho, acc = _step(pos, n_mesh, 0, 0)
    assert abs(rho.double().sum().item() / (n - int(bad.sum())) - 1.0) <= 2.0 ** -24
    assert (acc[bad] == 0).all() and torch.isfinite(acc).all()
    for mode in range(1, 8):
        got, a = _step(pos, n_mesh, mode, (mode - 1) % 3 + 1)
        assert torch.equal(a, acc), mode
        assert mode > 5 or torch.equal(got, rho), mode
