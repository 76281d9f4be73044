"""The FP64 mode sums per k-bin against the same sums over the modes read back: few and many
bins (the copies of the LDS bins go from 16 to 1), empty bins, and every tile of the pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# both sides add the same squares in FP64: at most 2^21 terms of rounding 1.1e-16 in another
# order stay below 1e-12 of the (positive) sum
@pytest.mark.parametrize("n_mesh", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("n_bins", [1, 2, 16, 17, 64, 65, 129, 1024])
def test_binned_power_is_the_sum_over_the_modes(n_mesh, n_bins):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    from oracle import pm
    box = 100.0
    rng = np.random.default_rng(n_mesh + n_bins)
    pos = torch.from_numpy((rng.random((5000, 3)) * box).astype(np.float32)).cuda()
    n2, w = pm.mode_n2_and_weight(n_mesh)
    b = pm.bin_of_n2(n2, pm.bin_edges_n2(n_mesh, n_bins))
    ctx = PMNu(n_mesh, 5000, box, n_bins, 8, [0.3])
    _, counts, _ = ctx.bins()
    modes = torch.empty(n2.shape + (2,), dtype=torch.float32, device="cuda")
    for tile in range(3):
        binding.pm_nu_set_fft_tiles(ctx.h, [0, 0, tile, 0, 0, 0])
        ctx.deposit(pos)
        binding.pm_nu_copy_modes(ctx.h, 0, modes)
        got = ctx.spectrum(0)["p_cdm"]
        d = modes.cpu().numpy().astype(np.float64)
        p = (d[..., 0] ** 2 + d[..., 1] ** 2) * w
        keep = b >= 0
        s = np.bincount(b[keep], weights=p[keep], minlength=n_bins)
        ok = counts > 0
        ref = box ** 3 / float(n_mesh) ** 6 * s[ok] / counts[ok]
        assert np.all(got[~ok] == 0.0)
        assert np.all(np.abs(got[ok] - ref) <= 1e-12 * ref), (tile, n_mesh, n_bins)
    ctx.close()
