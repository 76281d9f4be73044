"""The time grid's way to the device: boxes with histories of different lengths, in contexts of
one to many boxes (one to many workgroups of the upload), respond as a context of their own does,
and again for a second scale factor, whose grid goes through the same staging at once after."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _hist(k, n_nodes, seed):
    rng = np.random.default_rng(seed)
    a = np.geomspace(0.02, 0.4, n_nodes)
    pm = rng.uniform(1.0, 2.0, (n_nodes, k))
    return dict(a=a, pm_half=pm, pnu_half=0.9 * pm, pnu_half_init=0.9 * pm[0],
                theta_over_delta_init=np.zeros(k))


def _respond(n_kbins, hists, powers):
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(16, 8, 128.0, n_kbins, 64, [0.3] * len(hists))
    counts = ctx.bins()[1]
    for b, h in enumerate(hists):
        ctx.set_history(b, h)
        binding.pm_nu_set_power(ctx.h, b, np.where(counts > 0, powers[b], 0.0))
    got = []
    for a in (0.5, 0.6):
        ctx.response(a)
        got.append([ctx.spectrum(b)["pnu_half"] for b in range(len(hists))])
    ctx.close()
    return np.array(got)


@pytest.mark.parametrize("n_boxes", [1, 3, 70])
def test_boxes_of_different_history_lengths(n_boxes):
    k = 5
    hists = [_hist(k, 2 + (11 * b) % 60, b) for b in range(n_boxes)]
    powers = [np.random.default_rng(100 + b).uniform(1.0, 2.0, k) for b in range(n_boxes)]
    got = _respond(k, hists, powers)
    assert np.all(np.isfinite(got)) and got[..., 1:].max() > 0
    for b in (0, n_boxes // 2, n_boxes - 1):
        # one context sums in one wave a bin or four: rounding of sums of at most 500 terms
        alone = _respond(k, [hists[b]], [powers[b]])[:, 0]
        assert np.allclose(got[:, b], alone, rtol=500 * 2.0 ** -53, atol=0)
