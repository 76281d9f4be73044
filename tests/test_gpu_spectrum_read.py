"""A box's spectrum read back: every bin count's last value, and several threads reading
different boxes of one context at once."""
import threading

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library shares)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_kbins", [1, 7, 256, 300])
def test_reading_back_what_was_set(n_kbins):
    """Before a response P_cdm is the set power times and divided by the mode count: two
    roundings each way, 4 x 2^-53."""
    from paper_1209_0461_amd import PMNu, binding
    n_boxes = 3
    ctx = PMNu(32, 8, 128.0, n_kbins, 8, [0.3] * n_boxes)
    _, counts, _ = ctx.bins()
    rng = np.random.default_rng(n_kbins)
    want = [np.where(counts > 0, rng.uniform(1.0, 2.0, n_kbins), 0.0) for _ in range(n_boxes)]
    for b in range(n_boxes):
        binding.pm_nu_set_power(ctx.h, b, want[b])
    wrong = []

    def read(b):
        for _ in range(50):
            got = ctx.spectrum(b)["p_cdm"]
            if not np.all(np.abs(got - want[b]) <= 4 * 2.0 ** -53 * want[b]):
                wrong.append(b)

    threads = [threading.Thread(target=read, args=(b,)) for b in range(n_boxes)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    ctx.close()
