"""The exact free-streaming kernel I(x) on the device where its pieces meet: the origin, the
region in which neither the single terms nor the tail dominate, large x, and the ends of the
FP64 range, where products of the terms' denominators would overflow."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def reference(x):
    """4/(3 zeta(3)) sum_{n>=1} (-1)^{n+1} n/(n^2+x^2)^2 in 80-bit arithmetic by the weights
    c_k/d of Cohen, Rodriguez Villegas and Zagier's Algorithm 1 with 64 terms (truncation below
    x^3/5.8^64, rounding below 1e3 x 5e-20); beyond 1e8 its leading term 1/(4 x^4), which is off
    by a relative 1/x^2."""
    x = np.asarray(x, dtype=np.longdouble)
    n = 64
    u0, u1 = np.longdouble(2), np.longdouble(6)
    for _ in range(1, n):
        u0, u1 = u1, 6 * u1 - u0
    d = u1 / 2
    b, c, s = np.longdouble(-1), -d, np.zeros_like(x)
    for k in range(n):
        c = b - c
        s += c / d * (k + 1) / ((k + 1) ** 2 + x * x) ** 2
        b = (k + n) * (k - n) * b / ((k + np.longdouble(0.5)) * (k + 1))
    s = np.where(x > 1e8, 1 / (4 * np.maximum(x, 1) ** 4), s)
    zeta3 = np.longdouble("1.2020569031595942853997381615114500")
    return 4 / (3 * zeta3) * s


@pytest.mark.parametrize("x", [
    np.concatenate([[0.0, 1e-300, 1e-9], np.geomspace(1e-6, 1.0, 400)]),
    np.linspace(1.0, 64.0, 4001),
    np.geomspace(64.0, 1e8, 2000),
    np.array([1e9, 1e17, 1e19, 9.9e34, 1.1e35, 1e60, 1e74]),
], ids=["origin", "middle", "large", "ends"])
def test_series_against_extended_precision(x):
    """Each of the 7 fractions and the tail is rounded in about 8 operations and the sums
    cancel by a factor of up to 15 between them: 8 x 15 x 2^-53 = 1.4e-14."""
    import torch
    from paper_1209_0461_amd import binding
    xd = torch.from_numpy(x).cuda()
    out = torch.empty_like(xd)
    binding.pm_nu_kernel_values(xd, out, series=True)
    got = out.cpu().numpy().astype(np.longdouble)
    assert np.abs(got / reference(x) - 1).max() <= 1.4e-14


def test_series_at_infinity_and_nan():
    import torch
    from paper_1209_0461_amd import binding
    xd = torch.tensor([float("inf"), float("nan"), 1e200], dtype=torch.float64, device="cuda")
    out = torch.empty_like(xd)
    binding.pm_nu_kernel_values(xd, out, series=True)
    v = out.cpu().numpy()
    assert v[0] == 0.0 and np.isnan(v[1]) and v[2] == 0.0
