"""What the tuner takes from its cache file and what it times."""
import json
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context(n_mesh, n_part):
    from paper_1209_0461_amd import PMNu
    ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3])
    ctx.set_history(0, dict(a=np.array([0.1]), pm_half=np.ones((1, 8)), pnu_half=np.ones((1, 8)),
                            pnu_half_init=np.ones(8), theta_over_delta_init=np.zeros(8)))
    return ctx


def _lines(path):
    with open(path) as f:
        return [json.loads(l) for l in f if l.strip()]


def test_line_without_this_version_is_timed_again(tmp_path):
    import torch
    from paper_1209_0461_amd import binding
    n_mesh, n_part = 64, 20000
    pos = torch.rand((n_part, 3), device="cuda") * 100.0
    acc = torch.zeros_like(pos)
    cache = str(tmp_path / "tuning.jsonl")
    ctx = _context(n_mesh, n_part)
    binding.pm_nu_autotune(ctx.h, pos, acc, 0.2, cache)
    ctx.close()
    new = _lines(cache)[0]
    old_keys = [re.sub(r"/v\d+/", "/", new["key"]), re.sub(r"/v\d+/", "/v1/", new["key"])]
    assert new["key"] not in old_keys
    # stored numbers that no timing picks: one thread per particle, and each pass's last tile
    stale = dict(new, deposit_mode=0, deposit_block=64, interp_mode=3, fft=[2, 2, 2, 2, 2, 2])
    with open(cache, "w") as f:
        for k in old_keys:
            f.write(json.dumps(dict(stale, key=k)) + "\n")
    ctx = _context(n_mesh, n_part)
    binding.pm_nu_autotune(ctx.h, pos, acc, 0.2, cache)
    got = json.loads(binding.pm_nu_tuning(ctx.h))
    ctx.close()
    assert got["deposit_block"] != 64                 # 64 is no candidate of the tuner
    after = _lines(cache)
    assert [l["key"] for l in after] == old_keys + [new["key"]]   # lines of others are kept
    assert after[-1]["fft"] == got["fft"]


@pytest.mark.parametrize("n_mesh,n_part", [(32, 3000), (256, 20000)])
def test_density_after_tuning(n_mesh, n_part):
    """The tuner leaves a whole step's density whatever it stored while it timed the passes, and a
    cleared mesh for the next deposit by atomics."""
    import torch
    from paper_1209_0461_amd import binding
    pos = torch.rand((n_part, 3), device="cuda") * 100.0
    acc = torch.zeros_like(pos)
    rho = [torch.empty((n_mesh,) * 3, device="cuda") for _ in range(3)]
    ctx = _context(n_mesh, n_part)
    binding.pm_nu_set_keep_density(ctx.h, 1)
    binding.pm_nu_autotune(ctx.h, pos, acc, 0.2, None)
    binding.pm_nu_copy_density(ctx.h, 0, rho[0])
    for r, mode in ((rho[1], 4), (rho[2], 0)):
        binding.pm_nu_set_launch(ctx.h, mode, 256, 0, 256)
        ctx.deposit(pos)
        binding.pm_nu_copy_density(ctx.h, 0, r)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(rho[1], rho[2])
    # modes 6..9 keep delta in FP32: a node is off by at most 5 roundings of 2^-24
    assert (rho[0].double() - rho[1].double()).abs().max() <= 2.0 ** -21 * rho[1].max()


def test_modes_that_are_the_same_kernel_are_timed_once():
    """256 chunks: modes 7 and 9 launch what 6 and 8 launch, so the tuner never names them."""
    import torch
    from paper_1209_0461_amd import binding
    n_mesh, n_part = 128, 262000
    pos = torch.rand((n_part, 3), device="cuda") * 100.0
    cell = (pos / 12.5).floor().long()
    pos = pos[torch.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2])].contiguous()
    acc = torch.zeros_like(pos)
    for _ in range(6):
        ctx = _context(n_mesh, n_part)
        binding.pm_nu_autotune(ctx.h, pos, acc, 0.2, None)
        assert json.loads(binding.pm_nu_tuning(ctx.h))["deposit_mode"] not in (7, 9)
        ctx.close()
