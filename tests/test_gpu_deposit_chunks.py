"""Deposit variants chosen by the number of particles: every chunk size sums the same 64-bit
fixed-point weights, so the density equals that of one thread per particle bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _density(pos, n_mesh, box, mode):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(n_mesh, pos.shape[0], box, 8, 8, [0.3])
    binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
    ctx.deposit(torch.from_numpy(pos).cuda())
    out = torch.empty((n_mesh,) * 3, dtype=torch.float32, device="cuda")
    binding.pm_nu_copy_density(ctx.h, 0, out)
    torch.cuda.synchronize()
    ctx.close()
    return out.cpu().numpy()


# one chunk of 512 and its neighbours; a mesh above 32^3; the last particle count that takes
# the small chunks on a larger mesh and the first that does not
@pytest.mark.parametrize("n_mesh,n_part", [(8, 1), (32, 511), (32, 512), (32, 513), (32, 40000),
                                           (64, 100003), (64, 511 * 4096), (64, 511 * 4096 + 1)])
@pytest.mark.parametrize("compact", [True, False])
def test_mode_4_chunks_sum_exactly(n_mesh, n_part, compact):
    rng = np.random.default_rng(n_part)
    box = 100.0
    pos = rng.random((n_part, 3)) * box
    if compact:                       # sorted by coarse cell: chunks that fit their LDS tile
        cell = np.floor(pos / box * 8).astype(int)
        pos = pos[np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    pos = pos.astype(np.float32)
    assert np.array_equal(_density(pos, n_mesh, box, 4), _density(pos, n_mesh, box, 0))


def _modes(pos, n_mesh, box, mode):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    ctx = PMNu(n_mesh, pos.shape[0], box, 8, 8, [0.3])
    binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
    p = torch.from_numpy(np.ascontiguousarray(pos)).cuda()
    out = torch.empty((n_mesh, n_mesh, n_mesh // 2 + 1, 2), dtype=torch.float32, device="cuda")
    got = []
    for _ in range(2):                      # the registry and the side grid are used again
        ctx.deposit(p)
        binding.pm_nu_copy_modes(ctx.h, 0, out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    uses = binding.pm_nu_side_grid_uses(ctx.h)
    ctx.close()
    assert np.array_equal(got[0], got[1])
    return got[0], uses


def _spread(n_side, box, n_mesh, sigma, order="morton"):
    from synth import morton_codes
    rng = np.random.default_rng(n_side)
    g = (np.arange(n_side) + 0.5) * (box / n_side)
    q = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    q = np.mod(q + sigma * box / n_mesh * rng.standard_normal(q.shape), box)
    if order == "morton":
        q = q[np.argsort(morton_codes(n_side).astype(np.int64), kind="stable")]
    q = q.astype(np.float32)
    q[q >= box] = 0.0
    return q


# boxes of one pass and of several (tiles of 6144, 9216 or, up to 256 chunks, 18432 nodes), up to the slot's 26624 and
# beyond it; a mesh axis covered whole (C order, small meshes), where the upper neighbour
# wraps; chunks across the mesh's edge; coordinates outside the box; particles that are skipped
@pytest.mark.parametrize("case", ["narrow", "wide", "wider", "c_order", "c_order_256", "edge",
                                  "outside", "not_finite", "tiny_mesh", "crowded", "shuffled",
                                  "many_chunks", "many_chunks_c_order"])
@pytest.mark.parametrize("mode", [6, 7, 8, 9])
def test_patch_deposit_passes_sum_exactly(case, mode):
    n_mesh, box = 64, 128.0
    if case == "narrow":
        pos = _spread(64, box, n_mesh, 0.2)
    elif case == "wide":
        pos = _spread(64, box, n_mesh, 1.0)
    elif case == "wider":
        pos = _spread(64, box, n_mesh, 2.0)[:-77]
    elif case == "c_order":
        pos = _spread(64, box, n_mesh, 0.3, "c")
    elif case == "c_order_256":
        n_mesh = 256
        pos = _spread(128, box, n_mesh, 0.6, "c")[: 40 * 4096 + 5]
        pos[:, 1] *= 0.3
    elif case == "edge":
        pos = np.mod(_spread(64, box, n_mesh, 0.5) - np.float32(0.07 * box), np.float32(box))
    elif case == "outside":
        pos = _spread(64, box, n_mesh, 0.5)
        pos[::3] += np.float32(box)
        pos[1::5] -= np.float32(3 * box)
    elif case == "not_finite":
        pos = _spread(64, box, n_mesh, 0.5)
        pos[5, 0], pos[9000, 1], pos[9001, 2] = np.nan, np.inf, -np.inf
        pos[4096 * 7:4096 * 8] = np.nan
    elif case == "tiny_mesh":
        n_mesh = 32
        pos = _spread(50, box, n_mesh, 0.5)
    elif case == "many_chunks":              # more than 256: the smaller tile
        n_mesh = 128
        pos = _spread(128, box, n_mesh, 1.0)
    elif case == "many_chunks_c_order":
        n_mesh = 128
        pos = _spread(104, box, n_mesh, 0.5, "c")
    elif case == "crowded":
        pos = (0.3 * box + 0.02 * box * np.random.default_rng(1).random((50 * 4096, 3))).astype(np.float32)
    else:
        pos = _spread(40, box, n_mesh, 0.5)
        pos = pos[np.random.default_rng(2).permutation(len(pos))]
    ref, _ = _modes(pos, n_mesh, box, 0)
    got, uses = _modes(pos, n_mesh, box, mode)
    assert np.array_equal(got, ref)
    if case in ("narrow", "wide", "edge", "many_chunks"):
        assert uses == 0                     # every box fits a patch
