"""Device memory that a context holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _held(make):
    """What make() returns and the bytes it left allocated."""
    import torch
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    made = make()
    torch.cuda.synchronize()
    return made, before - torch.cuda.mem_get_info()[0]


def test_a_loaded_network_holds_no_training_workspace():
    import torch
    from paper_1209_0461_amd import binding
    from test_gpu_surrogate import _ctx, _data
    ctxs = [_ctx() for _ in range(9)]
    x, y = (torch.from_numpy(v).cuda() for v in _data(512, 3))
    binding.pm_nu_surrogate_init(ctxs[0].h, x, y, 4)
    blob = binding.pm_nu_surrogate_save(ctxs[0].h)
    out = torch.empty_like(y)

    def load():
        for c in ctxs[1:]:
            binding.pm_nu_surrogate_load(c.h, blob)
            binding.pm_nu_surrogate_predict(c.h, x, out)
    # weights, moments and the weight image are 0.6 MB; buffers go in pieces of 2 MB
    assert _held(load)[1] <= 8 * 4 * MB
    binding.pm_nu_surrogate_grad(ctxs[1].h, x, y, torch.empty(35329, device="cuda"))
    for c in ctxs:
        c.close()


# contexts whose patch slots are the compact ones: many boxes of a mesh that deposits by atomics
# unless told otherwise, at a particle a node, sparse, and a mesh smaller than a slot
BATCHES = [(32, 32 ** 3, 128), (32, 12000, 200), (16, 4096, 1500)]


@pytest.mark.parametrize("n_mesh,n_part,n_boxes", BATCHES)
def test_a_batch_holds_little_for_a_deposit_it_does_not_use(n_mesh, n_part, n_boxes):
    from paper_1209_0461_amd import PMNu
    first = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3])          # what the first context loads
    ctx, held = _held(lambda: PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3] * n_boxes))
    first.close()
    ctx.close()
    # bytes a node: two fixed-point meshes, the FP32 density, five complex grids, the forces
    nodes = n_boxes * n_mesh ** 3
    grids = nodes * (8 + 8 + 4 + 5 * 8 * (n_mesh // 2 + 1) / n_mesh + 12)
    patches = n_boxes * -(-n_part // 4096) * 9216 * 8
    small = n_boxes * 64 * 1024                                # partial sums, histories, lists
    assert held <= grids + patches + small + 32 * MB


@pytest.mark.parametrize("n_mesh,n_part,n_boxes", BATCHES)
@pytest.mark.parametrize("order", ["compact", "displaced", "shuffled"])
def test_compact_slots_sum_exactly(n_mesh, n_part, n_boxes, order):
    import torch
    from paper_1209_0461_amd import PMNu, binding
    rng = np.random.default_rng(n_part)
    pos = rng.random((n_part, 3)) * 100.0
    if order != "shuffled":
        cell = np.floor(pos / 12.5).astype(int)
        pos = pos[np.argsort((cell[:, 0] * 8 + cell[:, 1]) * 8 + cell[:, 2], kind="stable")]
    if order == "displaced":
        pos = np.mod(pos + 2.0 * 100.0 / n_mesh * rng.standard_normal(pos.shape), 100.0)
    pos = torch.from_numpy(pos.astype(np.float32)).cuda()[None].repeat(n_boxes, 1, 1).contiguous()
    ctx = PMNu(n_mesh, n_part, 100.0, 8, 8, [0.3] * n_boxes)
    got = {}
    for mode in (0, 6, 7) + ((8, 9) if n_mesh >= 32 else ()):
        binding.pm_nu_set_launch(ctx.h, mode, 256, 1, 256)
        got[mode] = torch.empty((n_mesh, n_mesh, n_mesh // 2 + 1, 2), device="cuda")
        for _ in range(2):
            ctx.deposit(pos)
        binding.pm_nu_copy_modes(ctx.h, n_boxes - 1, got[mode])
        torch.cuda.synchronize()
    ctx.close()
    for mode in got:
        assert torch.equal(got[mode], got[0]), mode
