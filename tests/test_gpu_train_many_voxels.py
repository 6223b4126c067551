"""A training step over more than 2^26 voxels in all levels, where one
wavefront per voxel is more threads than a launch takes: its gradients are the
sum of those of its two halves, which are small enough to take the path that
reads the records directly."""
import pytest

pytestmark = pytest.mark.gpu


def test_gradients_are_the_halves():
    import torch
    from paper_2101_10994_amd import ngl
    if torch.cuda.mem_get_info()[0] < 96 << 30:
        pytest.skip("needs 96 GiB of device memory")
    L, m, H, P = 8, 8, 32, 6000
    r = lambda n: torch.arange(n, dtype=torch.int32, device="cuda")
    cells = torch.stack(torch.meshgrid(r(500), r(512), r(256), indexing="ij"), -1).reshape(-1, 3)
    tree = ngl.DeviceOctree(cells, L)
    del cells
    assert sum(int(n) for n in tree.nvox[2:]) > 1 << 26 > max(int(n) for n in tree.nvox)
    gen = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *k: torch.randn(k, generator=gen, device="cuda")
    gm = ngl.Model(tree, [0.1 * rnd(int(n), m) for n in tree.ncorner], [0.3 * rnd(H, m + 3) for _ in range(L)],
                   [0.1 * rnd(H) for _ in range(L)], [0.3 * rnd(H) for _ in range(L)], 0.1 * rnd(L))
    x = (torch.rand((3, P), generator=gen, device="cuda") * 2 - 1).contiguous()
    up = rnd(L, P)
    whole = ngl.backward_all_lods(gm, x, up)
    a, b = (ngl.backward_all_lods(gm, x[:, s].contiguous(), up[:, s].contiguous()) for s in (slice(0, 3000), slice(3000, P)))
    for g, u, v in zip(whole.dfeat, a.dfeat, b.dfeat):
        # 24-bit sums of the same terms in another order
        ref = u + v
        assert (g - ref).abs().max() <= 1e-5 * ref.abs().max()
        assert ref.abs().max() > 0
