"""query_sdf_all_lods on the matrix cores: row L is the query at LOD L bit for
bit, at tile remainders and for every width, and a point that is not a number
gets what the per-lane decoder gives it."""
import numpy as np
import pytest

from paper_2101_10994_amd import workloads as W

from cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 63, 257, 4099, 65537])
@pytest.mark.parametrize("m,H,xyz", [(8, 16, False), (16, 64, True), (32, 128, True), (64, 256, True)])
def test_rows(P, m, H, xyz):
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.tiny_shape(), 16, 3, m, H, sigma=0.1, with_xyz=xyz)
    rng = np.random.default_rng(P)
    n = P - P // 3
    pts = np.concatenate([W.points_in_cells(rng, case.ijk, 16, n), W.uniform_points(rng, P - n)])
    x = torch.from_numpy(W.soa(pts.astype(np.float32))).cuda()
    gm = case.gpu_model()
    rows = ngl.query_sdf_all_lods(gm, x)
    for lod in range(1, case.L + 1):
        assert torch.equal(rows[lod - 1], ngl.query_sdf(gm, x, lod)["sdf"]), lod


def test_not_a_number():
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.tiny_shape(), 16, 3, 32, 128, sigma=0.1)
    x = np.zeros((3, 130), np.float32)
    x[0, 5], x[1, 64], x[:, 129] = np.nan, np.inf, -np.inf
    gm = case.gpu_model()
    xd = torch.from_numpy(x).cuda()
    rows = ngl.query_sdf_all_lods(gm, xd)
    ngl.set_option(ngl.OPT_F32_DECODER, 0)
    try:
        lanes = ngl.query_sdf_all_lods(gm, xd)
    finally:
        ngl.set_option(ngl.OPT_F32_DECODER, 1)
    assert torch.equal(torch.isnan(rows), torch.isnan(lanes))
    assert torch.equal(torch.isinf(rows), torch.isinf(lanes))
    f = torch.isfinite(lanes)
    assert (rows[f] - lanes[f]).abs().max() <= 1e-5


@pytest.mark.parametrize("fd,wd", [("f32", "f32"), ("f16", "bf16")])
def test_few_points_are_the_batch(fd, wd):
    """Up to 16 points are one tile and keep their order, more are ordered by
    depth: a point's result is the same bits in any batch."""
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.tiny_shape(), 16, 3, 32, 128, sigma=0.1, feat_dtype=fd, w_dtype=wd)
    rng = np.random.default_rng(9)
    pts = np.concatenate([W.points_in_cells(rng, case.ijk, 16, 200), W.uniform_points(rng, 200)])
    x = torch.from_numpy(W.soa(rng.permutation(pts).astype(np.float32))).cuda()
    gm = case.gpu_model()
    full = ngl.query_sdf(gm, x, 3)["sdf"]
    for n in (1, 15, 16, 17, 64, 272, 273):
        assert torch.equal(ngl.query_sdf(gm, x[:, :n].contiguous(), 3)["sdf"], full[:n]), n
