"""query_sdf_all_lods takes rows of blocks or a lane per point by the size of
the batch and the decoder: each side of that rule gives the bits of its form
(the query at each LOD, or the per-lane option)."""
import numpy as np
import pytest

from paper_2101_10994_amd import workloads as W

from cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,H,fd,P,rows", [
    (8, 32, "f32", 81_920, True), (8, 32, "f32", 81_921, False), (32, 128, "f32", 81_921, True),
    (32, 128, "f16", (1 << 20) + 1, True), (32, 64, "f32", 1 << 20, True), (32, 64, "f32", (1 << 20) + 1, False),
    (64, 256, "f32", 81_921, False), (64, 64, "bf16", 100_003, False), (16, 16, "f32", 40_961, False)])
def test_form(m, H, fd, P, rows):
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.tiny_shape(), 16, 3, m, H, sigma=0.1, feat_dtype=fd)
    rng = np.random.default_rng(P)
    pts = np.concatenate([W.points_in_cells(rng, case.ijk, 16, P // 2), W.uniform_points(rng, P - P // 2)])
    x = torch.from_numpy(W.soa(pts.astype(np.float32))).cuda()
    gm = case.gpu_model()
    got = ngl.query_sdf_all_lods(gm, x)
    if rows:
        ref = torch.stack([ngl.query_sdf(gm, x, lod)["sdf"] for lod in (1, 2, 3)])
    else:
        old = ngl.get_option(ngl.OPT_COOP_GATHER)
        ngl.set_option(ngl.OPT_COOP_GATHER, 0)
        try:
            ref = ngl.query_sdf_all_lods(gm, x)
        finally:
            ngl.set_option(ngl.OPT_COOP_GATHER, old)
    assert torch.equal(got, ref)
