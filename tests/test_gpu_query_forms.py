"""Queries over 16-bit features take streamed rows or level by level, and points
in order of depth or not, by width, number of levels and number of points: the
bits of the one-lane kernel on both sides of each rule."""
import numpy as np
import pytest

from paper_2101_10994_amd import workloads as W

from cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,H", [(8, 32), (16, 64), (32, 64), (64, 64)])
@pytest.mark.parametrize("fd,wd", [("f16", "f32"), ("bf16", "bf16"), ("f32", "f32")])
def test_forms_are_the_one_lane_bits(fd, wd, m, H):
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.paper_shape(0), 128, 6, m, H, sigma=0.1, feat_dtype=fd, w_dtype=wd)
    gm = case.gpu_model()
    rng = np.random.default_rng(m)
    pts = np.concatenate([W.points_in_cells(rng, case.ijk, 128, 300), W.uniform_points(rng, 300)])
    x = torch.from_numpy(W.soa(rng.permutation(pts).astype(np.float32))).cuda()
    old = ngl.get_option(ngl.OPT_COOP_GATHER)
    try:
        for n in (32, 33, 600):
            xs = x[:, :n].contiguous()
            app = torch.from_numpy(rng.uniform(0, 1, n).astype(np.float32)).cuda()
            for lod in range(1, 7):
                for kw in ({}, dict(alpha_pp=app)) if lod < 6 else ({},):
                    got = []
                    for coop in (0, 1):
                        ngl.set_option(ngl.OPT_COOP_GATHER, coop)
                        got.append(ngl.query_sdf(gm, xs, lod, **kw)["sdf"])
                    assert torch.equal(got[0], got[1]), (n, lod, kw.keys())
    finally:
        ngl.set_option(ngl.OPT_COOP_GATHER, old)
