"""How long the first phase of a trace lasts follows from the number of rays;
every output stays the single launch's, bit for bit, at the edges of that rule
(fewer rays than a wavefront serves, one and two evaluations, the full count)."""
import pytest

from paper_2101_10994_amd import workloads as W

from cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(1, 1), (8, 8), (160, 128), (160, 256), (163, 257), (640, 768), (640, 800)])
def test_default_pause_is_bitwise_the_single_launch(w, h):
    import torch
    from paper_2101_10994_amd import ngl
    case = make_case(W.paper_shape(0), 64, 5, 32, 128, embedded=True)
    gm = case.gpu_model()
    o, d = ngl.camera_rays(W.PAPER.eye, (0, 0, 0), (0, 1, 0), 45.0, w, h)
    for lod, alpha in ((5, 0.0), (3, 0.4)):
        hits = ngl.trace_octree(gm, o, d, (lod + 1 if alpha > 0 else lod) + 1)
        ref = ngl.sphere_trace(gm, o, d, lod, alpha, hits, 100, 1e-4, phased=False)
        g = ngl.sphere_trace(gm, o, d, lod, alpha, hits, 100, 1e-4)
        for key in ("t", "status", "steps", "hit_vox"):
            assert torch.equal(g[key], ref[key]), (lod, alpha, key)
