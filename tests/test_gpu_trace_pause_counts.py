"""Which rays a phased trace parks: those that run on after the pause count
that was set, whatever the number of rays, and only the default count follows
their number.  The workspace begins with the rays parked by each phase."""
import pytest

from paper_2101_10994_amd import workloads as W

from cases import make_case

pytestmark = pytest.mark.gpu


def trace(gm, o, d, hits, steps, pause1, pause2=0):
    """steps per ray and the rays parked by the first and second phase
    (-1, -1 where the trace was one launch)."""
    import torch
    from paper_2101_10994_amd import ngl
    keys, old = (ngl.OPT_TRACE_PAUSE1, ngl.OPT_TRACE_PAUSE2), None
    old = [ngl.get_option(k) for k in keys]
    try:
        for k, v in zip(keys, (pause1, pause2)):
            ngl.set_option(k, v)
        g = ngl.sphere_trace(gm, o, d, gm.num_lods, 0.0, hits, steps, 1e-4)
        g["ws"].fill_(255)
        g = ngl.sphere_trace(gm, o, d, gm.num_lods, 0.0, hits, steps, 1e-4, out=g)
        return g["steps"], [int(v) for v in g["ws"][:8].view(torch.int32)]
    finally:
        for k, v in zip(keys, old):
            ngl.set_option(k, v)


def scene(w, h):
    from paper_2101_10994_amd import ngl
    gm = make_case(W.paper_shape(0), 32, 4, 16, 64, embedded=True).gpu_model()
    o, d = ngl.camera_rays(W.PAPER.eye, (0, 0, 0), (0, 1, 0), 45.0, w, h)
    return gm, o, d, ngl.trace_octree(gm, o, d, 5)


def runs_on(steps, k):
    """A ray parked after k evaluations has at least k, one with more was parked."""
    return int((steps > k).sum()), int((steps >= k).sum())


@pytest.mark.parametrize("w,h", [(96, 64), (384, 384)])
def test_counts_are_obeyed(w, h):
    s = scene(w, h)
    for p in (2, 9, 16, 23, 25):
        steps, parked = trace(*s, 100, p)
        lo, hi = runs_on(steps, p)
        assert 0 < lo <= parked[0] <= hi and parked[1] == 0, (p, parked, lo, hi)
    steps, parked = trace(*s, 100, 24)
    lo, hi = runs_on(steps, max(1, w * h // 20480))
    assert lo <= parked[0] <= hi


def test_second_count_not_above_the_first_is_ignored():
    s = scene(384, 384)
    assert trace(*s, 100, 24, 16)[1] == trace(*s, 100, 24, 0)[1]
    steps, parked = trace(*s, 100, 24, 30)  # above: both stand
    for p, n in zip((24, 30), parked):
        lo, hi = runs_on(steps, p)
        assert lo <= n <= hi


def test_short_traces_are_one_launch():
    s = scene(96, 64)
    for steps in (1, 2, 8, 24):
        assert trace(*s, steps, 24)[1][1] == -1, steps
    assert trace(*s, 25, 24)[1][1] == 0


def test_late_pauses_of_a_batch():
    """Counts that the default no longer reaches on few rays give the single
    launch's outputs bit for bit."""
    import torch
    from paper_2101_10994_amd import ngl
    from test_gpu_batch import phased_batch_run
    old = ngl.get_option(ngl.OPT_TRACE_PAUSE1)
    try:
        ngl.set_option(ngl.OPT_TRACE_PAUSE1, 0)
        ref = phased_batch_run()
        for pause in (25, 9):
            ngl.set_option(ngl.OPT_TRACE_PAUSE1, pause)
            got = phased_batch_run()
            for key in ("t", "status", "steps", "hit_vox"):
                assert torch.equal(got[key], ref[key]), (pause, key)
    finally:
        ngl.set_option(ngl.OPT_TRACE_PAUSE1, old)
