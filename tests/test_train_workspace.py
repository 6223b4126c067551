"""A training workspace serves every smaller batch of its model: its size does
not fall as the batch grows (host only: a model view with null-sized tables
is enough for the size)."""
import ctypes as C

import pytest

from paper_2101_10994_amd import ngl


def model_view(m, h, xyz, L, nvox):
    s, dummy = ngl.ngl_model(), (C.c_float * 8)()
    at = (C.addressof(dummy) + 15) // 16 * 16
    s.num_lods, s.feat_dim, s.hidden, s.with_xyz, s.feat_dtype, s.w_dtype = L, m, h, xyz, 0, 0
    for d in range(L + 2):
        s.nvox[d] = min(8 ** d, nvox)
        s.cell[d] = s.parent[d] = s.child_mask[d] = s.first_child[d] = at
    for l in range(L):
        s.ncorner[l] = 2 * s.nvox[l + 2]
        s.corners[l] = s.feat[l] = s.W1[l] = s.b1[l] = s.w2[l] = s.corner_adj_off[l] = s.corner_adj[l] = at
    s.b2 = at
    return s, dummy


@pytest.mark.parametrize("m,h,xyz,L", [(32, 128, 1, 5), (8, 32, 0, 3), (16, 64, 1, 8), (64, 256, 1, 5), (32, 16, 1, 1)])
@pytest.mark.parametrize("nvox", [1, 3000, 400_000])
def test_size_grows_with_the_batch(m, h, xyz, L, nvox):
    s, keep = model_view(m, h, xyz, L, nvox)
    nb, last = C.c_size_t(), 0
    edges = [1 << k for k in range(20)] + [16296, 4096, 16384, 262144, 393216]
    for P in sorted({max(0, e + d) for e in edges for d in (-65, -64, -1, 0, 1, 63, 64, 65)}):
        assert ngl.lib().ngl_train_workspace(C.addressof(s), P, C.addressof(nb)) == 0, ngl.lib().ngl_last_error()
        assert nb.value >= last, P
        last = nb.value
