"""The device octree at every number of levels against the host build, array
for array: cells on the faces, edges and corners of the grid (their lattice
points lie past the last cell), full grids, scattered and repeated cells,
and cells outside the grid among valid ones."""
import numpy as np
import pytest

from test_gpu_octree_device import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", range(1, 9))
def test_faces_and_scattered_cells(L):
    r = 2 ** (L + 1)
    rng = np.random.default_rng(L)
    cells = rng.integers(0, r, (2000, 3))
    face = rng.integers(0, r, (600, 3))
    face[np.arange(600), rng.integers(0, 3, 600)] = rng.choice([0, r - 1], 600)
    edges = np.array([[x, y, z] for x in (0, r - 1) for y in (0, r - 1) for z in (0, r - 1)])
    line = np.stack([np.arange(r), np.full(r, r - 1), np.full(r, r - 1)], 1)
    ijk = np.concatenate([cells, face, edges, line, cells[:300]])
    compare(ijk[rng.permutation(len(ijk))].astype(np.int32), L)


@pytest.mark.parametrize("L", [1, 2, 3])
def test_full_grid(L):
    r = 2 ** (L + 1)
    g = np.stack(np.meshgrid(*[np.arange(r)] * 3, indexing="ij"), -1).reshape(-1, 3)
    compare(np.random.default_rng(0).permutation(g).astype(np.int32), L)


def test_cells_outside_are_counted_and_skipped():
    import torch
    from paper_2101_10994_amd import ngl
    ijk = np.array([[0, 0, 0], [31, 31, 31], [32, 0, 0], [0, -1, 0], [5, 6, 1 << 30]], np.int32)
    with pytest.raises(ngl.NGLError, match="3 cells outside"):
        ngl.DeviceOctree(torch.from_numpy(ijk).cuda(), 4)
