"""GPU tests of the corner-expanded map layout (dock_grids_bind_corners)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 2, 2, 2), (4, 2, 3, 5), (5, 9, 17, 33), (10, 12, 11, 66)])
def test_corner_layout_ragged(shape):
    """Every word of the layout, on lattices whose axes differ: one cell and one
    type, fewer cells than a block holds, whole and ragged blocks."""
    import torch
    from paper_2410_10447_amd import dock
    M, nz, ny, nx = shape
    maps = np.random.default_rng(nx).normal(size=shape).astype(np.float32)
    G = dock.Grids(torch.from_numpy(maps).cuda(), 0.375, (0.0, 0.0, 0.0))
    G.bind_corners()
    torch.cuda.synchronize()
    want = np.zeros((M - 2, nz - 1, ny - 1, nx - 1, 4, 8), np.float32)
    for t in range(M - 2):
        for j, m in enumerate((t, M - 2, M - 1)):
            for k in range(8):
                dz, dy, dx = k >> 2, (k >> 1) & 1, k & 1
                want[t, ..., j, k] = maps[m, dz:nz - 1 + dz, dy:ny - 1 + dy, dx:nx - 1 + dx]
    got = G.corners[:G.corner_bytes()].view(torch.float32).cpu().numpy().reshape(want.shape)
    assert np.array_equal(got, want)
