"""Diagnostics of a field of more items than one launch has threads for (8^3 x-nodes, 16.8
million k-points, 34 GB), on the compiled and the runtime-shape kernels: the mass and the
moments of a constant field are those of the grid."""
import numpy as np
import pytest
import torch

from paper_2205_02380_amd import chasm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("runtime", [False, True])
def test_diagnostics_of_many_items(runtime):
    print(f"diagnostics of 2^24 and more items, runtime={runtime}", flush=True)
    grid = inputs.Grid((8,) * 3, (-1.0, -2.0, -1.5), (1.0, 2.5, 1.0), (256, 256, 257), (-1.0, -2.0, -1.5), (1.0, 2.5, 1.0))
    f = torch.ones(grid.shape(), dtype=torch.float32, device="cuda:0")
    with chasm.Advect(f, grid, 4, 3, 0.0, runtime_shape=runtime) as a:
        mass, l2, moments = a.mass()
    del f
    torch.cuda.empty_cache()
    vol = np.prod([hi - lo for lo, hi in zip(grid.x_lo + grid.k_lo, grid.x_hi + grid.k_hi)])
    # means of the half-open grids' nodes
    means = [lo + 0.5 * (n - 1) * h for lo, n, h in zip(grid.x_lo + grid.k_lo, grid.nx + grid.nk, grid.hx + grid.hk)]
    assert mass == pytest.approx(vol, rel=1e-12)
    assert moments == pytest.approx([m * vol for m in means], rel=1e-12, abs=1e-12 * vol)
