"""Theta_V (Sec. 4) where the kernels' launch shapes have edges: more x-points than resident
blocks of the persistent one-block form (N_k = 8, 16), a last staged batch of a few
x-points (N_k = 32), unequal x axes (the per-axis modulation rows), two nuclei with
unequal charges.  FP64, sampled x-points (the first, the last and seeded ones) against
the oracle's threefold transforms; 1e-12 of max|Theta|, the bound of the other FP64 Theta_V
tests (rounding of about 40 FP64 operations in a chain, measured there at 1e-15)."""
import numpy as np
import pytest
import torch

from oracle import tkm
from paper_2205_02380_amd import inputs, theta

pytestmark = pytest.mark.gpu
NUC = [(0.15, -0.2, 0.05), (-0.4, 0.1, 0.3)]
Z = [1.0, 2.0]


@pytest.mark.parametrize("nk,nx", [(8, (1, 1, 1)), (8, (19, 17, 29)), (16, (7, 9, 11)), (16, (2, 1, 1)), (32, (5, 3, 2)),
                                   (32, (13, 12, 14)), (64, (2, 3, 1))])
def test_theta_edges_of_the_launch_shapes(nk, nx):
    print(f"theta nk={nk} nx={nx}", flush=True)
    kr = 3.2
    grid = inputs.Grid(nx, (-1.0, -1.2, -0.8), (1.1, 1.0, 0.9), (nk,) * 3, (-kr,) * 3, (kr,) * 3)
    f = inputs.gaussian_field(grid, inputs.random_packets(2, 31 + nk), dtype=torch.float64, device="cuda:0")
    with theta.Theta(grid, NUC, Z, dtype="f64") as th:
        out = th.apply(f)
        torch.cuda.synchronize()
    n = grid.cube
    picks = sorted({0, n - 1, *np.random.default_rng(nk).integers(0, n, 3 if nk < 64 else 1).tolist()})
    ff, oo = f.reshape(nk, nk, nk, n), out.reshape(nk, nk, nk, n)
    x = [grid.x_axis(d) for d in range(3)]
    for p in picks:
        i1, i2, i3 = p % nx[0], (p // nx[0]) % nx[1], p // (nx[0] * nx[1])
        fx = ff[..., p].cpu().numpy()
        ref = sum(z * tkm.theta_point(fx, (x[0][i1] - a[0], x[1][i2] - a[1], x[2][i3] - a[2]), grid.k_lo, grid.hk)
                  for a, z in zip(NUC, Z))
        err = np.max(np.abs(oo[..., p].cpu().numpy() - ref)) / np.max(np.abs(ref))
        print(f"  x {p}: {err:.2e}", flush=True)
        assert err < 1e-12
