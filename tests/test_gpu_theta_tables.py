"""Theta_V (Sec. 4) where the kernel tables of the (x1, x2) pairs are made range by range:
more pairs than a table holds (N_k = 16, 32), more x1 nodes than their first sums hold
(N_k = 32), a batch of x-points inside one pair (N_k = 64), several batch members to a pair,
and one to four nuclei of unequal charges.  FP64, sampled x-points (the first, the last and
seeded ones) against the oracle's threefold transforms; 1e-12 of max|Theta|, the bound of the
other FP64 Theta_V tests (rounding of about 40 FP64 operations in a chain)."""
import numpy as np
import pytest
import torch

from oracle import tkm
from paper_2205_02380_amd import inputs, theta

pytestmark = pytest.mark.gpu
NUC = [(0.15, -0.2, 0.05), (-0.4, 0.1, 0.3), (0.7, 0.6, -0.5), (-0.1, -0.8, 0.2)]
Z = [1.0, 2.0, 0.5, 1.5]


@pytest.mark.parametrize("nk,nx,nnuc,nbatch", [(8, (3, 2, 5), 4, 3), (16, (37, 29, 2), 1, 1), (16, (3, 5, 4), 3, 2),
                                               (32, (7, 11, 2), 2, 2), (32, (301, 1, 1), 1, 1), (64, (1, 2, 29), 1, 2)])
def test_theta_tables_by_ranges(nk, nx, nnuc, nbatch):
    print(f"theta nk={nk} nx={nx} nuclei={nnuc} batch={nbatch}", flush=True)
    kr = 3.2
    grid = inputs.Grid(nx, (-1.0, -1.2, -0.8), (1.1, 1.0, 0.9), (nk,) * 3, (-kr,) * 3, (kr,) * 3)
    n = grid.cube
    f = torch.stack([inputs.gaussian_field(grid, inputs.random_packets(2, 31 + nk + b), dtype=torch.float64, device="cuda:0")
                     for b in range(nbatch)])
    with theta.Theta(grid, NUC[:nnuc], Z[:nnuc], dtype="f64", nbatch=nbatch) as th:
        out = th.apply(f)
        torch.cuda.synchronize()
    picks = sorted({0, n - 1, *np.random.default_rng(nk).integers(0, n, 3 if nk < 64 else 1).tolist()})
    x = [grid.x_axis(d) for d in range(3)]
    for b in range(nbatch):
        ff, oo = f[b].reshape(nk, nk, nk, n), out[b].reshape(nk, nk, nk, n)
        for p in picks:
            i1, i2, i3 = p % nx[0], (p // nx[0]) % nx[1], p // (nx[0] * nx[1])
            fx = ff[..., p].cpu().numpy()
            ref = sum(z * tkm.theta_point(fx, (x[0][i1] - a[0], x[1][i2] - a[1], x[2][i3] - a[2]), grid.k_lo, grid.hk)
                      for a, z in zip(NUC[:nnuc], Z))
            err = np.max(np.abs(oo[..., p].cpu().numpy() - ref)) / np.max(np.abs(ref))
            print(f"  b {b} x {p}: {err:.2e}", flush=True)
            assert err < 1e-12
