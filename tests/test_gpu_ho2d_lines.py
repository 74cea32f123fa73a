"""The x sweep of the 2-D oscillator on lines that take its other branches, against the
FP64 oracle with the bound of the other oscillator tests: more interface rows than the 32
whose coefficients are fetched ahead, more patch solves than threads, stencils of more
than 64 taps, lines of which only two fit in LDS, even node counts, one patch, a last
patch of one cell, and the dense path.  And nodes that are not finite: they reach only the
patches whose stencils hold them and the columns that share their transforms."""
import math

import numpy as np
import pytest
import torch

from oracle import ho2d as oho
from paper_2205_02380_amd import ho2d

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
W = (math.pi / 5.0) ** 2


def run(f0, nx, nk, M, g, tau, steps, inflow="zero"):
    hx, hk = 24.0 / (nx - 1), 12.8 / nk
    f = torch.tensor(f0, dtype=torch.float64, device=DEV)
    with ho2d.HO2D(f, nx, -12.0, hx, nk, -6.4, hk, M, g, W, tau, inflow=inflow) as s:
        s.step(steps)
    torch.cuda.synchronize()
    return f.cpu().numpy()


def start(nx, nk):
    x, k = oho.axes(nx, -12.0, 24.0 / (nx - 1), nk, -6.4, 12.8 / nk)
    return x, k, oho.f0(x[None, :], k[:, None])


@pytest.mark.parametrize("inflow", ["zero", "extrapolate"])
@pytest.mark.parametrize("nx,nk,M,g", [(301, 64, 8, 20), (700, 64, 8, 20), (241, 128, 60, 40), (1021, 64, 60, 20),
                                       (300, 128, 30, 12), (121, 512, 120, 20), (62, 64, 15, 6), (301, 96, 8, 40),
                                       (1021, 66, 60, 33)])
def test_other_lines_match_oracle(nx, nk, M, g, inflow):
    print(f"ho2d nx={nx} nk={nk} patch={M} ghost={g} {inflow}", flush=True)
    x, k, f0 = start(nx, nk)
    got = run(f0, nx, nk, M, g, 0.002, 3, inflow)
    ref = oho.lpc1(f0, x, k, 24.0 / (nx - 1), 12.8 / nk, M, g, W, 0.002, 3, inflow)
    assert np.max(np.abs(got - ref)) < 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("nx,nk,M,g,node", [(121, 128, 30, 6, 50), (121, 512, 30, 6, 50), (121, 96, 30, 6, 50),
                                            (121, 64, 30, 6, 120), (121, 96, 30, 6, 120), (1021, 64, 60, 20, 500)])
def test_an_infinite_node_stays_within_its_patches(nx, nk, M, g, node):
    # the node's patch, the patches with an interface within g of it, and a column on each
    # side: a shift of less than a cell and the neighbour in the pair of a transform
    print(f"ho2d infinite node nx={nx} nk={nk} node={node}", flush=True)
    x, k, f0 = start(nx, nk)
    P = -(-(nx - 1) // M)
    iface = [min(q * M, nx - 1) for q in range(P + 1)]
    hit = [l for l in range(P) if iface[l] - g <= node <= iface[l + 1] + g]
    lo, hi = iface[hit[0]] - 1, iface[hit[-1] + 1] + 1
    bad = f0.copy()
    bad[3, node] = np.inf
    got = run(bad, nx, nk, M, g, 1e-4, 1)
    ref = oho.lpc1(f0, x, k, 24.0 / (nx - 1), 12.8 / nk, M, g, W, 1e-4, 1)
    assert not np.isfinite(got[:, node]).any()
    far = (np.arange(nx) < lo) | (np.arange(nx) > hi)
    assert far.any() and np.isfinite(got[:, far]).all()
    assert np.max(np.abs(got - ref)[:, far]) < 1e-11 * np.max(np.abs(ref))
