"""Calls of many steps that record diagnostics after every step: the paired SLAB passes
(x1 x2 x3, then x3 x2 x1, ...; K steps in K + 1 passes), which these handles and observed
ones run, their graphs (head, middles of one and four pairs, even and odd tail) and the
CUBE graphs of one and eight steps.  Repeated calls are bitwise equal, on fields of more
units than the chip holds blocks; graph replay equals eager issue bitwise, fields and
history; and every call stays with the FP64 oracle, within the bounds of the other
parity tests: FP64 1e-12 per step, FP32 1e-5, times K / 10 past ten steps."""
import numpy as np
import pytest
import torch

import oracle
from paper_2205_02380_amd import chasm, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, F64 = torch.float32, torch.float64


def _grid(N, nk, kr=2.0):
    return inputs.Grid((N,) * 3, (-N / 4.0,) * 3, (N / 4.0,) * 3, nk, (-kr,) * 3, (kr * 0.9,) * 3)


def _field(grid, seed, dtype):
    return inputs.gaussian_field(grid, inputs.random_packets(3, seed, c_range=(-1.5, 1.5)), dtype=dtype, device=DEV)


@pytest.mark.parametrize("N,M,g,nk,dtype", [(16, 8, 4, 20, F64), (24, 8, 6, 16, F64), (32, 8, 6, 14, F64),
                                            (48, 16, 8, 11, F64), (64, 16, 8, 6, F64), (48, 16, 8, 13, F32),
                                            (64, 16, 8, 8, F32)])
@pytest.mark.parametrize("K", [2, 5])
def test_diagnosed_calls_repeat_bitwise(N, M, g, nk, dtype, K):
    grid = inputs.cubic_grid(N, N / 3.0, nk, 4.0)
    torch.manual_seed(N + K)
    f0 = torch.randn(grid.shape(), dtype=dtype, device=DEV)
    f, first = f0.clone(), None
    kidx = inputs.k_sample(grid, 6 / grid.nkpts, 3)
    with chasm.Advect(f, grid, M, g, 0.02, schedule="slab", reduce_each_step=True) as a:
        for call in range(8):
            f.copy_(f0)
            a.step(K)
            first = f.clone() if first is None else first
            assert torch.equal(f, first), call
    start = np.stack([f0[i3, i2, i1].double().cpu().numpy() for i1, i2, i3 in kidx])
    got = np.stack([first[i3, i2, i1].double().cpu().numpy() for i1, i2, i3 in kidx])
    ref = oracle.advect6d(start, grid.nx, grid.hx, grid.nk, grid.k_lo, grid.hk, (M,) * 3, g, 0.02, K, kidx=kidx)
    assert np.max(np.abs(got - ref)) < (1e-12 * K if dtype == F64 else 1e-5) * np.max(np.abs(ref))


@pytest.mark.parametrize("N,M,g,dtype,sched", [(32, 8, 6, F32, "slab"), (16, 8, 4, F64, "slab"), (48, 16, 8, F32, "slab"),
                                               (32, 8, 6, F32, "cube"), (16, 8, 4, F64, "cube")])
@pytest.mark.parametrize("oop", [False, True])
def test_diagnosed_graphs_equal_eager_bitwise(N, M, g, dtype, sched, oop):
    grid = _grid(N, (4, 4, 2))
    a_out, b_out = _field(grid, 700 + N, dtype), _field(grid, 700 + N, dtype)
    with chasm.Advect(a_out, grid, M, g, 0.05, schedule=sched, reduce_each_step=True, out_of_place=oop) as a, \
            chasm.Advect(b_out, grid, M, g, 0.05, schedule=sched, reduce_each_step=True, out_of_place=oop,
                         graph=True) as b:
        for k in (1, 2, 3, 11, 20, 4):
            a.step(k)
            b.step(k)
            torch.cuda.synchronize()
            assert torch.equal(a_out, b_out), k
        assert np.array_equal(a.history(), b.history())


@pytest.mark.parametrize("N,M,g,dtype,Ks", [(16, 8, 4, F64, (1, 10, 11, 13, 20)), (16, 8, 4, F32, (10, 11, 13, 20)),
                                            (48, 16, 8, F32, (1, 2, 3, 10, 11)), (64, 16, 8, F32, (6, 10, 11)),
                                            (48, 8, 4, F32, (10,)), (48, 16, 8, F64, (4, 11))])
@pytest.mark.parametrize("graph", [False, True])
def test_diagnosed_slab_calls_match_oracle(N, M, g, dtype, Ks, graph):
    grid = _grid(N, (4, 3, 2) if N == 16 else (2, 2, 1))
    dt = 0.35 if N == 16 else 0.2
    for K in Ks:
        print(f"diagnosed slab N={N} M={M} {dtype} K={K} graph={graph}", flush=True)
        f = _field(grid, 720 + N + K, dtype)
        start = f.double().cpu().numpy()
        with chasm.Advect(f, grid, M, g, dt, schedule="slab", reduce_each_step=True, graph=graph) as a:
            a.step(K)
        torch.cuda.synchronize()
        ref = oracle.advect6d(start, grid.nx, grid.hx, grid.nk, grid.k_lo, grid.hk, (M,) * 3, g, dt, K)
        err = float(np.max(np.abs(f.double().cpu().numpy() - ref)) / np.max(np.abs(ref)))
        assert err < (1e-12 * K if dtype == F64 else 1e-5 * max(1, K / 10)), (K, err)
