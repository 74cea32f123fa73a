"""Several steps in one launch (the cube resident in LDS, the SLAB passes sweeping axis by
axis): a CUBE call of K steps is bitwise the K calls of one step for every shape class,
step count on both sides of the launch's bound of 64 steps, visiting order, placement
and batched stepping of handles with different counts; a SLAB call of 65 steps (a full
launch and a remainder) stays with the FP64 oracle, and a SLAB handle that observes
keeps the field of one that records diagnostics.  Shifts of both signs, zero, and more
than a cell.  The FP64 bound is the 1e-12 per step of the other parity tests; the FP32
bound 1e-5 + 1e-6 per step (rounding of one sweep is about 1e-7)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2205_02380_amd import chasm, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _grid(N, nk=(4, 3, 2), kr=2.0):
    return inputs.Grid((N,) * 3, (-N / 4.0,) * 3, (N / 4.0,) * 3, nk, (-kr,) * 3, (kr * 0.9,) * 3)


def _field(grid, seed, dtype):
    return inputs.gaussian_field(grid, inputs.random_packets(3, seed, c_range=(-1.5, 1.5)), dtype=dtype, device=DEV)


@pytest.mark.parametrize("N,M,g,dtype", [(8, 4, 3, torch.float32), (8, 8, 7, torch.float64), (16, 8, 6, torch.float32),
                                         (16, 4, 8, torch.float64), (24, 12, 6, torch.float32), (24, 8, 6, torch.float64),
                                         (32, 8, 6, torch.float32)])
@pytest.mark.parametrize("dt", [0.1, 0.35])
def test_cube_call_of_many_steps_is_bitwise_the_single_steps(N, M, g, dtype, dt):
    grid = _grid(N)
    for K in (2, 3, 65):
        print(f"cube N={N} M={M} g={g} {dtype} dt={dt} K={K}", flush=True)
        one, many, oop = (_field(grid, 800 + N, dtype) for _ in range(3))
        with chasm.Advect(one, grid, M, g, dt, schedule="cube") as a, \
                chasm.Advect(many, grid, M, g, dt, schedule="cube", graph=True) as b, \
                chasm.Advect(oop, grid, M, g, dt, schedule="cube", out_of_place=True) as c:
            for _ in range(K):
                a.step(1)
            b.step(K)
            c.step(K)
        torch.cuda.synchronize()
        assert torch.equal(one, many) and torch.equal(one, oop), K


def test_step_many_cube_handles_of_different_counts():
    specs = [(16, 8, 6, 0.1, 70), (16, 8, 6, 0.3, 3), (24, 8, 6, 0.2, 5), (16, 8, 6, 0.05, 0), (24, 8, 6, 0.1, 1)]
    fs, advs, refs = [], [], []
    for i, (N, M, g, dt, K) in enumerate(specs):
        grid = _grid(N)
        f, r = _field(grid, 820 + i, torch.float32), _field(grid, 820 + i, torch.float32)
        with chasm.Advect(r, grid, M, g, dt) as a:
            for _ in range(K):
                a.step(1)
        fs.append(f)
        refs.append(r)
        advs.append(chasm.Advect(f, grid, M, g, dt))
    chasm.step_many(advs, [s[4] for s in specs])
    torch.cuda.synchronize()
    for a in advs:
        a.close()
    for f, r in zip(fs, refs):
        assert torch.equal(f, r)


@pytest.mark.parametrize("N,M,g,dtype,K", [(16, 8, 4, torch.float64, 65), (16, 8, 4, torch.float32, 66),
                                           (48, 16, 8, torch.float64, 3), (64, 16, 8, torch.float32, 5),
                                           (64, 16, 8, torch.float64, 2)])
def test_slab_call_of_many_steps_matches_oracle(N, M, g, dtype, K):
    grid = _grid(N, (2, 2, 1) if N > 16 else (3, 2, 2))
    dt = 0.3 if N == 16 else 0.6                     # |alpha| up to 1.2: every shift class
    f = _field(grid, 840 + N, dtype)
    start = f.double().cpu().numpy()
    print(f"slab N={N} {dtype} K={K}", flush=True)
    with chasm.Advect(f, grid, M, g, dt, schedule="slab") as a:
        a.step(K)
    torch.cuda.synchronize()
    ref = oracle.advect6d(start, grid.nx, grid.hx, grid.nk, grid.k_lo, grid.hk, (M,) * 3, g, dt, K)
    err = float(np.max(np.abs(f.double().cpu().numpy() - ref)) / np.max(np.abs(start)))
    print(f"  err {err:.2e}", flush=True)
    assert err < (1e-12 * K if dtype == torch.float64 else 1e-5 + 1e-6 * K)


def test_observed_slab_handle_keeps_the_stepwise_field():
    """Unobserved steps of an observed handle run the paired passes, like those of a handle
    that records diagnostics: the same field, bitwise, before the observed step."""
    grid = _grid(48, (2, 2, 2))
    f, r = _field(grid, 860, torch.float32), _field(grid, 860, torch.float32)
    with chasm.Advect(f, grid, 16, 8, 0.2, schedule="slab", observe=True) as a, \
            chasm.Advect(r, grid, 16, 8, 0.2, schedule="slab", reduce_each_step=True, observe=True) as b:
        a.step(4)
        b.step(4)
        oa, ob = a.observables(), b.observables()
    torch.cuda.synchronize()
    assert torch.equal(f, r)
    for x, y in zip(oa, ob):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("N,M,g,dtype,calls", [(16, 8, 4, torch.float32, 1000), (16, 8, 4, torch.float64, 500),
                                               (32, 8, 6, torch.float32, 100)])
def test_cube_calls_of_many_steps_repeat_bitwise(N, M, g, dtype, calls):
    # a wave that read LDS ahead of another's writes would show now and then only
    grid = _grid(N, (8, 8, 8))
    f0 = _field(grid, 860 + N, dtype)
    f, first, bad = f0.clone(), None, 0
    with chasm.Advect(f, grid, M, g, 0.1, schedule="cube") as a:
        for _ in range(calls):
            f.copy_(f0)
            a.step(4)
            first = f.clone() if first is None else first
            bad += int(not torch.equal(f, first))
    print(f"cube N={N} {dtype}: {bad} of {calls} differ", flush=True)
    assert bad == 0
