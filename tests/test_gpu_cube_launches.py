"""CUBE calls of a few steps around the counts from which a launch takes several of them
(they differ with the type, the size of the field and shifts of a cell or more): every
call, and every call of several handles with their own counts, is bitwise the same
number of calls of one step."""
import pytest
import torch

from paper_2205_02380_amd import chasm, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _job(N, nk, dtype, seed):
    grid = inputs.Grid((N,) * 3, (-N / 4.0,) * 3, (N / 4.0,) * 3, nk, (-2.0,) * 3, (1.8,) * 3)
    torch.manual_seed(seed)
    return grid, torch.randn(grid.shape(), dtype=dtype, device=DEV)


@pytest.mark.parametrize("N,nk,dtype", [(8, (8, 8, 8), torch.float32), (8, (22, 21, 20), torch.float32),
                                        (16, (4, 4, 4), torch.float32), (16, (11, 10, 10), torch.float32),
                                        (24, (8, 7, 7), torch.float32), (32, (3, 3, 3), torch.float32),
                                        (32, (6, 5, 5), torch.float32), (16, (9, 8, 8), torch.float64)])
@pytest.mark.parametrize("dt", [0.1, 0.6])        # shifts within a cell, and of up to 2.4
def test_calls_of_a_few_steps_equal_single_steps(N, nk, dtype, dt):
    print(f"cube N={N} nk={nk} {dtype} dt={dt}", flush=True)
    grid, f0 = _job(N, nk, dtype, N + nk[0])
    M, g = (4, 3) if N == 8 else (8, 6)
    f, one = f0.clone(), f0.clone()
    with chasm.Advect(f, grid, M, g, dt, schedule="cube") as a, chasm.Advect(one, grid, M, g, dt, schedule="cube") as b:
        for K in (2, 3, 4, 5, 6, 7, 8):
            a.step(K)
            for _ in range(K):
                b.step(1)
            torch.cuda.synchronize()
            assert torch.equal(f, one), K


def test_handles_of_different_counts_share_launches_bitwise():
    specs = [(0.1, 20), (0.6, 3), (0.6, 9), (0.1, 2), (0.3, 66), (0.6, 1)]
    jobs = [_job(16, (11, 10, 10), torch.float32, 40 + i) for i in range(len(specs))]
    refs = []
    for (grid, f0), (dt, K) in zip(jobs, specs):
        r = f0.clone()
        with chasm.Advect(r, grid, 8, 6, dt) as a:
            for _ in range(K):
                a.step(1)
        refs.append(r)
    advs = [chasm.Advect(f, grid, 8, 6, dt) for (grid, f), (dt, _) in zip(jobs, specs)]
    chasm.step_many(advs, [K for _, K in specs])
    torch.cuda.synchronize()
    for a in advs:
        a.close()
    for (_, f), r in zip(jobs, refs):
        assert torch.equal(f, r)
