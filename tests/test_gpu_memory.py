"""Device memory: a call that cannot have the memory it needs fails by itself, and later
calls work; and no field is allocated that nothing uses."""
import pytest
import torch

from paper_2205_02380_amd import chasm, ho2d, inputs, theta

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_a_failed_create_leaves_no_error_behind():
    big = inputs.Grid((1000, 1000, 1000), (-1.0,) * 3, (1.0,) * 3, (8, 8, 8), (-4.0,) * 3, (4.0,) * 3)   # 2 TB
    small = inputs.Grid((4, 4, 4), (-1.0,) * 3, (1.0,) * 3, (8, 8, 8), (-4.0,) * 3, (4.0,) * 3)
    f = torch.ones(small.shape(), device=DEV)
    for again in range(2):
        with pytest.raises(chasm.ChasmError) as e:
            theta.Theta(big, [(0.0, 0.0, 0.0)])
        assert e.value.status == chasm.CHASM_ENOMEM
        with theta.Theta(small, [(0.3, 0.2, 0.1)]) as t:
            out = t.apply(f)
        assert torch.isfinite(out).all()
        wide = inputs.Grid((16, 16, 16), (-1.0,) * 3, (1.0,) * 3, (256, 256, 100), (-4.0,) * 3, (4.0,) * 3)
        d = chasm.make_desc(wide, 8, 6, 0.02, flags=chasm.CHASM_FLAG_OUT_OF_PLACE | chasm.CHASM_FLAG_REDUCE_EACH_STEP,
                            nbatch=16)                                                          # 1.7 TB
        with pytest.raises(chasm.ChasmError) as e:
            chasm.chasm_advect_create(d, f.data_ptr(), 0)
        assert e.value.status == chasm.CHASM_ENOMEM
        grid = inputs.cubic_grid(16, 8.0, 4, 2.0)
        g = torch.ones(grid.shape(), device=DEV)
        with chasm.Advect(g, grid, 8, 6, 0.02) as a:
            a.step(1)
        torch.cuda.synchronize()


def test_marginals_without_memory_fail_again():
    # room for the item rows (4.0 GB) but not for their sums (3.8 GB) as well
    grid = inputs.Grid((2, 2, 70), (-1.0,) * 3, (1.0,) * 3, (1, 1, 6750000), (-1.0,) * 3, (1.0,) * 3)
    f = torch.zeros(grid.shape(), device=DEV)
    with chasm.Advect(f, grid, (1, 1, 15), 1, 0.02) as a:
        torch.cuda.empty_cache()
        filler = torch.empty(torch.cuda.mem_get_info()[0] - (9 << 29), dtype=torch.uint8, device=DEV)
        for again in range(2):
            with pytest.raises(chasm.ChasmError) as e:
                a.marginals()
            assert e.value.status == chasm.CHASM_ENOMEM
        del filler
    del f
    torch.cuda.empty_cache()


def _taken(make):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    with make():
        return before - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("kw,field", [(dict(), False), (dict(observe=True), False), (dict(reduce_each_step=True), True),
                                      (dict(schedule="slab"), True)])
def test_stage_field_only_where_steps_use_it(kw, field):
    grid = inputs.cubic_grid(32, 12.0, 12, 4.0)
    f = torch.zeros(grid.shape(), device=DEV)                    # 226 MB
    base = _taken(lambda: chasm.Advect(f, grid, 8, 6, 0.02, **kw))
    more = _taken(lambda: chasm.Advect(f, grid, 8, 6, 0.02, out_of_place=True, **kw)) - base
    size = f.numel() * 4
    # small buffers share pieces of some MB: the difference is not exact
    assert (more > size // 8 * 7) if field else (more < size // 8), (more, size)


def test_oscillator_fields_of_its_path():
    # transforms: two pairs of fields; dense: the predictor and its derivative as well
    def fields(nk):
        f = torch.zeros((nk, 1021), dtype=torch.float64, device=DEV)
        return _taken(lambda: ho2d.HO2D(f, 1021, -12.0, 0.02, nk, -6.4, 12.8 / nk, 60, 20, 0.4, 1e-4)) / (f.numel() * 8.0)
    assert 4.0 <= fields(1024) < 5.5
    assert fields(1026) >= 6.0
