"""The default grid and each wave's share of the queue: results do not depend
on how few systems spread over the waves, at sizes around one system, one lane
per wave, and one and two full waves per SIMD."""
import numpy as np
import pytest

import oracle as O
from paper_2011_01740_amd import inputs as I
from tests.test_gpu_rkck import _ens, gpu_ck

pytestmark = pytest.mark.gpu


def _same(a, b):
    for k in ("y", "t", "h", "records", "stats", "status"):
        assert np.array_equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4097, 65535, 65537, 131073])
def test_default_grid_at_any_size(n):
    P, y0 = I.quad_linspace(n)
    o = O.Opts(n_phases=2, n_record=2, rtol=1e-6, atol=1e-6)
    ref = gpu_ck(0, P, y0, o, block=64, grid=64)
    _same(gpu_ck(0, P, y0, o), ref)
    _same(gpu_ck(0, P, y0, o, block=192), ref)
    assert np.all(ref.stats[O.ST_PHASES] == 2)


@pytest.mark.parametrize("n", [5, 1030, 66000, 150001, 262144, 270001])
@pytest.mark.parametrize("launch", [dict(), dict(block=64, refill=5), dict(grid=256),
                                    dict(block=128, grid=512)])
def test_first_share_by_place(n, launch):
    """Grids of whole rounds of the chip give each wave its first share by its
    place in the launch, in index order and in a given one."""
    P, y0 = I.quad_linspace(n)
    o = O.Opts(n_phases=1, n_record=1, rtol=1e-6, atol=1e-6)
    ref = gpu_ck(0, P, y0, o, block=256, grid=3)
    _same(gpu_ck(0, P, y0, o, **launch), ref)
    ens = _ens()
    with ens.Ensemble(0, ens.ENS_RKCK45, n) as e:
        e.set_params(P)
        e.set_order(np.random.default_rng(n).permutation(n).astype(np.int64))
        e.set_state(y0)
        e.solve(t_phase=o.t_phase, n_phases=1, n_record=1, rtol=1e-6, atol=1e-6, **launch)
        assert np.array_equal(e.read(ens.ENS_STATE), ref.y)
        assert np.array_equal(e.read(ens.ENS_STATS), ref.stats)


@pytest.mark.parametrize("n,spread", [(3000, 1), (3000, 1000), (3000, 2999), (3000, 3000),
                                      (200, 70), (70000, 1025), (70000, 66000)])
@pytest.mark.parametrize("launch", [dict(), dict(refill=64), dict(block=64, grid=2, refill=7),
                                    dict(block=128, grid=300)])
def test_share_of_the_head(n, spread, launch):
    P, y0 = I.prv_linspace(n)
    o = O.Opts(n_phases=2, n_record=2, rtol=1e-6, atol=1e-6)
    ref = gpu_ck(3, P, y0, o, block=256, grid=256, budgets=[(2, 3)])
    _same(gpu_ck(3, P, y0, o, spread=spread, budgets=[(2, 3)], **launch), ref)


@pytest.mark.parametrize("block", [64, 128, 192, 256])
@pytest.mark.parametrize("n", [1, 5000, 70000, 400000])
def test_default_grid_gives_every_cu_the_same_blocks(n, block):
    import torch
    P, y0 = I.quad_linspace(n)
    g = gpu_ck(0, P, y0, O.Opts(n_phases=1, n_record=1, rtol=1e-6, atol=1e-6), block=block)
    assert g.launch["block"] == block
    assert g.launch["grid"] % torch.cuda.get_device_properties(0).multi_processor_count == 0
