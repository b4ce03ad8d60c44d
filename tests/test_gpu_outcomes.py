"""The rare outcomes of an adaptive attempt, which the kernel keeps apart from
the common path: the step cap at any attempt (also one that ends a phase or
retries an event), and non-finite states in any component, against the
oracle and against the kernel's own longer solves.  Every comparison is exact."""
import numpy as np
import pytest

import oracle as O
from paper_2011_01740_amd import inputs as I
from tests.parity import CK_ATOL, CK_RTOL, PERTURB, close, per_system, sensitivity_mask
from tests.test_gpu_rkck import _ens, gpu_ck

pytestmark = pytest.mark.gpu

SCHEMES = [O.CASH_KARP, O.DORMAND_PRINCE]


def _solver(scheme):
    ens = _ens()
    return ens.ENS_RKDP45 if scheme == O.DORMAND_PRINCE else ens.ENS_RKCK45


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("model", [0, 2, 3])
@pytest.mark.parametrize("cap", [1, 2, 17, 64, 301])
def test_step_cap_at_any_attempt(model, scheme, cap):
    n = 70
    if model == 0:
        P, y0, sh, t_phase = *I.quad_linspace(n), None, 0.05
    elif model == 2:
        P, y0 = I.km_grid(7, 10)
        sh, t_phase = list(I.KM_WATER), 0.02
    else:
        P, y0 = I.prv_linspace(n)
        sh, t_phase = list(I.PRV_DEFAULT), 1.0
    o = O.Opts(n_phases=30, n_record=4, max_steps=cap, t_phase=t_phase, scheme=scheme)
    g = gpu_ck(model, P, y0, o, shared=sh, solver=_solver(scheme))
    a = O.rkck45(model, P, None if sh is None else np.array(sh), y0, o)
    total = [r.stats[O.ST_ACCEPTED] + r.stats[O.ST_REJECTED] + r.stats[O.ST_EVRETRY] for r in (g, a)]
    assert np.array_equal(*total) and np.all(total[0] <= cap)
    assert np.array_equal(g.status & ~O.SYS_DT_MIN, a.status & ~O.SYS_DT_MIN)
    assert np.array_equal(g.stats[O.ST_PHASES], a.stats[O.ST_PHASES])
    assert np.array_equal(g.stats[O.ST_NRHS], a.stats[O.ST_NRHS])
    # (a capped system stops at the time its steps reached, which follows the
    # step sizes' rounding: its state is checked below, against its own)


@pytest.mark.parametrize("scheme,model", [(O.CASH_KARP, 0), (O.CASH_KARP, 2), (O.CASH_KARP, 3),
                                          (O.DORMAND_PRINCE, 0), (O.DORMAND_PRINCE, 3)])
@pytest.mark.parametrize("cap", [1, 17, 301])
def test_two_capped_solves_are_one(model, scheme, cap):
    """Stopped at `cap` attempts and resumed for as many, bit for bit the
    solve of 2 cap attempts (Dormand--Prince only where a resumed first stage
    is the one that was carried)."""
    n = 70
    if model == 0:
        P, y0, sh, t_phase = *I.quad_linspace(n), None, 0.05
    elif model == 2:
        P, y0 = I.km_grid(7, 10)
        sh, t_phase = list(I.KM_WATER), 0.02
    else:
        P, y0 = I.prv_linspace(n)
        sh, t_phase = list(I.PRV_DEFAULT), 1.0
    o = O.Opts(n_phases=10**6, n_record=0, t_phase=t_phase)
    one = gpu_ck(model, P, y0, o, shared=sh, solver=_solver(scheme), max_steps=2 * cap)
    two = gpu_ck(model, P, y0, o, shared=sh, solver=_solver(scheme), max_steps=cap, solves=2)
    go = (one.status & O.SYS_SETTLED) == 0
    assert go.any()
    for k in ("y", "t", "h"):
        assert np.array_equal(getattr(one, k)[..., go], getattr(two, k)[..., go])
    total = two.stats[O.ST_ACCEPTED] + two.stats[O.ST_REJECTED] + two.stats[O.ST_EVRETRY]
    assert np.all(total[go] == cap)


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("model,tangent", [(0, 0), (0, 1), (1, 0), (1, 3), (2, 0), (2, 2), (3, 0)])
def test_non_finite_component_stops_the_system(model, tangent, scheme):
    """NaN or an infinity in one component of the state (or of a tangent):
    the first attempt finds it, the state stays as given, the neighbour in the
    wave is not touched."""
    D = {0: 1, 1: 3, 2: 2, 3: 3}[model]
    base = {0: [-0.5], 1: [10.0] * 3, 2: [1.0, 0.0], 3: [0.2, 0.0, 10.2]}[model]
    base = base + [0.5] * (D * tangent)
    rows = [(c, v) for c in range(len(base)) for v in (np.nan, np.inf, -np.inf)]
    n = 2 * len(rows)
    y0 = np.tile(np.array(base)[:, None], (1, n))
    for k, (c, v) in enumerate(rows):
        y0[c, 2 * k] = v
    p = {0: [0.3], 1: [5.0], 2: [0.5e5, 2e5], 3: [5.0]}[model]
    P = np.tile(np.array(p)[:, None], (1, n))
    o = O.Opts(n_phases=2, n_record=2, rtol=1e-8, atol=1e-8)
    g = gpu_ck(model, P, y0, o, solver=_solver(scheme), tangent=tangent)
    bad, ok = slice(0, n, 2), slice(1, n, 2)
    assert np.all(g.status[bad] & O.SYS_NONFINITE)
    assert np.all(g.stats[O.ST_ACCEPTED][bad] == 0) and np.all(g.stats[O.ST_REJECTED][bad] == 0)
    assert np.array_equal(g.y[:, bad], y0[:, bad], equal_nan=True)
    assert np.all(g.h[bad] == o.dt0) and np.all(g.t[bad] == 0.0)
    assert not np.any(g.status[ok] & O.SYS_NONFINITE)
    assert np.all(np.isfinite(g.y[:, ok])) and np.all(g.stats[O.ST_PHASES][ok] == 2)
    assert np.all(g.y[:, ok] == g.y[:, 1:2])


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("model,dt,tol", [(0, 0.05, 1e-11), (2, 1e-3, 1e-9), (3, 0.01, 5e-8)])
def test_step_size_floor(model, dt, tol, scheme):
    """Every step at the floor (dt0 = dt_min = dt_max), over the error bound in
    some systems and within it in their neighbours: status, accepted, rejected,
    event-retry and evaluation counts are the oracle's, the state to the
    adaptive tolerance.  Compared are the systems whose outcome is the same
    at half and twice the bound and for a perturbed start.  (The valves are
    those that stay off their seat: below a flow of 1 or so every change of
    the start's last digits gives other impacts, in the oracle too.)"""
    n = 70
    if model == 0:
        P, y0, sh, kw = *I.quad_linspace(n), None, dict(t_phase=0.5, n_phases=3)
    elif model == 2:
        P, y0, sh, kw = *I.km_grid(7, 10), I.KM_WATER, dict(t_phase=0.1, n_phases=2)
    else:
        P, y0, sh, kw = *I.prv_linspace(n, 3.0, 10.0), I.PRV_DEFAULT, dict(n_phases=2)

    def oracle(f=1.0, eps=0.0):
        o = O.Opts(dt0=dt, dt_min=dt, dt_max=dt, rtol=f * tol, atol=f * tol, n_record=4,
                   max_steps=2000, scheme=scheme, **kw)
        return o, O.rkck45(model, P, None if sh is None else np.array(sh), y0 * (1.0 + eps), o)
    o, a = oracle()
    keep = np.ones(n, bool)
    for b in (oracle(f=0.5)[1], oracle(f=2.0)[1], oracle(eps=PERTURB)[1]):
        keep &= (b.status == a.status) & np.all(b.stats == a.stats, axis=0)
    keep &= sensitivity_mask([a.y], [b.y], 1e-9, 1e-11)
    floor = (a.status & O.SYS_DT_MIN) != 0
    assert keep.mean() >= 0.5 and (floor & keep).any() and (~floor & keep).any()
    g = gpu_ck(model, P, y0, o, shared=None if sh is None else list(sh), solver=_solver(scheme))
    assert np.array_equal(g.status[keep], a.status[keep])
    for k in (O.ST_ACCEPTED, O.ST_REJECTED, O.ST_EVRETRY, O.ST_NRHS, O.ST_PHASES):
        assert np.array_equal(g.stats[k][keep], a.stats[k][keep]), k
    assert np.all(g.stats[O.ST_REJECTED] == 0)
    assert np.all(per_system(close(g.y, a.y, CK_RTOL, CK_ATOL))[keep])
