"""What the performance of the framework is measured on.

A case is one call sequence that a program of this framework makes: a
fixed-step sweep, an adaptive sweep (a small one, a wide one with a pilot and
the longest-first queue, one with a second drive, one with a tangent), a batch
of relief valves, and the surrogate's data preparation, training, forward and
screening.  Handles are kept from pass to pass as a program that runs several
sweeps keeps them; parameters and states are handed over anew in every pass.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2011_01740_amd import ens, sur
from paper_2011_01740_amd import inputs as I

DEV = "cuda:0"
RK4_MODELS = {"lorenz": ens.ENS_LORENZ, "quad": ens.ENS_QUAD, "div": ens.ENS_DIV,
              "sin": ens.ENS_SIN}
ADAPTIVE = {"quad": ens.ENS_QUAD, "lorenz": ens.ENS_LORENZ, "km": ens.ENS_KM,
            "km_dual": ens.ENS_KM, "km6": ens.ENS_KM6}
#: attempted steps of one system in one phase, on average over the sweeps'
#: parameter ranges, and operations of one attempt: what a sweep cannot do without
ATTEMPTS = {"quad": 12, "lorenz": 70, "km": 500, "km_dual": 700, "km6": 700}
ATTEMPT_FLOPS = {"quad": 150, "lorenz": 450, "km": 700, "km_dual": 1000, "km6": 1000}
RK4_FLOPS = {"lorenz": 71, "quad": 22, "div": 30, "sin": 60}
NET_FLOPS = 2 * (256 * 256 + 256 * 256 + 64 * 256)   # of one point, forward


def listed():
    return [
        # the paper's Lorenz sweep (Sec. 4.1): the smallest fixed-step call, tensors in and out
        dict(name="lorenz_4096", kind="rk4", model="lorenz", n=4096, steps=1000, host=False),
        # its introductory example at its own N, arrays in host memory
        dict(name="quad_65536_host", kind="rk4", model="quad", n=65536, steps=1000, host=True),
        # the throughput workload: every system of the benchmark's ensemble
        dict(name="lorenz_8388608", kind="rk4", model="lorenz", n=1 << 23, steps=1000, host=False),
        # a first look at a Keller--Miksis grid: host arrays, all records read back
        dict(name="km_20x20_host", kind="sweep", model="km", rows=20, cols=20, phases=2, pilot=0,
             record=2, solver="ck", tangent=0, locate=0, tol=1e-10, host=True),
        # a dual-frequency study, Dormand--Prince, maxima located inside the steps, ragged size
        dict(name="dual_45x45_dp", kind="sweep", model="km_dual", rows=45, cols=45, phases=4,
             pilot=0, record=4, solver="dp", tangent=0, locate=1, tol=1e-9, host=False),
        # largest Lyapunov exponents of a grid
        dict(name="km_64x64_tangent", kind="sweep", model="km", rows=64, cols=64, phases=8,
             pilot=0, record=8, solver="ck", tangent=1, locate=0, tol=1e-10, host=False),
        # the response map: a pilot, the longest systems first, the last cycles recorded
        dict(name="km_512x512_pilot", kind="sweep", model="km", rows=512, cols=512, phases=64,
             pilot=16, record=32, solver="ck", tangent=0, locate=0, tol=1e-10, host=False),
        # three valve ensembles with their own budgets in one launch (Sec. 4.3)
        dict(name="valves_3", kind="valve", n=1 << 15, budget=200, record=16, solver="ck"),
        # the surrogate: normalisation and data set from a solved 512 x 512 grid
        dict(name="dataset_262144", kind="dataset", n=1 << 18),
        # its training at the batch that the screened sweep uses
        dict(name="train_65536_b4096", kind="train", n=65536, batch=4096, epochs=10),
        # predictions for a ragged handful of points
        dict(name="forward_1000", kind="forward", n=1000, host=False),
        # screening of the dense grid
        dict(name="screen_4096x4096", kind="screen", rows=4096, cols=4096, grid=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rk4", "sweep", "sweep", "sweep", "valve", "dataset", "train", "forward",
                       "screen"])
    if kind == "rk4":
        model = rng.choice(["lorenz", "lorenz", "quad", "div", "sin"])
        n = _log(rng, 64, 1 << 21)
        return dict(kind=kind, model=model, n=n, steps=_log(rng, 50, 1000),
                    host=n <= 70000 and rng.random() < 0.5)
    if kind == "sweep":
        model = rng.choice(["km", "km", "km", "km_dual", "km6", "lorenz", "quad"])
        rows, cols = _log(rng, 1, 200), _log(rng, 3, 400)
        phases = _log(rng, 1, 12)
        tangent = 1 if rng.random() < 0.2 else 0
        locate = 1 if model.startswith("km") and not tangent and rng.random() < 0.3 else 0
        pilot = max(1, phases // 4) if phases >= 4 and rows * cols > 4096 and rng.random() < 0.7 else 0
        return dict(kind=kind, model=model, rows=rows, cols=cols, phases=phases, pilot=pilot,
                    record=min(phases - pilot, _log(rng, 1, 8)),
                    solver=rng.choice(["ck", "ck", "dp"]), tangent=tangent, locate=locate,
                    tol=rng.choice([1e-10, 1e-10, 1e-8]), host=rows * cols < 2000)
    if kind == "valve":
        return dict(kind=kind, n=_log(rng, 16, 1 << 15), budget=_log(rng, 4, 150),
                    record=_log(rng, 1, 16), solver=rng.choice(["ck", "ck", "dp"]))
    if kind == "dataset":
        return dict(kind=kind, n=_log(rng, 100, 1 << 18))
    if kind == "train":
        batch = 64 * _log(rng, 1, 64)
        return dict(kind=kind, n=batch + _log(rng, 1, 60000 // 2), batch=batch,
                    epochs=_log(rng, 1, 5))
    if kind == "forward":
        n = _log(rng, 1, 1 << 18)
        return dict(kind=kind, n=n, host=n < 100000 and rng.random() < 0.4)
    return dict(kind=kind, rows=_log(rng, 8, 4096), cols=_log(rng, 8, 4096),
                grid=_log(rng, 16, 512))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 + int(seed))
    return g


def _rk4_inputs(case, seed):
    """P [1][n], y0 [D][n] on the device."""
    n, g = case["n"], _gen(seed)
    p = torch.rand((1, n), generator=g, device=DEV, dtype=torch.float64)
    if case["model"] == "lorenz":     # rho on [0, 21], IC 10 + U[-1, 1]
        d = torch.rand((3, n), generator=g, device=DEV, dtype=torch.float64)
        return 21.0 * p, 10.0 + (2.0 * d - 1.0)
    # the introductory example: p on [0.1, 1], x0 = -0.5 (and a little spread)
    d = torch.rand((1, n), generator=g, device=DEV, dtype=torch.float64)
    return 0.1 + 0.9 * p, -0.5 + 0.1 * (d - 0.5)


def _sweep_inputs(case, seed):
    """P, y0, shared as host arrays."""
    rng = np.random.default_rng(7000 + seed)
    rows, cols = case["rows"], case["cols"]
    n, model = rows * cols, case["model"]
    shared = None
    if model.startswith("km"):
        # the (p_A, f) grid of the frequency-response study, its corners moved a little
        j = rng.uniform(0.97, 1.03, 4)
        P, y0 = I.km_grid(rows, cols, pa_lo=0.2e5 * j[0], pa_hi=1.2e5 * j[1], f_lo=20e3 * j[2],
                          f_hi=1e6 * j[3])
        shared = list(I.KM_WATER)
        if model == "km_dual":
            shared[8], shared[9], shared[10] = 0.5e5, 150e3, 0.7
        if model == "km6":
            shared = shared[:7]
            P = np.vstack([P, rng.uniform(0.0, 0.5e5, n), rng.uniform(50e3, 400e3, n),
                           rng.uniform(-1.0, 1.0, n), rng.uniform(8e-6, 12e-6, n)])
    elif model == "lorenz":
        P = rng.uniform(0.0, 15.0, (1, n))
        y0 = 10.0 + rng.uniform(-1.0, 1.0, (3, n))
    else:
        P = rng.uniform(0.1, 1.0, (1, n))
        y0 = np.full((1, n), -0.5)
    if case["tangent"]:
        y0 = np.vstack([y0, np.full_like(y0, 1.0 / math.sqrt(y0.shape[0]))])
    return P, y0, shared


def _net(seed):
    return I.mlp_init(4 + seed % 5).astype(np.float32).astype(np.float64)


def _records(n, seed):
    """Cycle maxima [64][n] of a solved grid: mostly near-periodic responses
    around 1 .. 3, each with its own spread, in cycle order."""
    g = _gen(seed)
    level = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * 1.1
    spread = 10.0 ** (-4.0 + 3.5 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64))
    r = torch.randn((64, n), generator=g, device=DEV, dtype=torch.float64)
    return torch.exp(level + spread * r)


def _grid_params(rows, cols, seed):
    """(p_A, f) [2][rows * cols] on the device, inside the training box."""
    j = np.random.default_rng(9000 + seed).uniform(0.0, 0.02, 4)
    pa = torch.linspace(0.2e5 * (1 + j[0]), 1.2e5 * (1 - j[1]), rows, device=DEV,
                        dtype=torch.float64)
    f = torch.exp(torch.linspace(math.log(20e3 * (1 + j[2])), math.log(1e6 * (1 - j[3])), cols,
                                 device=DEV, dtype=torch.float64))
    return torch.stack([pa.repeat_interleave(cols), f.repeat(rows)]).contiguous()


IN_LO = np.array([0.2e5, math.log(20e3)])
IN_HI = np.array([1.2e5, math.log(1e6)])


def _norm(seed):
    r = np.random.default_rng(11000 + seed)
    return np.sort(r.uniform(0.3, 0.9, 64))[::-1].copy(), r.uniform(0.2, 0.4, 64)


def _train_set(case, seed):
    """Inputs in [-1, 1] and standardised targets, a smooth map with sharp edges."""
    g = _gen(seed)
    n = case["n"]
    x = torch.rand((n, 2), generator=g, device=DEV) * 2.0 - 1.0
    w = torch.randn((2, 64), generator=g, device=DEV) * 3.0
    y = torch.sin(x @ w) + 0.5 * torch.sign(torch.sin(4.0 * x[:, :1] + 3.0 * x[:, 1:]))
    y = (y - y.mean(0)) / y.std(0)
    return x.contiguous(), y.contiguous()


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    k = case["kind"]
    if k == "rk4":
        P, y0 = _rk4_inputs(case, seed)
        if case["host"]:
            P, y0 = P.cpu().numpy(), y0.cpu().numpy()
        e = ens.Ensemble(RK4_MODELS[case["model"]], ens.ENS_RK4, case["n"])
        return dict(case=case, e=e, P=P, y0=y0)
    if k == "sweep":
        P, y0, shared = _sweep_inputs(case, seed)
        e = ens.Ensemble(ADAPTIVE[case["model"]],
                         ens.ENS_RKDP45 if case["solver"] == "dp" else ens.ENS_RKCK45,
                         P.shape[1], tangent=case["tangent"])
        if shared is not None:
            e.set_shared(0, shared)
        if not case["host"]:
            P, y0 = torch.from_numpy(P).to(DEV), torch.from_numpy(y0).to(DEV)
        return dict(case=case, e=e, P=P, y0=y0)
    if k == "valve":
        # three ensembles, each twice as large as the one before it at a tenth of its budget
        n, K = case["n"], case["budget"]
        sizes = [(n, K), (2 * n, max(1, K // 10)), (4 * n, max(1, K // 100))]
        parts = [I.prv_random(m, seed=100 * seed + j) for j, (m, _) in enumerate(sizes)]
        off = np.concatenate([[0], np.cumsum([m for m, _ in sizes])]).astype(np.int64)
        e = ens.Ensemble(ens.ENS_PRV,
                         ens.ENS_RKDP45 if case["solver"] == "dp" else ens.ENS_RKCK45,
                         int(off[-1]), offsets=off)
        for j, (_, b) in enumerate(sizes):
            e.set_shared(j, list(I.PRV_DEFAULT))
            e.set_budget(j, b, b)
        P = torch.from_numpy(np.concatenate([p for p, _ in parts], axis=1)).to(DEV)
        y0 = torch.from_numpy(np.concatenate([y for _, y in parts], axis=1)).to(DEV)
        return dict(case=case, e=e, P=P, y0=y0)
    if k == "dataset":
        s = sur.Surrogate(max_batch=4096)
        P = _grid_params(1, case["n"], seed)
        return dict(case=case, s=s, P=P, rec=_records(case["n"], seed))
    if k == "train":
        s = sur.Surrogate(max_batch=case["batch"])
        s.set_adam(lr=3e-3)
        x, y = _train_set(case, seed)
        rows = torch.arange(case["n"], device=DEV, dtype=torch.int64)
        E = case["epochs"]
        lrs = [3e-3 * 0.5 * (1.0 + math.cos(math.pi * ep / E)) + 1e-5 for ep in range(E)]
        return dict(case=case, s=s, x=x, y=y, rows=rows, lrs=lrs, flat=_net(seed), seed=seed)
    s = sur.Surrogate(max_batch=4096)
    s.set_params(_net(seed))
    if k == "forward":
        x = torch.rand((case["n"], 2), generator=_gen(seed), device=DEV) * 2.0 - 1.0
        return dict(case=case, s=s, x=x.cpu().numpy() if case["host"] else x)
    mean, std = _norm(seed)
    s.set_norm(IN_LO, IN_HI, mean, std)
    G = case["grid"]
    s.fit_label_map(_records(G * G, seed), G)
    P = _grid_params(case["rows"], case["cols"], seed)
    n = P.shape[1]
    s.reserve(n)
    out = s.screen_outputs(n, P.device)
    out[3].fill_(-1)       # past the last index of a point to re-solve
    return dict(case=case, s=s, P=P, out=out)


# ------------------------------------------------------------------ run
def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "rk4":
        e = st["e"]
        e.set_params(st["P"])
        e.set_state(st["y0"])
        e.solve(dt=0.01, n_steps=case["steps"])
        d = not case["host"]
        return {"y": e.read(ens.ENS_STATE, device=d), "acc": e.read(ens.ENS_ACC, device=d)}
    if k == "sweep":
        e = st["e"]
        e.set_params(st["P"])
        e.set_state(st["y0"])
        o = dict(n_record=case["record"], rtol=case["tol"], atol=case["tol"],
                 locate_max=case["locate"])
        rest = case["phases"] - case["pilot"]
        if case["pilot"]:
            # the rest on one wave per SIMD, the longest systems first
            e.solve(n_phases=case["pilot"], **o)
            e.order_by_work()
            e.solve(n_phases=rest, grid=256, **o)
        else:
            e.solve(n_phases=rest, **o)
        return _read(e, not case["host"])
    if k == "valve":
        e = st["e"]
        e.set_params(st["P"])
        e.set_state(st["y0"])
        e.solve(n_phases=case["budget"], n_record=case["record"], use_graph=1, spread=case["n"])
        return _read(e, True)
    s = st["s"]
    if k == "dataset":
        n = case["n"]
        mean, std = np.empty(64), np.empty(64)
        sur._check(sur._lib().sur_fit_norm(s.h, sur._dptr(IN_LO), sur._dptr(IN_HI),
                                           ctypes.c_void_p(st["rec"].data_ptr()), n,
                                           sur._dptr(mean), sur._dptr(std)), s.h)
        x, y = s.build_dataset(st["P"], st["rec"], n)
        return {"mean": mean, "std": std, "x": x, "y": y}
    if k == "train":
        s.set_params(st["flat"])
        losses = s.train_epochs(st["x"], st["y"], st["rows"], case["batch"], st["lrs"],
                                st["seed"])
        # the master weights are float32; get_params hands them out as doubles
        return {"losses": losses, "params": s.get_params().astype(np.float32)}
    if k == "forward":
        return {"out": s.forward(st["x"])}
    label, resolve, pmax, idx = s.screen(st["P"], 0.02, 1e30, 0.0, label_margin=0.15,
                                         out=st["out"])
    return {"label": label, "resolve": resolve, "pmax": pmax, "idx": st["out"][3],
            "count": int(idx.numel())}


def _read(e, device):
    f = {"y": ens.ENS_STATE, "t": ens.ENS_TIME, "h": ens.ENS_H, "records": ens.ENS_RECORDS,
         "stats": ens.ENS_STATS, "status": ens.ENS_STATUS}
    return {k: e.read(v, device=device) for k, v in f.items()}


# ------------------------------------------------------------------ work
def work(case):
    k = case["kind"]
    if k == "rk4":
        D = 3 if case["model"] == "lorenz" else 1
        return {"bytes": 8.0 * case["n"] * (1 + 2 * D + 1),
                "flops": float(case["n"]) * case["steps"] * RK4_FLOPS[case["model"]]}
    if k == "sweep":
        m, n = case["model"], case["rows"] * case["cols"]
        D, P = ens.MODEL_DIMS[ADAPTIVE[m]][:2]
        T = case["tangent"]
        b = 8.0 * n * (P + 2 * D * (1 + T) + 2 + 6 + case["record"] * (1 + T)) + 4.0 * n
        return {"bytes": b, "flops": float(n) * case["phases"] * ATTEMPTS[m] * ATTEMPT_FLOPS[m]
                * (1.5 if T else 1.0)}
    if k == "valve":
        n, K = case["n"], case["budget"]
        ph = n * K + 2 * n * max(1, K // 10) + 4 * n * max(1, K // 100)
        return {"bytes": 8.0 * 7 * n * (1 + 6 + 2 + 6 + 2 * case["record"]) + 4.0 * 7 * n,
                "flops": 270.0 * 450.0 * ph}
    if k == "dataset":
        return {"bytes": case["n"] * (64 * 8.0 + 16 + 8 + 64 * 4), "flops": case["n"] * 64.0 * 60}
    if k == "train":
        steps = case["epochs"] * (case["n"] // case["batch"])
        # forward, data gradients back to layer 2, weight gradients
        per_row = NET_FLOPS + 2.0 * (64 * 256 + 256 * 256) + NET_FLOPS
        return {"bytes": steps * (case["batch"] * 66 * 4.0 + 6 * 4.0 * sur.N_PARAMS),
                "flops": steps * case["batch"] * per_row}
    if k == "forward":
        return {"bytes": case["n"] * 66 * 4.0 + 2.0 * sur.N_PARAMS, "flops": float(case["n"]) * NET_FLOPS}
    n = case["rows"] * case["cols"]
    return {"bytes": n * (16.0 + 6.0) + 2.0 * sur.N_PARAMS, "flops": float(n) * NET_FLOPS}


# ------------------------------------------------------------------ exact
def exact(case, seed):
    k = case["kind"]
    if k == "rk4":
        if case["n"] * case["steps"] > (1 << 21) * 200 or case["model"] == "lorenz" and case["steps"] > 1000:
            return None
        return _rk4_exact(case, seed)
    if k == "sweep":
        if case["model"] not in ("km", "quad", "lorenz") or case["tangent"] or case["locate"] or \
                case["solver"] != "ck" or case["pilot"] or case["rows"] * case["cols"] > 1000 or \
                case["phases"] > 2:
            return None
        return _cash_karp_exact(case, seed)
    if k == "dataset":
        rec, P = _records(case["n"], seed), _grid_params(1, case["n"], seed)
        ln = torch.log(torch.sort(rec, dim=0, descending=True).values)
        mean = ln.mean(1)
        std = torch.sqrt(((ln - mean[:, None]) ** 2).mean(1))
        x = torch.stack([P[0], torch.log(P[1])], 1)
        lo = torch.from_numpy(IN_LO).to(DEV)
        hi = torch.from_numpy(IN_HI).to(DEV)
        return {"mean": mean.cpu().numpy(), "std": std.cpu().numpy(),
                "x": (x - lo) * (2.0 / (hi - lo)) - 1.0, "y": ((ln - mean[:, None]) / std[:, None]).T}
    if k == "train":
        return _train_exact(case, seed)
    if k == "forward":
        x = torch.rand((case["n"], 2), generator=_gen(seed), device=DEV) * 2.0 - 1.0
        return {"out": _net_exact(_layers(_net(seed)), x.double())[-1]}
    if k == "screen":
        P = _grid_params(case["rows"], case["cols"], seed)
        mean, std = (torch.from_numpy(v).to(DEV) for v in _norm(seed))
        Ws = _layers(_net(seed))
        pmax = []
        for c in range(0, P.shape[1], 1 << 19):
            p, f = P[0, c:c + (1 << 19)], torch.log(P[1, c:c + (1 << 19)])
            x = torch.stack([(p - IN_LO[0]) * (2.0 / (IN_HI[0] - IN_LO[0])) - 1.0,
                             (f - IN_LO[1]) * (2.0 / (IN_HI[1] - IN_LO[1])) - 1.0], 1)
            pmax.append((_net_exact(Ws, x)[-1] * std + mean).max(1).values)
        return {"label": None, "resolve": None, "pmax": torch.cat(pmax), "idx": None,
                "count": None}
    return None


def _rk4_exact(case, seed):
    P, y = _rk4_inputs(case, seed)
    p, dt, model = P[0], 0.01, case["model"]

    def f(y):
        if model == "lorenz":
            return torch.stack([10.0 * (y[1] - y[0]), y[0] * (p - y[2]) - y[1],
                                y[0] * y[1] - (8.0 / 3.0) * y[2]])
        x = y[0]
        return {"quad": lambda: x * x - p, "div": lambda: 1.0 / x - p * x,
                "sin": lambda: p * torch.sin(x)}[model]()[None]

    m = y[0].clone()
    for _ in range(case["steps"]):
        k1 = f(y)
        k2 = f(y + 0.5 * dt * k1)
        k3 = f(y + 0.5 * dt * k2)
        k4 = f(y + dt * k3)
        y = y + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
        m = torch.maximum(m, y[0])
    return {"y": y, "acc": m}


CK_A = [[], [1 / 5], [3 / 40, 9 / 40], [3 / 10, -9 / 10, 6 / 5], [-11 / 54, 5 / 2, -70 / 27, 35 / 27],
        [1631 / 55296, 175 / 512, 575 / 13824, 44275 / 110592, 253 / 4096]]
CK_C = [0.0, 1 / 5, 3 / 10, 3 / 5, 1.0, 7 / 8]
CK_B5 = [37 / 378, 0.0, 250 / 621, 125 / 594, 0.0, 512 / 1771]
CK_B4 = [2825 / 27648, 0.0, 18575 / 48384, 13525 / 55296, 277 / 14336, 1 / 4]


def _km_rhs(P, sh):
    """Sec. 4.2 of the paper, one drive."""
    rho, cl, pv, sig, mu, gam, pinf, re = sh[:8]
    pa, w = P[0], 2.0 * np.pi * P[1]
    q2 = (2.0 * np.pi / (re * w)) ** 2
    c0 = (pinf - pv + 2.0 * sig / re) * q2 / rho
    c1 = (1.0 - 3.0 * gam) / (rho * cl) * (pinf - pv + 2.0 * sig / re) * 2.0 * np.pi / (re * w)
    c2 = (pinf - pv) * q2 / rho
    c3, c4 = 2.0 * sig / (rho * re) * q2, 4.0 * mu / (rho * re * re) * 2.0 * np.pi / w
    c5, c7 = pa * q2 / rho, re * w * pa / (rho * cl) * q2
    c9 = re * w / (2.0 * np.pi * cl)

    def f(t, y):
        a, b = y
        s, c = np.sin(2.0 * np.pi * t), np.cos(2.0 * np.pi * t)
        num = (c0 + c1 * b) * a ** (-3.0 * gam) - c2 * (1.0 + c9 * b) - c3 / a - c4 * b / a \
            - (1.0 - c9 * b / 3.0) * 1.5 * b * b - c5 * s * (1.0 + c9 * b) - c7 * c * a
        return np.stack([b, num / (a - c9 * a * b + c4 * c9)])

    return f


def _cash_karp_exact(case, seed):
    """Every system on its own step size, as the adaptive solver documents it, in numpy."""
    P, y, shared = _sweep_inputs(case, seed)
    n, model, tol, R = P.shape[1], case["model"], case["tol"], case["record"]
    if model == "km":
        f = _km_rhs(P, shared)
    elif model == "quad":
        f = lambda t, y: y * y - P  # noqa: E731
    else:
        f = lambda t, y: np.stack([10.0 * (y[1] - y[0]), y[0] * (P[0] - y[2]) - y[1],  # noqa: E731
                                   y[0] * y[1] - (8.0 / 3.0) * y[2]])
    y = y.copy()
    t, h, ymax = np.zeros(n), np.full(n, 1e-2), np.full(n, -np.inf)
    phase = np.zeros(n, dtype=np.int64)
    rec = np.full((R, 1, n), np.nan)
    with np.errstate(all="ignore"):
        while (phase < case["phases"]).any():
            live = phase < case["phases"]
            trunc = t + h >= 1.0
            ht = np.where(trunc, 1.0 - t, h)
            ks = []
            for s in range(6):
                ys = y + ht * sum((a * kk for a, kk in zip(CK_A[s], ks)), np.zeros_like(y))
                ks.append(f(t + CK_C[s] * ht, ys))
            y5 = y + ht * sum(b * kk for b, kk in zip(CK_B5, ks))
            err = ht * sum((b - d) * kk for b, d, kk in zip(CK_B5, CK_B4, ks))
            E = (np.abs(err) / (tol + tol * np.maximum(np.abs(y), np.abs(y5)))).max(0)
            acc = (E <= 1.0) | (ht <= 1e-14)
            fac = np.where(E > 0, 0.9 * np.maximum(E, 1e-300) ** -0.2, 5.0)
            hn = np.clip(ht * np.clip(fac, 0.2, np.where(acc, 5.0, 1.0)), 1e-14, 0.1)
            go = live & acc
            y = np.where(go, y5, y)
            ymax = np.where(go, np.maximum(ymax, y[0]), ymax)
            end = go & trunc
            i = np.nonzero(end)[0]
            rec[phase[i] % R, 0, i] = ymax[i]
            phase[i] += 1
            ymax[i] = -np.inf
            t = np.where(end, 0.0, np.where(go, t + ht, t))
            h = np.where(live & ~end, hn, h)
    return {"y": y, "t": t, "h": h, "records": rec, "stats": None, "status": None}


def _layers(flat):
    p, at, Ws = torch.from_numpy(flat).to(DEV), 0, []
    for o, i in ((256, 2), (256, 256), (256, 256), (64, 256)):
        Ws.append(p[at:at + o * i].reshape(o, i).clone())
        Ws.append(p[at + o * i:at + o * i + o].clone())
        at += o * i + o
    return Ws


def _net_exact(W, x):
    a1 = torch.sin(x @ W[0].T + W[1])
    z2 = a1 @ W[2].T + W[3]
    a2 = torch.nn.functional.gelu(z2)
    z3 = a2 @ W[4].T + W[5]
    a3 = torch.nn.functional.gelu(z3)
    return a1, z2, a2, z3, a3, a3 @ W[6].T + W[7]


def _gelu_grad(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _splitmix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _train_exact(case, seed):
    x, y = (v.double() for v in _train_set(case, seed))
    W = _layers(_net(seed))
    n, B, E = case["n"], case["batch"], case["epochs"]
    wt = torch.ones(64, device=DEV, dtype=torch.float64)
    wt[0] = 32.0
    wt *= 64.0 / wt.sum()
    m, v, t, losses = [0.0] * 8, [0.0] * 8, 0, []
    for ep in range(E):
        lr = 3e-3 * 0.5 * (1.0 + math.cos(math.pi * ep / E)) + 1e-5
        with np.errstate(over="ignore"):
            key = _splitmix(np.uint64(seed) + np.uint64(0x9E3779B97F4A7C15)
                            * (np.arange(n, dtype=np.uint64) + np.uint64(ep * n + 1)))
        order = torch.from_numpy(np.argsort(key, kind="stable")).to(DEV)
        total = 0.0
        for b in range(n // B):
            r = order[b * B:(b + 1) * B]
            a1, z2, a2, z3, a3, out = _net_exact(W, x[r])
            d = out - y[r]
            total += float((wt * d * d).mean())
            g4 = 2.0 * wt * d / (B * 64)
            g3 = (g4 @ W[6]) * _gelu_grad(z3)
            g2 = (g3 @ W[4]) * _gelu_grad(z2)
            grads = [None, None, g2.T @ a1, g2.sum(0), g3.T @ a2, g3.sum(0), g4.T @ a3, g4.sum(0)]
            t += 1
            for j in range(2, 8):
                m[j] = 0.9 * m[j] + 0.1 * grads[j]
                v[j] = 0.999 * v[j] + 0.001 * grads[j] ** 2
                W[j] = W[j] - lr * (m[j] / (1 - 0.9 ** t)) / (torch.sqrt(v[j] / (1 - 0.999 ** t)) + 1e-8)
        losses.append(total / (n // B))
    return {"losses": np.array(losses), "params": torch.cat([w.reshape(-1) for w in W]).cpu().numpy()}
