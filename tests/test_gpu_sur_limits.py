"""The surrogate's calls at the ends of their ranges: screens and forwards of
more points than one launch takes, and records without spread."""
import decimal

import numpy as np
import pytest

from paper_2011_01740_amd import inputs as I

pytestmark = pytest.mark.gpu


def _sur():
    import torch
    from paper_2011_01740_amd import sur
    assert torch.cuda.is_available()
    return sur


def _need_memory(gib):
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2**30:
        pytest.skip(f"needs {gib} GiB of free device memory")


def test_screen_of_more_points_than_a_launch_takes():
    """2^29 + 12345 points (a launch ends below 2^32 threads): every output is
    that of screens of 2^27 points at a time, and the re-solve list is the
    positions of the mask's ones."""
    import torch
    _need_memory(40)
    sur = _sur()
    n, part = 2**29 + 12345, 2**27
    g = torch.Generator("cuda").manual_seed(3)
    P = torch.rand(2, n, device="cuda", dtype=torch.float64, generator=g)
    P += 0.5
    with sur.Surrogate(max_batch=64) as s:
        s.set_params(I.mlp_init(7))
        s.set_norm(np.array([0.5, np.log(0.5)]), np.array([1.5, np.log(1.5)]),
                   np.full(64, 0.6), np.full(64, 0.3))
        pmax = s.screen(P[:, :4096].contiguous(), margin=0.0, spread=1e30, flag_margin=0.0)[2]
        margin = float(torch.median(torch.abs(pmax - np.log(2))))   # half of the points
        opts = dict(margin=margin, spread=1e30, flag_margin=0.0)
        label, resolve, pmax, idx = s.screen(P, **opts)
        for k in range(0, n, part):
            sub = P[:, k:k + part].contiguous()
            l1, r1, p1, _ = s.screen(sub, **opts)
            e = k + sub.shape[1]
            assert torch.equal(label[k:e], l1) and torch.equal(resolve[k:e], r1)
            assert torch.equal(pmax[k:e], p1)
        del sub, l1, r1, p1
        at, k = [], 0
        while k < n:
            at.append(torch.nonzero(resolve[k:k + part]).flatten() + k)
            k += part
        assert torch.equal(idx, torch.cat(at)) and 0 < len(idx) < n
    del P, label, resolve, pmax, idx, at
    torch.cuda.empty_cache()


def test_forward_of_more_points_than_a_launch_takes():
    """2^29 + 77 points: the same bits as forwards of 2^24 points at a time."""
    import torch
    _need_memory(160)
    sur = _sur()
    n, part = 2**29 + 77, 2**24
    x = torch.rand(n, 2, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    x *= 2
    x -= 1
    with sur.Surrogate(max_batch=64) as s:
        s.set_params(I.mlp_init(7))
        y = s.forward(x)
        for k in range(0, n, part):
            assert torch.equal(y[k:k + part], s.forward(x[k:k + part]))
    del x, y
    torch.cuda.empty_cache()


def _firm_logs(count, seed):
    """Values whose logarithm lies within 0.2 ulp of a double, so that every
    logarithm with an error below 0.8 ulp returns that double."""
    rng = np.random.default_rng(seed)
    out = []
    with decimal.localcontext() as ctx:
        ctx.prec = 40
        while len(out) < count:
            c = float(np.exp(rng.normal()))
            exact = decimal.Decimal(c).ln()
            v = float(exact)
            if abs(exact - decimal.Decimal(v)) <= decimal.Decimal(0.2 * np.spacing(abs(v))):
                out.append((c, v))
    return out


def _equal_points(v, n):
    """Mean and standard deviation of n equal values v: 256 partial sums of
    the points t, t + 256, ... in order, added by a tree, the deviation from
    the rounded mean likewise."""
    def total(x):
        q, rem = divmod(n, 256)
        sums = np.cumsum(np.concatenate([[0.0], np.full(q + 1, x)]))   # (adds one after another)
        red = np.where(np.arange(256) < rem, sums[q + 1], sums[q])
        k = 128
        while k:
            red[:k] += red[k:2 * k]
            k //= 2
        return red[0]
    mean = total(v) / n
    return mean, np.sqrt(total((v - mean) ** 2) / n)


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 255, 1000, 16384, 16385, 20000])
@pytest.mark.parametrize("ranks", [64, 1])
def test_fit_norm_of_equal_points(n, ranks):
    """A rank that is the same at every point has the spread that rounding of
    its sums leaves: none, and the call is refused, or about 1e-16, and it is
    fitted.  All ranks equal, or the largest one only.  Mean and refusal are
    exact; the deviation, a sum of at most 79 + 8 squares, to 1e-13."""
    import torch
    sur = _sur()
    lo, hi = np.array([0.5, -1.0]), np.array([1.5, 1.0])
    rng = np.random.default_rng(n)
    for c, v in _firm_logs(12, 5):
        rec = np.full((64, n), c)
        if ranks == 1:
            rec[1:] = c * rng.uniform(0.2, 0.9, (63, n))
        rd = torch.from_numpy(rec).cuda()
        mean, std = _equal_points(v, n)
        got = np.empty((2, 64))
        with sur.Surrogate(max_batch=64) as s:
            rc = sur._lib().sur_fit_norm(s.h, sur._dptr(lo), sur._dptr(hi),
                                         sur.ens.C.c_void_p(rd.data_ptr()), n,
                                         sur._dptr(got[0]), sur._dptr(got[1]))
        assert (rc == 0) == (std > 0.0 and n > 1), (c, std)
        if rc == 0:
            assert np.all(got[0, :ranks] == mean)
            assert np.allclose(got[1, :ranks], std, rtol=1e-13, atol=0.0)


@pytest.mark.parametrize("n", [2**32 - 255, 2**32, 2**32 + 64, 2**40])
def test_train_epochs_refuses_rows_beyond_32_bits(n):
    """Refused before anything is allocated or read (the row list here is one
    row long): more rows than a launch has threads or a pair's number bits."""
    import torch
    sur = _sur()
    from paper_2011_01740_amd import ens
    C = ens.C
    z = torch.zeros(64, device="cuda")
    rows = torch.zeros(1, dtype=torch.int64, device="cuda")
    lr = np.array([1e-3])
    with sur.Surrogate(max_batch=64) as s:
        rc = sur._lib().sur_train_epochs(s.h, C.c_void_p(z.data_ptr()), C.c_void_p(z.data_ptr()),
                                         C.c_void_p(rows.data_ptr()), n, 64, 1, sur._dptr(lr), 1,
                                         None)
    assert rc == ens.ENS_E_INVAL


def test_train_epochs_scratch_of_orders_made_one_at_a_time():
    """An epoch of 2^27 rows takes less than 48 bytes a row of the card: keys
    twice, pair numbers twice, the order (32 bytes a row) and the sort's
    copies of a key and a number (12)."""
    import threading
    import torch
    sur = _sur()
    _need_memory(16)
    n, batch = 2**27, 65536
    rows = torch.arange(n, device="cuda") % 64
    x = torch.rand(64, 2, device="cuda") * 2 - 1
    y = torch.rand(64, 64, device="cuda")
    least, done = [2**62], threading.Event()

    def watch():
        while not done.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])
            done.wait(0.002)
    with sur.Surrogate(max_batch=batch) as s:
        s.set_params(I.mlp_init(7))
        s.train_epochs(x, y, rows[:2 * batch], batch, [1e-3], 1)
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        t = threading.Thread(target=watch)
        t.start()
        try:
            losses = s.train_epochs(x, y, rows, batch, [1e-3], 1)
        finally:
            done.set()
            t.join()
    print(f"{(free - least[0]) / n:.2f} bytes a row")
    assert np.all(np.isfinite(losses))
    assert 40 * n < free - least[0] < 48 * n


@pytest.mark.parametrize("n", [1, 65, 16385])
def test_outputs_at_any_float_address(n):
    """Targets and network outputs need the alignment of a float only."""
    import torch
    sur = _sur()
    rng = np.random.default_rng(n)
    rd = torch.from_numpy(np.exp(rng.normal(size=(64, n)))).cuda()
    pd = torch.from_numpy(rng.uniform(0.5, 1.5, (2, n))).cuda()
    C = sur.ens.C
    with sur.Surrogate(max_batch=64) as s:
        s.set_norm([0.5, -1.0], [1.5, 1.0], np.zeros(64), np.ones(64))
        s.set_params(I.mlp_init(7))
        x, y = s.build_dataset(pd, rd, n)
        out = s.forward(x)
        for shift in (1, 2, 3):
            buf = torch.full((n * 64 + 4,), -7.0, device="cuda")
            at = buf.data_ptr() + 4 * shift
            sur._check(sur._lib().sur_build_dataset(s.h, C.c_void_p(pd.data_ptr()),
                                                    C.c_void_p(rd.data_ptr()), n,
                                                    C.c_void_p(x.data_ptr()), C.c_void_p(at)), s.h)
            assert torch.equal(buf[shift:shift + n * 64].reshape(n, 64), y)
            assert torch.all(buf[:shift] == -7.0) and torch.all(buf[shift + n * 64:] == -7.0)
            sur._check(sur._lib().sur_forward(s.h, C.c_void_p(x.data_ptr()), n, C.c_void_p(at),
                                              sur.ens.ENS_DEVICE), s.h)
            assert torch.equal(buf[shift:shift + n * 64].reshape(n, 64), out)
            assert torch.all(buf[:shift] == -7.0) and torch.all(buf[shift + n * 64:] == -7.0)
