"""The surrogate's calls at the ends of their ranges: screens and forwards of
more points than one launch takes."""
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
