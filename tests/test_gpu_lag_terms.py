"""Lag correlations keep, lag by lag, the rounding of that lag's own terms."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1408_3048_amd import Plan  # noqa: E402

EPS = 2.2e-16


def _plan(lens, lam):
    off = np.concatenate([[0], np.cumsum(lens)])
    n = int(off[-1])
    return off, Plan(torch.arange(n, dtype=torch.int32, device="cuda") % 5, None, 5, off,
                     np.tile([1.0, 0.0, 1.0], (len(lens), 1)), n_stokes=1, lam=lam, rcond_min=0.0)


def _exact(u, v, k):
    """c(k) and the sum of its terms' magnitudes, in extended precision."""
    u, v = u.astype(np.longdouble), v.astype(np.longdouble)
    t = u * v if k == 0 else np.concatenate([u[:-k] * v[k:], u[k:] * v[:-k]])
    return t.sum(), np.abs(t).sum()


def _check(u, v, off, lam, c, step=1):
    for j, (a, b) in enumerate(zip(off[:-1], off[1:])):
        K = min(lam, int(b - a) - 1)
        for k in np.unique(np.r_[0:K + 1:step, K]):
            ex, s = _exact(u[a:b], v[a:b], int(k))
            # a chain of 2 x 1024 additions per partial sum, which bounds the transforms' part
            # (4 eps log2(8192) of norms of at most 8 s) as well
            assert abs(c[j, k] - ex) <= 2100 * EPS * s, (j, k, float(c[j, k]), float(ex), float(s))
        assert not c[j, K + 1:].any()


@pytest.mark.parametrize("lam,n,step", [(300, 5000, 7), (1000, 9000, 23), (2048, 30000, 61),
                                        (4095, 20000, 101), (4096, 9000, 101), (5000, 9000, 103)])
def test_bursts_far_apart(lam, n, step):
    """u and v of which one is nonzero in a short burst, the other in two: most lags have no terms
    and are exactly zero, the others few, beside a loud stretch that meets nothing."""
    off, plan = _plan([n, n], lam)
    r = np.random.default_rng(lam)
    u, v = np.zeros(2 * n), np.zeros(2 * n)
    for j in (0, 1):
        b = off[j] + 100
        u[b:b + 20] = r.standard_normal(20)
        v[b + lam // 2:b + lam // 2 + 5] = 1e-3 * r.standard_normal(5)
        v[b + lam - 10:b + lam + 9] = 1e-9 * r.standard_normal(19)
        v[off[j + 1] - 700:off[j + 1] - 600] = 1e6 * r.standard_normal(100)
    u[off[1]:] *= 1e-200
    c = plan.lag_correlations(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()).cpu().numpy()
    _check(u, v, off, lam, c, step)
    plan.close()


@pytest.mark.parametrize("lam,lens", [(600, [601, 700, 300]), (2048, [2100, 2048, 40, 3000]),
                                      (4096, [4100, 5000, 1025])])
def test_lags_of_few_terms(lam, lens):
    """Dense u and v on intervals little longer than the band, or shorter: the last lags have few
    terms."""
    off, plan = _plan(lens, lam)
    r = np.random.default_rng(lam)
    u, v = r.standard_normal(int(off[-1])), 1e5 * r.standard_normal(int(off[-1]))
    c = plan.lag_correlations(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()).cpu().numpy()
    _check(u, v, off, lam, c, 13)
    plan.close()


def test_zero_and_infinite_samples():
    """A zero u gives exact zeros beside any v; an infinite sample reaches the lags it has terms
    in, and no others."""
    lam, n = 700, 3000
    off, plan = _plan([n, n], lam)
    r = np.random.default_rng(5)
    u, v = r.standard_normal(2 * n), r.standard_normal(2 * n)
    u[:n] = 0.0
    u[n + 50:n + 200] = 0.0
    u[n + 300:] = 0.0
    v[n:n + 900] = 0.0
    v[n + 950] = np.inf  # meets u's samples n .. n + 50 and n + 200 .. n + 300 alone
    c = plan.lag_correlations(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()).cpu().numpy()
    assert not c[0].any()
    a, b = u[n:], v[n:]
    with np.errstate(invalid="ignore"):
        ref = np.array([(a * b).sum() if k == 0 else (a[:-k] * b[k:]).sum() + (a[k:] * b[:-k]).sum()
                        for k in range(lam + 1)])
    assert np.array_equal(np.isfinite(c[1]), np.isfinite(ref))
    plan.close()


def test_more_intervals_than_one_launch_takes():
    """20000 short intervals, whose transforms take several turns through the scratch."""
    r = np.random.default_rng(11)
    lens = r.integers(2, 40, 20000)
    lam = 600
    off, plan = _plan(lens, lam)
    n = int(off[-1])
    u, v = r.standard_normal(n), r.standard_normal(n)
    c = plan.lag_correlations(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()).cpu().numpy()
    own = np.repeat(np.arange(lens.size), lens)
    for k in range(40):
        t = u * v if k == 0 else u[:n - k] * v[k:] + u[k:] * v[:n - k]
        m = np.abs(u * v) if k == 0 else np.abs(u[:n - k] * v[k:]) + np.abs(u[k:] * v[:n - k])
        same = own[:n - k] == own[k:]
        ex = np.bincount(own[:n - k][same], t[same], lens.size)
        s = np.bincount(own[:n - k][same], m[same], lens.size)
        assert (np.abs(c[:, k] - ex) <= 2100 * EPS * s).all(), k
    assert not c[:, 40:].any()
    plan.close()
