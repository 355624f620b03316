"""Solves and the caller's stream: a solve overlaps with what other threads do there."""

import threading
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import synth  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402
from paper_1408_3048_amd._lib import MMError  # noqa: E402


def ends_before_later_work(plan, b, **kw):
    """While a thread solves on the default stream, another enqueues 2 s of work there: the
    solve, about half a second of iterations to a tolerance that it cannot meet, reads its
    states on a stream of its own and ends first."""
    def solve(max_iter):
        t = time.perf_counter()
        try:
            plan.pcg_solve(b, max_iter=max_iter, **kw)
        except MMError:
            pass
        return time.perf_counter() - t

    solve(200)
    per_iter = min(solve(400) for _ in range(3)) / 400
    max_iter = max(400, int(0.3 / per_iter))
    # a pause of the stream, without work for the CUs: cycles per second of the device's clock
    e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    e0.record()
    torch.cuda._sleep(10_000_000)
    e1.record()
    torch.cuda.synchronize()
    cycles = int(1e7 / e0.elapsed_time(e1) * 100)  # 0.1 s
    done = {}

    def worker():
        with torch.cuda.stream(torch.cuda.default_stream()):
            done["s"] = solve(max_iter)
            done["at"] = time.perf_counter()

    th = threading.Thread(target=worker)
    th.start()
    time.sleep(0.1)  # the solve is among its iterations
    for _ in range(20):
        torch.cuda._sleep(cycles)
    torch.cuda.synchronize()
    end = time.perf_counter()
    th.join()
    assert done["at"] < end - 0.5, (done["s"], per_iter, max_iter)


@pytest.mark.parametrize("history", [False, True])
@pytest.mark.parametrize("coarse", [False, True])
def test_solve_does_not_wait_for_later_work_on_the_callers_stream(coarse, history):
    sc = synth.raster_iqu(side=16, spp=8, interval_len=512, seed_key=12, n_det=4, lam=64,
                          fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
    plan = Plan.from_scan(sc, coarse=coarse)
    ends_before_later_work(plan, plan.rhs(torch.from_numpy(sc.noise).cuda()),
                           precond="2lvl" if coarse else "bj", tol=1e-30, history=history)
    plan.close()


def test_histories_of_a_batch_do_not_wait_for_it():
    r = np.random.default_rng(7)
    n, n_pix, B = 4096, 64, 3
    pix = np.concatenate([b * n_pix + r.permutation(np.arange(n) % n_pix) for b in range(B)])
    off = np.arange(B * 4 + 1) * (n // 4)
    psd = np.stack([r.uniform(0.5, 2, 4 * B), r.uniform(1, 2, 4 * B), np.ones(4 * B)], 1)
    plan = Plan(torch.from_numpy(pix.astype(np.int32)).cuda(), None, n_pix * B, off, psd,
                problem_intervals=np.arange(B + 1) * 4, n_stokes=1, lam=64)
    ends_before_later_work(plan, plan.rhs(torch.from_numpy(r.standard_normal(B * n)).cuda()),
                           precond="bj", tol=1e-30, history=True)
    plan.close()
