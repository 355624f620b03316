"""What a plan holds after its calls: captured graphs, and the work ranges its coarse space was
built with."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import synth  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402

KW = dict(n_det=4, lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))


def test_a_graph_comes_with_the_second_solve_and_goes_with_its_arguments():
    sc = synth.raster_iqu(side=23, spp=8, interval_len=1058, seed_key=90, **KW)
    plan = Plan.from_scan(sc, coarse=True)
    b = plan.rhs(torch.from_numpy(sc.noise).cuda())

    def counts(n, **kw):
        out = []
        for _ in range(n):
            plan.pcg_solve(b, tol=1e-9, **kw)
            out.append(plan.graph_count())
        return out

    assert counts(3, precond="2lvl", max_iter=2000) == [0, 1, 1]
    assert counts(3, precond="2lvl", max_iter=1999) == [0, 1, 1]
    assert counts(2, precond="adef2", max_iter=1999) == [1, 2]
    assert counts(2, precond="bj", max_iter=1999) == [2, 2]  # block Jacobi has none
    plan.coarse_from_krylov(b, tol=1e-9, max_iter=2000, eps_tol=0.3)
    assert plan.graph_count() == 0
    assert counts(2, precond="2lvl", max_iter=1999) == [0, 1]
    plan.close()
    off = Plan.from_scan(sc, coarse=True, graph=False)
    for _ in range(2):
        off.pcg_solve(b, precond="2lvl", tol=1e-9, max_iter=2000)
    assert off.graph_count() == 0
    off.close()


def test_no_graph_from_2_18_samples():
    sc = synth.raster_iqu(side=64, spp=8, interval_len=1 << 14, seed_key=91, **KW)
    plan = Plan.from_scan(sc, coarse=True)
    assert plan.n_samples == 1 << 18
    b = plan.rhs(torch.from_numpy(sc.noise).cuda())
    for _ in range(3):
        plan.pcg_solve(b, precond="2lvl", tol=1e-9, max_iter=2000)
    assert plan.graph_count() == 0
    plan.close()


def test_ranges_of_the_coarse_build():
    """4096 samples, halved to no less than 512 until the problem makes 2048 ranges: 2^17
    samples, just past 2048 ranges of 1024, in one batch and alone."""
    scans = [synth.raster_iqu(side=64, spp=4, interval_len=2 ** 12, seed_key=71, **KW),
             synth.raster_iqu(side=184, spp=8, interval_len=67712, seed_key=72, **KW)]
    pix, off, base = [], [np.zeros(1, np.int64)], 0
    for sc in scans:
        pix.append(sc.pix.astype(np.int64) + base)
        off.append(off[-1][-1] + sc.offsets[1:])
        base += sc.n_pix
    psd = np.concatenate([np.stack([sc.sigma, sc.fknee, sc.alpha], 1) for sc in scans])
    plan = Plan(torch.from_numpy(np.concatenate(pix).astype(np.int32)).cuda(),
                torch.from_numpy(np.concatenate([sc.weights for sc in scans])).cuda(), base,
                np.concatenate(off), psd, n_stokes=3, lam=64, f_samp=scans[0].f_samp,
                problem_intervals=np.cumsum([0] + [sc.n_intervals for sc in scans]), coarse=True)
    assert plan.az_pt_ranges().tolist() == [512, 1024]
    assert plan.pt_range() == 512
    plan.close()
    for sc, r in zip(scans, (512, 1024)):
        one = Plan.from_scan(sc, coarse=True)
        assert one.az_pt_ranges().tolist() == [r]
        one.close()
    none = Plan.from_scan(scans[0])
    assert none.az_pt_ranges().size == 0
    none.close()


def test_histories_of_more_problems_than_one_copy_takes():
    """700 problems of 64 samples, 1600 iterations each towards a tolerance out of reach: the
    histories come in several copies, and each is its own problem's."""
    B, n, it = 700, 64, 1600
    r = np.random.default_rng(4)
    pix = np.concatenate([b * 8 + r.permutation(np.arange(n) % 8) for b in range(B)])
    off = np.arange(B * 2 + 1) * (n // 2)
    psd = np.stack([r.uniform(0.5, 2, 2 * B), r.uniform(1, 2, 2 * B), np.ones(2 * B)], 1)
    d = torch.from_numpy(r.standard_normal(B * n)).cuda()
    kw = dict(n_stokes=1, lam=8, fft_len_f64=2048)
    plan = Plan(torch.from_numpy(pix.astype(np.int32)).cuda(), None, 8 * B, off, psd,
                problem_intervals=np.arange(B + 1) * 2, **kw)
    _, info = plan.pcg_solve(plan.rhs(d), tol=1e-300, max_iter=it, raise_on_error=False)
    per = info["problems"]
    assert max(p["iterations"] for p in per) * B > 1 << 20
    for b in (0, 1, 348, 654, 655, 656, 699):
        one = Plan(torch.from_numpy((pix[b * n:(b + 1) * n] - 8 * b).astype(np.int32)).cuda(), None,
                   8, np.array([0, n // 2, n]), psd[2 * b:2 * b + 2], **kw)
        _, i1 = one.pcg_solve(one.rhs(d[b * n:(b + 1) * n].contiguous()), tol=1e-300, max_iter=it,
                              raise_on_error=False)
        assert per[b]["iterations"] == i1["iterations"]
        assert np.array_equal(per[b]["history"], i1["history"]), b
        one.close()
    plan.close()
