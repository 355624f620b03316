"""Rules that choose a kernel's split or variant by the sizes of a problem: results on either
side of each line, against the oracle, against the general path or bit for bit where the
library promises it."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import synth  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402


def _gpu_plan(scans, **kw):
    """One plan of the given scans, each an independent problem."""
    pix, off, base = [], [np.zeros(1, np.int64)], 0
    for sc in scans:
        pix.append(sc.pix.astype(np.int64) + base)
        off.append(off[-1][-1] + sc.offsets[1:])
        base += sc.n_pix
    w = np.concatenate([sc.weights for sc in scans])
    psd = np.concatenate([np.stack([sc.sigma, sc.fknee, sc.alpha], 1) for sc in scans])
    prob = np.cumsum([0] + [sc.n_intervals for sc in scans])
    return Plan(torch.from_numpy(np.concatenate(pix).astype(np.int32)).cuda(),
                torch.from_numpy(w).cuda(), base, np.concatenate(off), psd, n_stokes=3,
                lam=scans[0].lam, f_samp=scans[0].f_samp, problem_intervals=prob, **kw)


def test_pt_range_of_coarse_columns_depends_on_the_problem_alone():
    """The P^T passes of the A Z build take ranges by the size of each problem: 512 samples for
    2^17 samples, 1024 for 2,166,784 (just past 2048 ranges of 1024).  Each problem of a batch
    equals its standalone plan bit for bit, and the mixed preconditioner is the FP64 plan's to
    the bar of FP32 columns (it depends on their span alone)."""
    kw = dict(n_det=4, lam=256, fknee_range=(2.0, 4.0), alpha_range=(1.0, 2.0))
    scans = [synth.raster_iqu(side=64, spp=4, interval_len=2 ** 12, seed_key=71, **kw),
             synth.raster_iqu(side=184, spp=8, interval_len=67712, seed_key=72, **kw)]
    opts = dict(coarse=True, az_fp16=False, fft_len_f64=4096, fft_len_f32=4096)
    pb = _gpu_plan(scans, precision="mixed", **opts)
    assert pb.pt_range() == 512
    off = pb.problem_pixels() * 3
    r = torch.randn(pb.n_vec, dtype=torch.float64, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(3))
    zb = pb.precond_2lvl(r)
    for b, sc in enumerate(scans):
        p1 = Plan.from_scan(sc, precision="mixed", **opts)
        z1 = p1.precond_2lvl(r[off[b]:off[b + 1]].contiguous())
        assert torch.equal(z1, zb[off[b]:off[b + 1]]), b
        p64 = Plan.from_scan(sc, precision="fp64", **opts)
        z64 = p64.precond_2lvl(r[off[b]:off[b + 1]].contiguous())
        assert float((z1 - z64).norm() / z64.norm()) < 1e-4, b  # A Z in FP32
        p1.close()
        p64.close()
    pb.close()


@pytest.mark.parametrize("lam,lens", [
    (0, [700, 1]),
    (64, [1, 2, 511, 512, 513, 2048, 2049, 300]),
    (512, [1, 512, 513, 1024, 5000]),
    (513, [1024, 1025, 4097, 40]),
    (1024, [9000, 1024, 1]),
    (1025, [4096, 4097, 20481, 7]),
    (4096, [8192, 16385, 4095]),
    (4097, [9000, 4097, 4098, 50]),
])
def test_lag_correlations_at_the_transforms_edges(lam, lens):
    """Lag correlations against direct sums in extended precision, for bands on either side of
    each transform length and intervals around the block and workgroup edges, with u and v of
    very different size.  Bar: rounding of N-point transforms, 4 eps log2(N) ||u|| ||v||."""
    off = np.concatenate([[0], np.cumsum(lens)])
    n = int(off[-1])
    pix = torch.arange(n, dtype=torch.int32, device="cuda") % 5
    psd = np.tile([1.0, 0.0, 1.0], (len(lens), 1))
    plan = Plan(pix, None, 5, off, psd, n_stokes=1, lam=lam, rcond_min=0.0)
    r = np.random.default_rng(lam)
    u = 1e-9 * (r.standard_normal(n) + np.sin(0.01 * np.arange(n)))
    v = r.standard_normal(n) + 0.05 * np.cumsum(r.standard_normal(n))
    c = plan.lag_correlations(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()).cpu().numpy()
    for j, m in enumerate(lens):
        U, V = (a[off[j]:off[j + 1]].astype(np.longdouble) for a in (u, v))
        K = min(lam, m - 1)
        ks = np.unique(np.r_[0:min(K, 8) + 1, np.linspace(0, K, 40).astype(int)])
        ex = np.array([(U * V).sum() if k == 0 else (U[:-k] * V[k:] + U[k:] * V[:-k]).sum()
                       for k in ks])
        bar = 4 * 2.2e-16 * 13 * float(np.sqrt((U * U).sum() * (V * V).sum()))
        assert np.abs(c[j, ks] - ex).max() <= bar, (lam, m)
        assert not c[j, K + 1:].any()
    plan.close()


@pytest.mark.parametrize("lam,lens", [
    (0, [4096, 4097, 100]),
    (300, [4095, 4096, 4097, 16383, 16384, 16385, 32768]),
    (1000, [14382, 14383, 14384, 28768, 28769]),  # one segment / two, two / three
    (6144, [12289, 16385, 40001, 4100]),
    (6145, [12291, 16386]),                       # direct sums
])
def test_taps_of_any_interval_length(lam, lens):
    """Taps and their derivatives of long intervals (chirp transforms) and on either side of
    their lines, against the oracle's inverse DFT.  Bar: rounding of two 8192-point transforms
    in the norm of the inverse PSD, and of its evaluation."""
    off = np.concatenate([[0], np.cumsum(lens)])
    n_t = int(off[-1])
    r = np.random.default_rng(lam)
    psd = np.stack([r.uniform(0.5, 2.0, len(lens)), r.uniform(2.0, 4.0, len(lens)),
                    r.uniform(1.0, 2.0, len(lens))], 1)
    psd[1, 1] = 0.0  # white noise
    plan = Plan(torch.arange(n_t, dtype=torch.int32, device="cuda") % 512, None, 512, off, psd,
                n_stokes=1, lam=lam, window="gauss", rcond_min=0.0, fft_len_f64=16384)
    dt = plan.tap_derivatives()
    eps = 2.2e-16
    for j, n in enumerate(lens):
        q = O.inverse_psd(n, *psd[j], 200.0)
        D = O.tap_derivatives(n, *psd[j], lam, 200.0)
        K = min(lam, n - 1)
        unit = (208 * eps * np.linalg.norm(q) + 32 * eps * np.abs(q).sum()) / n
        t = plan.interval_taps(j)
        assert t.shape == (K + 1,)
        assert np.abs(t - O.toeplitz_taps(n, *psd[j], lam, 200.0)).max() <= unit, (lam, n)
        # |dq| <= 2 q / sigma, alpha q / (2 f_knee)... and q |log(f_knee / f)| for f down to 1/n
        big = np.array([2 / psd[j, 0], psd[j, 2] / max(psd[j, 1], 0.5), np.log(200.0 * n)])
        assert (np.abs(dt[j, :, :K + 1] - D).max(1) <= 2 * unit * big).all(), (lam, n)
        assert not dt[j, :, K + 1:].any()
    plan.close()


@pytest.mark.parametrize("n_r,lam", [(4096, 900), (4096, 1536), (8192, 2048), (8192, 3072)])
def test_paired_tiles_at_their_edges(n_r, lam):
    """FP64 N^-1 and A x at the lengths whose tiles go in pairs: intervals of one tile, of an
    empty or one-sample second tile, of exactly full and of odd numbers of tiles, against the
    oracle's banded sums; a sample that is not finite stays within its own window's outputs and
    its own interval."""
    lmax = n_r - 2 * lam
    lens = [1, 2, 3, lmax - 1, lmax, lmax + 1, 2 * lmax - 1, 2 * lmax, 2 * lmax + 1, 3 * lmax + 5]
    off = np.concatenate([[0], np.cumsum(lens)])
    n, k = int(off[-1]), len(lens)
    r = np.random.default_rng(n_r + lam)
    psd = np.stack([r.uniform(0.5, 2.0, k), r.uniform(1.0, 2.0, k), r.uniform(1.0, 2.0, k)], 1)
    n_pix = 200
    pix = r.integers(0, n_pix, n).astype(np.int32)
    ang = r.uniform(0, np.pi, n)
    w = np.stack([np.cos(2 * ang), np.sin(2 * ang)], 1)
    plan = Plan(torch.from_numpy(pix).cuda(), torch.from_numpy(w).cuda(), n_pix, off, psd,
                n_stokes=3, lam=lam, rcond_min=0.0, fft_len_f64=n_r)
    assert plan.fft_lengths()[0] == n_r
    taps = [O.toeplitz_taps(m, *p, lam, 200.0) for m, p in zip(lens, psd)]
    y = r.standard_normal(n)
    ref = O.toeplitz_apply(y, off, taps)
    z = plan.apply_Ninv(torch.from_numpy(y).cuda()).cpu().numpy()
    assert np.abs(z - ref).max() <= 1e-12 * np.abs(ref).max()
    # map mode
    x = r.standard_normal(plan.n_vec)
    m = x.reshape(-1, 3)[np.searchsorted(np.unique(pix), pix)]
    za = O.toeplitz_apply(m[:, 0] + w[:, 0] * m[:, 1] + w[:, 1] * m[:, 2], off, taps)
    cid = np.searchsorted(np.unique(pix), pix)
    ax = np.stack([np.bincount(cid, za * c) for c in (np.ones(n), w[:, 0], w[:, 1])], 1).reshape(-1)
    got = plan.apply_A(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.abs(got - ax).max() <= 1e-12 * np.abs(ax).max()
    # one infinite sample in the middle of the first tile of the last interval
    bad = y.copy()
    t = int(off[-2]) + (lens[-1] + 3) // 4 // 2
    bad[t] = np.inf
    zb = plan.apply_Ninv(torch.from_numpy(bad).cuda()).cpu().numpy()
    tile = -(-lens[-1] // 4)
    clean = np.ones(n, bool)
    for a in range(int(off[-2]), n, tile):  # the tiles whose windows hold the sample
        if a - lam <= t < min(a + tile, n) + lam:
            clean[a:a + tile] = False
    assert np.array_equal(zb[:off[-2]], z[:off[-2]])
    assert not np.isfinite(zb[t])
    assert np.abs(zb - ref)[clean].max() <= 1e-12 * np.abs(ref).max()
    plan.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("side", [7, 16, 23])
def test_fused_pcg_updates_over_a_batch(side, precision):
    """The fused update, preconditioning, convergence-test and packing launches for problems of
    49 to 1058 pixels (around the vector kernels' blocks of 256) that stop at different
    iterations: the evaluation of one problem's true residual leaves the others' search
    directions (and their packed maps) alone.  Each problem equals its standalone solve bit for
    bit, iteration by iteration, and solves its system."""
    kw = dict(n_det=4, lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
    scans = [synth.raster_iqu(side=s, spp=8, interval_len=s * s * 4, seed_key=80 + s, **kw)
             for s in (side, 2 * side, side + 1 + side % 2)]
    opts = dict(precision="mixed", fft_len_f64=4096, fft_len_f32=4096)
    pb = _gpu_plan(scans, **opts)
    off = pb.problem_pixels() * 3
    d = torch.from_numpy(np.concatenate([sc.noise for sc in scans])).cuda()
    xb, ib = pb.pcg_solve(pb.rhs(d), precision=precision, tol=1e-9, max_iter=3000)
    assert len({p["iterations"] for p in ib["problems"]}) > 1
    for b, sc in enumerate(scans):
        p1 = Plan.from_scan(sc, **opts)
        rhs = p1.rhs(torch.from_numpy(sc.noise).cuda())
        x1, i1 = p1.pcg_solve(rhs, precision=precision, tol=1e-9, max_iter=3000)
        assert torch.equal(x1, xb[off[b]:off[b + 1]]), b
        assert i1["iterations"] == ib["problems"][b]["iterations"]
        assert np.array_equal(i1["history"], ib["problems"][b]["history"])
        pr = O.Problem.from_scan(sc)
        bn = rhs.cpu().numpy()
        res = np.linalg.norm(bn - pr.apply_A(x1.cpu().numpy())) / np.linalg.norm(bn)
        assert res <= 1.01e-9, (b, res)
        p1.close()
    pb.close()


def test_graphs_come_with_the_second_solve_and_go_with_the_coarse_space():
    """A small plan's first solve issues its launches, the second with the same arguments
    captures a graph that the later ones replay, other arguments and a new coarse space start
    over; every solve equals the plan without graphs bit for bit."""
    sc = synth.raster_iqu(side=23, spp=8, interval_len=1058, seed_key=90, n_det=4, lam=64,
                          fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
    pg = Plan.from_scan(sc, coarse=True, graph=True)
    pn = Plan.from_scan(sc, coarse=True, graph=False)
    b = pn.rhs(torch.from_numpy(sc.noise).cuda())

    def same(tol, max_iter, times):
        kw = dict(precond="2lvl", precision="fp64", tol=tol, max_iter=max_iter)
        xn, i_n = pn.pcg_solve(b, **kw)
        for k in range(times):
            xg, ig = pg.pcg_solve(b, **kw)
            assert torch.equal(xg, xn), (tol, max_iter, k)
            assert ig["iterations"] == i_n["iterations"]
            assert torch.equal(pg.apply_A(xg), pn.apply_A(xn))  # eager work between replays

    same(1e-9, 2000, 4)
    same(1e-6, 1999, 3)
    for p in (pg, pn):
        p.coarse_from_krylov(b, tol=1e-9, max_iter=2000, eps_tol=0.3)
    same(1e-9, 2000, 3)
    pg.close()
    pn.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("ns", [1, 3])
def test_segmented_sums_of_every_run_length(ns, dtype):
    """P^T over pixels of 1 (I) or 4 (IQU) to 1300 samples: runs that start and end at every
    lane, row of 16 lanes and 256-sample chunk, empty work ranges, pixels of several ranges.
    The sums are of small integers, so they are exact in any order."""
    r = np.random.default_rng(17)
    step = 1 if ns == 1 else 4
    hits = np.concatenate([np.arange(step, 70 * step, step), [1024, 252, 4, 256, 4, 260, 1300],
                           r.integers(1, 9, 600) * step, np.full(300, step)])
    pix = np.repeat(np.arange(hits.size), hits)
    order = r.permutation(pix.size)
    k = np.concatenate([np.arange(h) % 4 for h in hits])
    q = np.array([1.0, 0.0, -1.0, 0.0])[k]
    u = np.array([0.0, 1.0, 0.0, -1.0])[k]
    pix, w = pix[order].astype(np.int32), np.stack([q, u], 1)[order]
    n = pix.size
    plan = Plan(torch.from_numpy(pix).cuda(), torch.from_numpy(w).cuda() if ns == 3 else None,
                hits.size, np.array([0, n]), np.array([[1.0, 0.1, 1.0]]), n_stokes=ns, lam=8,
                precision="mixed")
    z = r.integers(-8, 9, n).astype(np.float64)
    got = plan.apply_PT(torch.from_numpy(z).to(dtype).cuda()).cpu().numpy().reshape(-1, ns)
    cols = [np.ones(n), w[:, 0], w[:, 1]][:ns]
    want = np.stack([np.bincount(pix, z * c, hits.size) for c in cols], 1)
    assert np.array_equal(got, want)
    plan.close()


def test_blocks_of_closed_plans_on_other_streams_and_threads():
    """Plans made, used and closed in turn on the default stream and on others, from one thread
    and from three at once: each takes over device and host blocks that the one before used a
    moment ago, and gives the same map bit for bit."""
    from concurrent.futures import ThreadPoolExecutor
    scans = [synth.raster_iqu(side=s, spp=8, interval_len=s * s * 4, seed_key=95 + s, n_det=4,
                              lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
             for s in (23, 24)]
    data = [torch.from_numpy(sc.noise).cuda() for sc in scans]
    torch.cuda.synchronize()

    def solve(k, stream):
        with torch.cuda.stream(stream):
            p = Plan.from_scan(scans[k])
            x, info = p.pcg_solve(p.rhs(data[k]), tol=1e-9, max_iter=2000)
            p.close()
            x = x.cpu()
        return x, info["history"]

    default = torch.cuda.default_stream()
    want = [solve(k, default) for k in (0, 1)]

    def check(streams):
        for i, st in enumerate(streams):
            x, h = solve(i % 2, st)
            assert torch.equal(x, want[i % 2][0]) and np.array_equal(h, want[i % 2][1]), i

    side = [torch.cuda.Stream() for _ in range(3)]
    check([default, side[0], side[1], default, side[0], default, default, side[1]])
    with ThreadPoolExecutor(3) as ex:
        list(ex.map(check, [[default, side[0], default], [side[1], default, side[1]],
                            [side[2], side[2], default]]))


def test_histories_of_a_batch_only_where_asked_for():
    """One copy fetches the residuals of a batch: each problem's history is its own, of its own
    length, and a solve without histories leaves the iterations alone."""
    scans = [synth.raster_iqu(side=s, spp=8, interval_len=s * s * 4, seed_key=80 + s, n_det=4,
                              lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
             for s in (7, 14, 9)]
    pb = _gpu_plan(scans, fft_len_f64=4096)
    b = pb.rhs(torch.from_numpy(np.concatenate([sc.noise for sc in scans])).cuda())
    x, info = pb.pcg_solve(b, tol=1e-9, max_iter=2000)
    y, bare = pb.pcg_solve(b, tol=1e-9, max_iter=2000, history=False)
    assert torch.equal(x, y)
    for k, p in enumerate(info["problems"]):
        assert p["history"].size == p["iterations"] > 0
        assert p["history"][-1] <= 1e-9 < p["history"][-2]
        assert bare["problems"][k]["iterations"] == p["iterations"]
        assert bare["problems"][k]["history"].size == 0
    pb.close()


@pytest.mark.parametrize("ns", [1, 3])
@pytest.mark.parametrize("max_cols", [1, 8, 19])
def test_dense_coarse_columns_in_groups(max_cols, ns):
    """A Z_D of a mixed plan is formed 8 columns at a time over the problems of a batch, whose
    column counts differ: E = Z^T A Z of every problem against A applied to one column of each
    problem after the other.  The bar is the rounding of A Z to 32 bits."""
    scans = [synth.raster_iqu(side=s, spp=8, interval_len=s * s * 4, seed_key=60 + s, n_det=4,
                              lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 2.0))
             for s in (23, 12, 31)]
    pix = np.concatenate([sc.pix + i * 1024 for i, sc in enumerate(scans)]).astype(np.int32)
    w = torch.from_numpy(np.concatenate([sc.weights for sc in scans])).cuda()
    off = np.cumsum([0] + [int(k) for sc in scans for k in np.diff(sc.offsets)])
    psd = np.concatenate([np.stack([sc.sigma, sc.fknee, sc.alpha], 1) for sc in scans])
    prob = np.cumsum([0] + [sc.n_intervals for sc in scans])
    p = Plan(torch.from_numpy(pix).cuda(), w if ns == 3 else None, 3 * 1024, off, psd,
             n_stokes=ns, lam=64, f_samp=scans[0].f_samp, problem_intervals=prob,
             precision="mixed", coarse=True, fft_len_f64=4096, fft_len_f32=4096)
    b = p.rhs(torch.from_numpy(np.concatenate([sc.noise for sc in scans])).cuda())
    p.coarse_from_krylov(b, tol=1e-9, max_iter=2000, eps_tol=1.5, max_cols=max_cols)
    Z, E, po = p.dense_columns(), p.coarse_matrix(), p.problem_pixels() * ns
    assert max(z.shape[0] for z in Z) == max_cols
    AZ = [torch.zeros_like(z) for z in Z]
    for k in range(max_cols):
        x = torch.zeros(p.n_vec, dtype=torch.float64, device="cuda")
        for i, z in enumerate(Z):
            if k < z.shape[0]:
                x[po[i]:po[i + 1]] = z[k]
        y = p.apply_A(x, precision="mixed")
        for i, z in enumerate(Z):
            if k < z.shape[0]:
                AZ[i][k] = y[po[i]:po[i + 1]]
    for z, az, e in zip(Z, AZ, E):
        z, az = z.cpu().numpy(), az.cpu().numpy()
        ref = 0.5 * (z @ az.T + az @ z.T)
        bar = 2.0 ** -23 * np.linalg.norm(z, axis=1)[:, None] * np.linalg.norm(az, axis=1)[None]
        assert (np.abs(e - ref) <= np.maximum(bar, bar.T)).all()
    p.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_dot_products_by_pt_ranges_in_a_batch_of_small_and_large_problems(precision):
    """p^T A p comes from P^T's ranges where a problem has at most 512 (2^18 samples) and from a
    launch of its own where it has more: a batch of 2^14, 2^18 (512 ranges), and just over 2^18
    samples equals the standalone plans bit for bit over the iterations it is given, and the
    recorded residuals are those of the solution."""
    kw = dict(n_det=4, lam=64, fknee_range=(0.5, 1.0), alpha_range=(1.0, 1.5))
    scans = [synth.raster_iqu(side=s, spp=8, interval_len=s * s * 4, seed_key=70 + s, **kw)
             for s in (16, 64, 65)]
    assert [len(sc.noise) for sc in scans] == [1 << 14, 1 << 18, 270400]
    opts = dict(precision="mixed", fft_len_f64=4096, fft_len_f32=4096)
    pb = _gpu_plan(scans, **opts)
    off = pb.problem_pixels() * 3
    d = torch.from_numpy(np.concatenate([sc.noise for sc in scans])).cuda()
    xb, ib = pb.pcg_solve(pb.rhs(d), precision=precision, tol=1e-8, max_iter=3000)
    for b, sc in enumerate(scans):
        p1 = Plan.from_scan(sc, **opts)
        rhs = p1.rhs(torch.from_numpy(sc.noise).cuda())
        x1, i1 = p1.pcg_solve(rhs, precision=precision, tol=1e-8, max_iter=3000)
        assert torch.equal(x1, xb[off[b]:off[b + 1]]), b
        assert np.array_equal(i1["history"], ib["problems"][b]["history"])
        res = float((rhs - p1.apply_A(x1)).norm() / rhs.norm())
        assert res <= 1.01e-8
        p1.close()
    pb.close()
