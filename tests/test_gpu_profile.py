"""The launches that a profiled solve reports are those it makes."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import synth  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402


@pytest.mark.parametrize("side,coarse,vec", [
    (16, False, 1),  # 2^14 samples, block Jacobi: p^T A p comes with P^T, the p update is left
    (65, False, 2),  # 270400 samples: a dot product before the x, r update
    (16, True, 2),   # two-level: the x, r update and the p update
    (65, True, 2),   # the dot product and the x, r update in one bracket
])
def test_vector_brackets_of_an_iteration(side, coarse, vec):
    sc = synth.raster_iqu(side=side, spp=8, interval_len=side * side * 4, seed_key=70 + side,
                          n_det=4, lam=64, fknee_range=(3.0, 6.0), alpha_range=(1.0, 1.5))
    plan = Plan.from_scan(sc, coarse=coarse)
    b = plan.rhs(torch.from_numpy(sc.noise).cuda())
    plan.profile(True)
    _, info = plan.pcg_solve(b, precond="2lvl" if coarse else "bj", tol=1e-8, max_iter=2000)
    got = plan.profile_read()
    assert got["vec"][0] == vec * info["iterations"]
    assert got["ninv64"][0] >= info["iterations"]
    plan.close()
