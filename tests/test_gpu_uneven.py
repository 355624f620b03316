"""Inputs of very uneven size: what is quiet keeps the accuracy of its own scale beside what is
loud, and what is zero stays zero."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402


@pytest.mark.parametrize("loud", [1e4, 1e10, 1e200, 1e305])
@pytest.mark.parametrize("n_r,lam", [(4096, 900), (8192, 2048)])
def test_quiet_tile_beside_a_loud_one(n_r, lam, loud):
    """FP64 N^-1 of an interval of two full tiles, which share one transform, the first loud
    outside the second's window: the second's outputs have the oracle's values to 1e-12 of their
    own largest, for quiet samples of size 1 and 1e-200 and on either side, and are exactly zero
    for a zero window."""
    lmax = n_r - 2 * lam
    n = 2 * lmax
    psd = np.array([[1.3, 1.5, 1.2]])
    plan = Plan(torch.arange(n, dtype=torch.int32, device="cuda") % 7, None, 7,
                np.array([0, n]), psd, n_stokes=1, lam=lam, rcond_min=0.0, fft_len_f64=n_r)
    taps = [O.toeplitz_taps(n, *psd[0], lam, 200.0)]
    r = np.random.default_rng(n_r)
    base = r.standard_normal(n)
    for flip in (False, True):
        gate = np.arange(n) < lmax - lam  # the samples of the first window alone
        out = np.arange(n) >= lmax        # the outputs of the second
        if flip:
            gate, out = gate[::-1], out[::-1]
        for quiet in (1.0, 1e-200, 0.0):
            y = np.where(gate, loud * base, quiet * base)
            z = plan.apply_Ninv(torch.from_numpy(y).cuda()).cpu().numpy()
            ref = O.toeplitz_apply(np.where(gate, 0.0, y), np.array([0, n]), taps)[out]
            if quiet == 0.0:
                assert not z[out].any(), flip
            else:
                assert np.abs(z[out] - ref).max() <= 1e-12 * np.abs(ref).max(), (flip, quiet)
            big = O.toeplitz_apply(np.where(gate, base, 0.0), np.array([0, n]), taps)
            far = np.abs(z[~out] / loud - big[~out])
            assert far.max() <= 1e-12 * np.abs(big).max() + quiet / loud * 1e3, (flip, quiet)
    plan.close()
