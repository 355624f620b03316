"""Plans of very many interval lengths, or of very long intervals: the taps are formed in turns
through a bounded scratch."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from paper_1408_3048_amd import Plan  # noqa: E402


def _taps(lens, lam, check):
    off = np.concatenate([[0], np.cumsum(lens)])
    r = np.random.default_rng(lam)
    psd = np.stack([r.uniform(0.5, 2.0, len(lens)), r.uniform(2.0, 4.0, len(lens)),
                    r.uniform(1.0, 2.0, len(lens))], 1)
    psd[::3] = psd[0]
    pix = torch.arange(int(off[-1]), dtype=torch.int32, device="cuda") % 512
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    plan = Plan(pix, None, 512, off, psd, n_stokes=1, lam=lam, rcond_min=0.0)
    grown = free0 - torch.cuda.mem_get_info()[0]
    for j in check:
        n, q = int(lens[j]), O.inverse_psd(int(lens[j]), *psd[j], 200.0)
        # rounding of two 8192-point transforms in the norm of the inverse PSD (per segment; their
        # sum's grows less than the norm), and of its evaluation
        unit = (208 * 2.2e-16 * np.linalg.norm(q) + 32 * 2.2e-16 * np.abs(q).sum()) / n
        t = plan.interval_taps(int(j))
        assert np.abs(t - O.toeplitz_taps(n, *psd[j], lam, 200.0)).max() <= unit, n
    plan.close()
    return grown


@pytest.mark.parametrize("lam,most", [(100, 1.45e9), (1500, 1.65e9)])
def test_taps_of_more_lengths_than_one_launch_holds(lam, most):
    """4500 lengths from 4097 to 8596 samples (600 MB of chirps), some twice with one PSD and some
    with two, in any order.  Memory: 28.5e6 samples at 40 bytes, the scratch and the spectra (the
    chirps at once, and both halves of the spectra at lambda = 1500, took 1.67 and 2.15 GB)."""
    r = np.random.default_rng(3)
    lens = 4097 + r.permutation(4500)
    lens[100:400] = lens[:300]
    assert _taps(lens, lam, np.r_[0:410:3, r.integers(0, 4500, 60)]) <= most


def test_taps_of_an_interval_of_many_segments():
    """2^23 + 3 samples at lambda = 6144: 2049 segments of 2048 frequencies, three a row."""
    _taps(np.array([(1 << 23) + 3, 5000]), 6144, [0, 1])


@pytest.mark.parametrize("lam", [511, 512])
def test_taps_on_either_side_of_the_chirps_lines(lam):
    """Chirp transforms from 4096 samples with 512 lags, from 6144 with fewer: the same bar."""
    _taps(np.array([4095, 4096, 4097, 6143, 6144, 6145]), lam, range(6))
