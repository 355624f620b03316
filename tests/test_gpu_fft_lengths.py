"""FFT lengths of the FP64 operator that a plan takes by itself, on either side of the lines where
one length's N^-1 becomes faster than another's."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1408_3048_amd import Plan  # noqa: E402


@pytest.mark.parametrize("logn,n_int,lam,n_r", [
    (18, 16, 512, 2048),    # 256 tiles on 256 CUs against 48 pairs
    (18, 16, 1024, 4096),   # 64 pairs against 32 of 8192 points
    (20, 32, 512, 4096),    # 192 pairs against 1024 tiles of 2048 points
    (20, 32, 2048, 8192),   # 128 pairs against 96 tiles of 16384 points
    (21, 32, 512, 4096),    # 352 pairs against 160 of 8192 points, on 256 CUs
    (21, 64, 1024, 4096),   # 512 against 192
    (21, 32, 2048, 8192),
    (22, 32, 2700, 8192),   # 768 pairs against 384 tiles of 16384 points
    (22, 32, 2900, 16384),  # 896 against 416
])
def test_lengths_by_workgroups(logn, n_int, lam, n_r):
    n = 1 << logn
    off = np.linspace(0, n, n_int + 1).astype(np.int64)
    plan = Plan(torch.arange(n, dtype=torch.int32, device="cuda") % 512, None, 512, off,
                np.tile([1.0, 0.0, 1.0], (n_int, 1)), n_stokes=1, lam=lam, rcond_min=0.0)
    assert plan.fft_lengths() == (n_r, 0)
    plan.close()
