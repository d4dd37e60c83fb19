"""The transform's passes at every size of an earlier pass (2..512 points in
FP32, 2..256 in FP64), alone and in pairs, against the exact sums at the ends
and in the middle of the range (the modes written last, the pruned edges)."""
import numpy as np
import pytest

from oracle import ftp_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,log2n", [("FP32_SUMS", L) for L in range(12, 25)] +
                         [("FP64", L) for L in range(12, 22)])
def test_sums_at_every_pass_size(precision, log2n):
    import paper_2101_12348_amd as F

    # H = 1: 2 n_f + 1 modes at an oversampling of two fill the grid to 2^log2n - 2
    # (log2n = 12 is the smallest grid: a few frequencies use its first modes)
    n_f = (1 << (log2n - 2)) - 1
    rng = np.random.default_rng(log2n)
    t = np.sort(rng.uniform(0.0, 30.0, 150))
    y, sigma = rng.normal(size=150), rng.uniform(0.1, 0.3, 150)
    df = 1.0 / 300.0
    plan = F.Plan([1.0], [0.0], precision=getattr(F, "FTP_" + precision))
    sums, st = plan.nfft_sums(t, y, sigma, df, n_f)
    tref = float(st[0].cpu())
    js = np.unique(np.clip([1, 2, 3, n_f // 4, n_f // 2 - 1, n_f // 2, n_f // 2 + 1, 3 * n_f // 4, n_f - 1, n_f], 1, n_f))
    zw, zy, _, _ = O.raw_sums(t, y, sigma, df, js, 2, 1, t_ref=tref)
    got = sums.cpu().numpy().reshape(n_f, 3, -1)[js - 1]
    got = got[..., 0] + 1j * got[..., 1] if got.shape[-1] == 2 else got[..., 0]
    ref = np.concatenate([zw, zy], axis=1)
    # a tenth of the degeneracy thresholds, themselves some hundred times the sums'
    # error relative to sum |g| (1 for w; at most max |y - ybar| for y)
    tol = 1e-6 if precision == "FP32_SUMS" else 1e-10
    scale = np.array([1.0, 1.0, np.max(np.abs(y)) + 1.0])
    assert np.max(np.abs(got - ref) / scale) <= tol
