"""The Aberth tier on a long list (a wavefront per frequency) and on a short one (a
workgroup): three observations leave thousands of frequencies without a trusted
count, and slices of the same sums leave few.  Every output is the same bit for
bit.  (Not against another solver: where three points can be met exactly MM nearly
vanishes and the power turns on the last bits of the root.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,n_f", [(5, 1200000), (6, 240000), (7, 240000), (8, 120000), (9, 120000), (10, 40000)])
def test_long_list_equals_short_lists(H, n_f):
    import torch
    import paper_2101_12348_amd as F

    rng = np.random.default_rng(3)
    t, y, sigma = np.sort(rng.uniform(0, 80, 3)), rng.standard_normal(3), np.full(3, 0.1)
    q = np.random.default_rng(H)
    c, s = (q.standard_normal(H) / np.arange(1, H + 1) ** 1.2 for _ in range(2))
    df = 1.0 / 800.0
    plan = F.Plan(c, s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM)
    sums, st = plan.nfft_sums(t, y, sigma, df, n_f)
    tref, ybar, yy, _ = st.cpu().numpy()
    args = (tref, ybar, yy, df)
    ref = plan.solve_sums(sums, *args)
    n_list = plan.stats()["n_fallback_aberth"]
    assert n_list * ((6 * H - 2 + 7) // 8) > 20480   # long
    n = 4000   # (the frequencies count from 1 in a call, so a slice starts there)
    out = plan.solve_sums(sums[:n], *args)
    for name in ref:
        assert torch.equal(out[name], ref[name][:n]), name
