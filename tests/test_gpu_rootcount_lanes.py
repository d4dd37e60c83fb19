"""The root-count check runs the Sturm chain in the form the solvers run: the same
lanes per chain on either side of 100 thousand frequencies (kernel names of a
profile), its counts the companion matrix's, and most chains trusted."""
import re

import pytest

from synthetic import tiny_case

pytestmark = pytest.mark.gpu


def _lanes(names, pattern):
    return {int(m.group(1)) for n in names if (m := re.search(pattern, n))}


@pytest.mark.parametrize("H,n_f", [(H, n) for H in (3, 5, 6, 7, 8, 9, 10) for n in (501, 100003)])
def test_counts_and_solver_use_the_same_chains(H, n_f):
    import torch
    from torch.profiler import ProfilerActivity, profile
    import paper_2101_12348_amd as F

    tmpl, lc = tiny_case(30 + H, n_obs=200, H=H, n_f=n_f, baseline=60.0 if n_f < 1000 else 2000.0, cadence="nightly")
    plan = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM)
    sums, st = plan.nfft_sums(lc.t, lc.y, lc.sigma, lc.df, n_f)
    tref, ybar, yy, _ = st.cpu().numpy()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        plan.solve_sums(sums, tref, ybar, yy, lc.df)
        sturm, real = plan.root_counts(sums, tref, ybar, yy, lc.df)
        torch.cuda.synchronize()
    names = {e.name for e in prof.events() if "ftp::" in e.name}
    solver = _lanes(names, r"k_newton_sturm4<\d+, \d+, (\d+)\b")
    assert len(solver) == 1 and solver == _lanes(names, r"k_root_counts<(\d+), false>"), names
    # data of 200 observations leave few chains near their thresholds: one in a hundred refused, two
    # at most; and the first round settles most frequencies where the counts are trusted
    sturm, real = sturm.cpu().numpy(), real.cpu().numpy()
    trusted = sturm >= 0
    assert trusted.mean() >= 0.98
    assert (sturm[trusted] == real[trusted]).all()
    assert plan.stats()["n_fallback"] <= 0.2 * n_f
