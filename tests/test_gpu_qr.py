"""Companion solve at every degree: several matrices per wavefront (many
frequencies), one per wavefront (few), and the work-list form (forced fallback)
give the same bits, and the powers of the Sturm-verified Newton solver."""
import numpy as np
import pytest

from synthetic import tiny_case

pytestmark = pytest.mark.gpu


def _np(out):
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("H", range(1, 16))
def test_companion_forms_agree(H):
    import paper_2101_12348_amd as F

    # 1601 frequencies: past the switch (6 per compute unit of 256), and the
    # last wavefront partly filled whatever the number of matrices it takes
    n_f = 1601
    tmpl, lc = tiny_case(40 + H, n_obs=300, H=H, n_f=n_f, baseline=60.0, cadence="nightly")
    args = (lc.t, lc.y, lc.sigma, lc.df)
    plan = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64)
    many = _np(plan.periodogram(*args, n_f))
    assert np.all(many["status"] == 0)
    sums, st = plan.nfft_sums(*args, n_f)
    tref, ybar, yy, _ = st.cpu().numpy()
    from_sums = _np(plan.solve_sums(sums, tref, ybar, yy, lc.df))
    # the first 101 frequencies alone, from the same sums
    few = _np(plan.solve_sums(sums[:101].contiguous(), tref, ybar, yy, lc.df))
    forced = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM,
                    flags=F.FTP_FLAG_FORCE_FALLBACK)
    listed = _np(forced.solve_sums(sums, tref, ybar, yy, lc.df))
    for k in ("power", "phase", "amp", "offset"):
        assert np.array_equal(few[k], from_sums[k][:101]), k
        assert np.array_equal(listed[k], from_sums[k]), k
    uni = _np(F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM).periodogram(*args, n_f))
    # the power is stationary at the root: a root error of 1e-5 rad changes it by 1e-10
    assert np.max(np.abs(uni["power"] - many["power"])) <= 1e-10
