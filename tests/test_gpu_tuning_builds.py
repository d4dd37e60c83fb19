"""The tuner measures each build of the Newton kernel once (best of two calls):
there is one for six wavefronts per SIMD and one for five, which newton_occ = 4
selects as well."""
import re

import pytest

from synthetic import tiny_case

pytestmark = pytest.mark.gpu


def _builds(fn):
    import torch
    from torch.profiler import ProfilerActivity, profile

    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return [int(m.group(1)) for e in prof.events() if (m := re.search(r"k_newton_sturm4<\d+, (\d+), \d+\b", e.name))]


def test_each_build_is_measured_once():
    import paper_2101_12348_amd as F

    n_f = 500
    tmpl, lc = tiny_case(12, n_obs=200, H=6, n_f=n_f, baseline=60.0, cadence="nightly")
    plan = F.Plan(tmpl.c, tmpl.s, solver=F.FTP_SOLVER_UNIFORM)
    args = (lc.t, lc.y, lc.sigma, lc.df, n_f)
    for occ, build in ((4, 5), (5, 5), (6, 6)):
        plan.set_tuning(newton_occ=occ)
        assert _builds(lambda: plan.periodogram(*args)) == [build]
    builds = _builds(lambda: plan.autotune(*args))   # from newton_occ = 6
    assert builds.count(5) == 2 and builds.count(6) > 20
