"""Frequencies per wavefront of the first Newton round: as few as one or two where
there are few frequencies, up to four or eight where there are many.  The first
n of a set of sums, at every n around the rule's steps and with the last wavefront
partly filled, against the same frequencies in a call of all of them."""
import numpy as np
import pytest

from synthetic import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [1, 3, 5, 6, 10, 11, 12, 15])
def test_first_frequencies_equal_those_of_a_larger_call(H):
    import torch
    import paper_2101_12348_amd as F

    n_all = 20000
    tmpl, lc = tiny_case(40 + H, n_obs=200, H=H, n_f=n_all, baseline=2000.0, cadence="nightly")
    plan = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM)
    sums, st = plan.nfft_sums(lc.t, lc.y, lc.sigma, lc.df, n_all)
    tref, ybar, yy, _ = st.cpu().numpy()
    args = (tref, ybar, yy, lc.df)
    ref = plan.solve_sums(sums, *args)
    for n in (1, 2, 3, 7, 9, 1023, 1025, 2047, 2049, 3073, 4097, 8193, 12289):
        out = plan.solve_sums(sums[:n], *args)
        for k in ref:
            assert torch.equal(out[k], ref[k][:n]), (n, k)
