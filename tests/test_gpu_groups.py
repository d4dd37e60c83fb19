"""Several frequencies per wavefront at every harmonic count (sixteen or 32 lanes
of the assembly, eight or sixteen of the Sturm chain), with the last group full,
partly filled and alone: the assembly from the grids against that from the same
sums, and the Sturm count against the companion matrix's real eigenvalues."""
import numpy as np
import pytest

from synthetic import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", range(1, 16))
def test_grouped_assembly_and_counts(H):
    import paper_2101_12348_amd as F

    for n_f in (1, 2, 3, 5, 17, 31):
        tmpl, lc = tiny_case(70 + H, n_obs=200, H=H, n_f=n_f, baseline=60.0, cadence="nightly")
        args = (lc.t, lc.y, lc.sigma, lc.df)
        plain = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64)
        uniform = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_UNIFORM)
        sums, st = plain.nfft_sums(*args, n_f)
        tref, ybar, yy, _ = st.cpu().numpy()
        for plan in (plain, uniform):
            ref = plan.solve_sums(sums, tref, ybar, yy, lc.df)
            out = plan.periodogram(*args, n_f)
            # (above H = 10 which method settles a frequency turns on the last bit of the
            # sums, and the given ones are rescaled: the method bits are left out)
            keep = 0xFF if H <= 10 else 0xFF & ~(8 | 16)
            assert np.array_equal(out["status"].cpu().numpy() & keep, ref["status"].cpu().numpy() & keep)
            # the power is stationary at the root: a root error of 1e-5 rad changes it by 1e-10
            assert np.max(np.abs((out["power"] - ref["power"]).cpu().numpy())) <= 1e-10
        sturm, real = (x.cpu().numpy() for x in plain.root_counts(sums, tref, ybar, yy, lc.df))
        trusted = (sturm >= 0) & (real >= 0)
        assert np.array_equal(sturm[trusted], real[trusted])
        assert np.all((sturm >= 2) | (sturm <= -1000))


@pytest.mark.parametrize("H", [2, 3, 6, 10])
def test_tied_roots_take_the_smallest_phase(H):
    import paper_2101_12348_amd as F

    # a template of even harmonics only has period pi: every maximum of the
    # power comes twice, and the candidate of smaller phase is the answer
    n_f = 67
    tmpl, lc = tiny_case(90 + H, n_obs=200, H=H, n_f=n_f, baseline=60.0, cadence="nightly")
    c, s = np.array(tmpl.c), np.array(tmpl.s)
    c[0::2] = s[0::2] = 0.0
    args = (lc.t, lc.y, lc.sigma, lc.df)
    outs = [{k: v.cpu().numpy() for k, v in
             F.Plan(c, s, precision=F.FTP_FP64, solver=solver).periodogram(*args, n_f).items()}
            for solver in (F.FTP_SOLVER_PLAIN, F.FTP_SOLVER_UNIFORM)]
    # stationary power: a root error of 1e-5 rad changes it by 1e-10; the phase by that error
    assert np.max(np.abs(outs[0]["power"] - outs[1]["power"])) <= 1e-10
    d = np.abs(outs[0]["phase"] - outs[1]["phase"])
    assert np.max(np.minimum(d, 2.0 * np.pi - d)) <= 1e-5


@pytest.mark.parametrize("H,n_band", [(1, 1), (5, 16), (6, 9), (10, 1), (10, 16), (11, 2), (13, 16)])
def test_shared_phase_band_tables(H, n_band):
    import paper_2101_12348_amd as F
    from oracle import ftp_oracle as O

    # from one band to the sixteen whose working set leaves one wavefront per
    # workgroup, on both sides of five and ten harmonics
    rng = np.random.default_rng(100 * H + n_band)
    tmpls = [(rng.normal(size=H) / (1 + np.arange(H)), rng.normal(size=H) / (1 + np.arange(H))) for _ in range(n_band)]
    bands = []
    for _ in range(n_band):
        t = np.sort(rng.uniform(0.0, 20.0, 60))
        sig = rng.uniform(0.1, 0.2, 60)
        bands.append((t, np.sin(2 * np.pi * t / 1.7) + sig * rng.normal(size=60), sig))
    df, n_f = 1.0 / 40.0, 37
    out = F.BandsPlan(tmpls, precision=F.FTP_FP64).periodogram_shared_phase(bands, df, n_f)
    ref = O.shared_phase_periodogram(bands, tmpls, df, n_f)
    # the stationary power: a root error of 1e-5 rad changes it by 1e-10; sums to 1e-10
    assert np.max(np.abs(out["power"].cpu().numpy() - ref["power"])) <= 1e-9


@pytest.mark.parametrize("H,width,n_f", [(1, 32, 40), (3, 96, 700), (6, 256, 700), (10, 256, 700), (10, 32, 40)])
def test_network_on_the_list_equals_layer_by_layer(H, width, n_f):
    import paper_2101_12348_amd as F

    # few starts leave a ragged list to the network (a third of the frequencies
    # and more); the fused layers and one GEMM per layer seed the same second round
    rng = np.random.default_rng(H + width)
    tmpl, lc = tiny_case(50 + H, n_obs=200, H=H, n_f=n_f, baseline=60.0, cadence="nightly")
    n = F.mlp_param_count(2 * (6 * H - 1), width, 4 * H)
    w = (rng.normal(size=n) / np.sqrt(width)).astype(np.float32)
    outs = []
    for fused in (1, 0):
        plan = F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=F.FTP_SOLVER_LEARNED, flags=F.FTP_FLAG_2H_STARTS)
        plan.set_tuning(mlp_fused=fused)
        plan.load_mlp(w, width)
        outs.append({k: v.cpu().numpy() for k, v in plan.periodogram(lc.t, lc.y, lc.sigma, lc.df, n_f).items()})
        assert H == 1 or plan.stats()["n_fallback"] > 0
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("H", [6, 7, 8, 9, 10])
def test_eight_chains_per_wavefront_where_there_are_many(H):
    import paper_2101_12348_amd as F

    # either side of 100 thousand frequencies, the last wavefront partly filled
    for n_f in (99997, 100003):
        tmpl, lc = tiny_case(30 + H, n_obs=200, H=H, n_f=n_f, baseline=2000.0, cadence="nightly")
        args = (lc.t, lc.y, lc.sigma, lc.df, n_f)
        uni, plain = (F.Plan(tmpl.c, tmpl.s, precision=F.FTP_FP64, solver=s).periodogram(*args)
                      for s in (F.FTP_SOLVER_UNIFORM, F.FTP_SOLVER_PLAIN))
        # the power is stationary at the root: a root error of 1e-5 rad changes it by 1e-10
        assert float((uni["power"] - plain["power"]).abs().max()) <= 1e-10
        assert int((uni["status"] & 7).max()) == 0
