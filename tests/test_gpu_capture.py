"""The per-frequency stage under graph capture (ftp_solve_sums_noalloc): the
scoring beside the fallback tiers runs in line there.  Every replay, with eager
work between, against the eager call: the same status, the power within 1e-12
(a pair that is not scored keeps the 7 the outputs are filled with)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [4, 11, 13])
def test_capture_equals_eager(H):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_12348_amd as F
    rng = np.random.default_rng(H)
    c, s = rng.standard_normal(H) / np.arange(1, H + 1), rng.standard_normal(H) / np.arange(1, H + 1)
    t = np.sort(rng.uniform(0.0, 100.0, 300))
    y = rng.standard_normal(300)
    sigma = rng.uniform(0.05, 0.2, 300)
    n_f, df = 3000, 1.0 / 500.0
    sums, st = F.Plan(c, s).nfft_sums(t, y, sigma, df, n_f)
    tref, ybar, yy, _ = [float(x) for x in st.cpu()]
    sums = torch.view_as_real(sums).contiguous()
    plan = F.Plan(c, s, solver=F.FTP_SOLVER_UNIFORM)
    stream = torch.cuda.Stream()
    ref, out = F.Plan.alloc_outputs(n_f, sums.device), F.Plan.alloc_outputs(n_f, sums.device)
    plan.solve_sums_noalloc(sums, tref, ybar, yy, df, ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        plan.solve_sums_noalloc(sums, tref, ybar, yy, df, out, stream=stream)
    for _ in range(3):
        for v in out.values():
            v.fill_(7)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out["status"], ref["status"])
        assert float((out["power"] - ref["power"]).abs().max()) <= 1e-12
        for v in out.values():
            v.fill_(7)
        plan.solve_sums_noalloc(sums, tref, ybar, yy, df, out)
        torch.cuda.synchronize()
        assert torch.equal(out["power"], ref["power"])
