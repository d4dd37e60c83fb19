"""Weight gradients at the boundaries of the batch's splits: one row alone (the
others have no roots and give no gradient) against a batch of that row, where a
row dropped or counted twice shows in full; and the sum of disjoint sets of rows,
whose operands are the same bit for bit, against all of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _boundaries(B):
    # splits of 256 rows, up to 32, each a multiple of 32 rows
    splits = min(32, (B + 255) // 256)
    rows = ((B + splits - 1) // splits + 31) // 32 * 32
    at = {0, 31, 32, 63, 64, B - 65, B - 64, B - 33, B - 32, B - 2, B - 1}
    for s in (1, 2, splits - 1, splits):
        at |= {s * rows - 1, s * rows, s * rows + 1}
    return sorted(b for b in at if 0 <= b < B)


@pytest.mark.parametrize("width", [64, 48])   # the row-tile kernel, one GEMM per layer
@pytest.mark.parametrize("B", [1, 65, 256, 257, 300, 511, 513, 8192, 8200, 8223, 12345])
def test_rows_at_split_boundaries(B, width):
    import torch
    import paper_2101_12348_amd as F

    din, dout, R = 70, 8, 4
    rng = np.random.default_rng(B)
    net = F.Mlp(din, width, dout, seed=7)
    X = torch.as_tensor(rng.standard_normal((B, din)).astype(np.float32), device="cuda").to(torch.bfloat16)
    roots = torch.as_tensor(rng.uniform(0, 2 * np.pi, (B, R)).astype(np.float32), device="cuda")

    def grad(mask):
        return net.loss_grad(X, roots, torch.where(mask, R, 0).to(torch.int32))[1].clone()

    row = torch.arange(B, device="cuda")
    for b in _boundaries(B):
        alone = net.loss_grad(X[b:b + 1], roots[b:b + 1], torch.full((1,), R, dtype=torch.int32, device="cuda"))[1]
        g = B * grad(row == b)
        # the row's gradients are rounded to bf16 with another factor 1 / B in each of four layers
        # (4 x 2^-8 of the largest); a row dropped or doubled is off by the whole
        assert float((g - alone).abs().max()) <= 2e-2 * float(alone.abs().max()), b
    parts = [grad(row % 3 == k) for k in range(3)]
    whole = grad(row >= 0)
    # FP32 sums of up to 12345 rows in another order
    assert float((sum(parts) - whole).abs().max()) <= 1e-5 * float(sum(p.abs() for p in parts).max())
