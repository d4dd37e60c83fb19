"""A batch of more rows than one launch of the row-tile training kernel can take
(2^22 tiles of 32): the same 4096 rows over and over, so every row's loss is
that of the small batch and the gradient is the small batch's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_batch_past_one_launch():
    import torch
    import paper_2101_12348_amd as F

    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    n, B, din, width, dout, R = 4096, (1 << 27) + 37, 1, 32, 2, 1
    rng = np.random.default_rng(3)
    net = F.Mlp(din, width, dout, seed=11)
    X = torch.as_tensor(rng.standard_normal((n, din)).astype(np.float32), device="cuda").to(torch.bfloat16)
    roots = torch.as_tensor(rng.uniform(0, 2 * np.pi, (n, R)).astype(np.float32), device="cuda")
    nroots = torch.ones(n, dtype=torch.int32, device="cuda")
    loss, grads = net.loss_grad(X, roots, nroots)
    loss, grads = loss.clone(), grads.clone()
    rep = B // n + 1
    big = [x.repeat((rep,) + (1,) * (x.dim() - 1))[:B].contiguous() for x in (X, roots, nroots)]
    lb, gb = net.loss_grad(*big)
    assert bool((lb[:rep // 2 * n].view(-1, n) == loss).all()) and bool((lb[-37:] == loss[:37]).all())
    assert bool((lb[-37 - n:-37] == loss).all())
    # gradients: bf16 rounding of each row's gradient, scaled by another 1 / B (2^-8 of the
    # largest), and FP32 sums of 4 million rows per split (1e-3)
    assert float((gb - grads).abs().max()) <= 2e-2 * float(grads.abs().max())
    net.close()
