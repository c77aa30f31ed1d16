"""Inference of more rows than one launch of the wide fused kernel can hold
(2^28 rows are 2^32 threads): every row is written, and the rows at both ends and
around 2^27 and 2^28 equal those of calls of their own bit for bit (2 GiB of
device memory)."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def test_rows_past_one_launch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum as ql
    widths, n = [1, 129, 1], (1 << 28) + 37
    print(f"widths {widths}: forward of {n} rows", flush=True)
    m = ql.Mlp(widths, max_batch=1000)
    m.set_weights(np.random.default_rng(3).normal(0.0, 0.3, mlp.n_params(widths)).astype(np.float32))
    X = torch.linspace(-4.0, 4.0, n, dtype=torch.float32, device="cuda").view(n, 1)
    Y = torch.full((n, 1), float("nan"), device="cuda")
    torch.cuda.synchronize()
    m.forward(X, Y)
    assert not bool(torch.isnan(Y).any())
    for r in (0, (1 << 27) - 500, (1 << 28) - 500, n - 1000):
        assert torch.equal(m.forward(X[r:r + 1000].clone()), Y[r:r + 1000]), r
    m.close()
