"""Device memory a network holds: the activations and errors of its layers at
their own widths (2 bytes a row and column), at most 64 slices of its gradient and
a loss partial per 16 rows, in FP32, and the weights' copies; narrow layers are not
padded to the matrix cores' blocks.  Its outputs and gradient are those of the
bfloat16 emulator within one flipped rounding, 2^-8, per product of the chain."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,rows", [([2, 2, 2, 1], 1 << 22), ([6, 20, 20, 4], 1 << 20),
                                         ([17, 33, 15, 31], 1 << 20)])
def test_memory_held(widths, rows):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum as ql
    print(f"memory of widths {widths}, {rows} rows", flush=True)
    npar = mlp.n_params(widths)
    ql.Mlp(widths, max_batch=rows).close()  # loads the code objects
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    m = ql.Mlp(widths, max_batch=rows)
    held = free - torch.cuda.mem_get_info()[0]
    batch = 2 * rows * (sum(widths[:-1]) + sum(widths[1:]))
    print(f"  held {held / 2 ** 20:.1f} MiB, batch arrays {batch / 2 ** 20:.1f}", flush=True)
    # small allocations and the allocator's granules of 2 MiB
    assert held <= batch + 4 * 64 * npar + rows // 4 + (16 << 20)
    rng = np.random.default_rng(rows)
    w = rng.normal(0.0, 0.3, npar).astype(np.float32)
    m.set_weights(w)
    tol = (len(widths) - 1) * 2.0 ** -8
    for n in (13, 2000):
        X = rng.normal(0.0, 1.0, (n, widths[0])).astype(np.float32)
        T = rng.normal(0.0, 1.0, (n, widths[-1])).astype(np.float32)
        loss, g = m.gradient(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
        lref, gref = mlp.loss_grad_bf16(w, widths, X, T)
        assert np.abs(g - gref).max() <= 2 * tol * np.abs(gref).max()
        assert abs(loss - lref) <= 2 * tol * lref
    m.close()
