"""Outputs of the network written over its inputs' memory equal those written
apart from them, bit for bit: the same address with narrower, equal and (up to
max_batch rows) wider outputs, and inputs that start inside the outputs.  Widths
of the fused kernels, narrow and wide, and of the layer-by-layer path; row counts
of one row tile, of one chunk of max_batch rows and of several with a remainder."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu

CHUNK = 700


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return torch, qlskum


@pytest.mark.parametrize("widths", [[6, 16, 4], [4, 40, 4], [3, 16, 5], [9, 200, 4], [7, 129, 64],
                                    [6, 300, 4]])
def test_outputs_over_inputs(env, widths):
    torch, ql = env
    rng = np.random.default_rng(sum(widths))
    w0, w1 = widths[0], widths[-1]
    m = ql.Mlp(widths, max_batch=CHUNK)
    m.set_weights(rng.normal(0.0, 0.3, mlp.n_params(widths)).astype(np.float32))
    for n in (1, 33, CHUNK) + ((10 * CHUNK + 17,) if w1 <= w0 else ()):
        # first element of X and of Y in one buffer
        places = [(0, 0)]
        if n <= CHUNK:
            places += [(n * w1 // 2, 0), (0, n * w0 // 2)]
        for ox, oy in places:
            print(f"overlap widths={widths} n={n} X at {ox} Y at {oy}", flush=True)
            buf = torch.zeros(max(ox + n * w0, oy + n * w1), device="cuda")
            X = buf[ox:ox + n * w0].view(n, w0)
            Y = buf[oy:oy + n * w1].view(n, w1)
            X.copy_(torch.tensor(rng.normal(0.0, 1.0, (n, w0)), dtype=torch.float32))
            torch.cuda.synchronize()
            ref = m.forward(X.clone()).cpu().numpy()
            m.forward(X, Y)
            np.testing.assert_array_equal(Y.cpu().numpy(), ref)
    m.close()
