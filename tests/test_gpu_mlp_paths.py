"""The network's paths at their edges: the fused one (widths up to 128 and up to
256, up to six layers) and, past either limit, layer by layer.

With small integers every bfloat16 operand and FP32 sum is exact, so a linear
layer of either path equals FP64 bit for bit.  Deep networks are held to the
bfloat16 emulator within one flipped rounding, 2^-8, per product of the chain
(layers forward, twice that with the way back), relative to the largest value.
Row counts around the tiles of 16 and 32, the 256-row slices of the weight
gradient (from 512 rows) and the row counts at which the tile changes."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return torch, qlskum


def _dev(torch, a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda").contiguous()


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a, np.float64) - b)) / max(np.max(np.abs(b)), 1e-30))


@pytest.mark.parametrize("K,N", [(1, 1), (17, 33), (128, 127), (129, 3), (40, 200),
                                 (256, 256), (255, 131), (257, 3), (33, 300)])
def test_linear_rows_exact(env, K, N):
    torch, ql = env
    rng = np.random.default_rng(K + 7 * N)
    w = rng.integers(-4, 5, mlp.n_params([K, N])).astype(np.float64)
    m = ql.Mlp([K, N], max_batch=1100)
    m.set_weights(w)
    for n in (1, 15, 33, 511, 512, 513, 1100, 31):  # a small batch after a large one
        print(f"linear K={K} N={N} n={n}", flush=True)
        X = rng.integers(-4, 5, (n, K)).astype(np.float64)
        _, ref = mlp.forward(w, [K, N], X)
        np.testing.assert_array_equal(m.forward(_dev(torch, X)).cpu().numpy(), ref)
        # the error 2 (y - t) / (n N) is a bfloat16 integer times a scale that
        # is a power of two only if n N is: compare with the scale's rounding
        E = rng.integers(-4, 5, (n, N))
        _, g = m.gradient(_dev(torch, X), _dev(torch, ref - E))
        d = mlp.bf16(np.float32(2.0 / (n * N)) * E.astype(np.float32)).astype(np.float64)
        gref = np.concatenate([(X.T @ d).ravel(), d.sum(axis=0)])
        # sums of n products of equally scaled integers: FP32 rounding only
        np.testing.assert_allclose(g, gref, rtol=0, atol=n * 2.0 ** -24 * 16 * np.abs(d).max())
    m.close()


@pytest.mark.parametrize("widths", [[2, 5, 1], [6, 17, 33, 4], [3, 16, 16, 16, 16, 16, 2],
                                    [128, 128, 128], [3, 16, 16, 16, 16, 16, 16, 2], [6, 130, 4],
                                    [6, 256, 129, 4], [256, 200, 256], [2, 300, 1]])
def test_deep_paths_match_emulator(env, widths):
    torch, ql = env
    rng = np.random.default_rng(len(widths))
    w = rng.normal(0.0, 0.3, mlp.n_params(widths)).astype(np.float32)
    m = ql.Mlp(widths, max_batch=2000)
    m.set_weights(w)
    tol = (len(widths) - 1) * 2.0 ** -8
    for n in (700, 8192 + 5, 32768 + 40):
        print(f"widths {widths}: forward of {n} rows", flush=True)
        X = rng.normal(0.0, 1.0, (n, widths[0])).astype(np.float32)
        assert _rel(m.forward(_dev(torch, X)).cpu().numpy(), mlp.forward_bf16(w, widths, X)) <= tol
    for n in (1, 47, 1999):
        print(f"widths {widths}: gradient of {n} rows", flush=True)
        X = rng.normal(0.0, 1.0, (n, widths[0])).astype(np.float32)
        T = rng.normal(0.0, 1.0, (n, widths[-1])).astype(np.float32)
        loss, g = m.gradient(_dev(torch, X), _dev(torch, T))
        lref, gref = mlp.loss_grad_bf16(w, widths, X, T)
        assert _rel(g, gref) <= 2 * tol and abs(loss - lref) <= 2 * tol * lref
    # one training step moves the weights by Adam's first step on that gradient;
    # the moments are formed with the FP32 values of beta1 and beta2
    l1 = m.train_step(_dev(torch, X), _dev(torch, T), 1e-3)
    g = g.astype(np.float64)
    mom, var = (1.0 - np.float64(np.float32(b)) for b in (0.9, 0.999))
    w1 = w - 1e-3 * (mom * g / (1 - 0.9)) / (np.sqrt(var * g * g / (1 - 0.999)) + 1e-8)
    assert l1 == loss
    np.testing.assert_allclose(m.get_weights(), w1, rtol=2e-6, atol=2e-9)
    m.close()
