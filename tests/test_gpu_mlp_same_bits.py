"""The fused path of the network gives the bits of the layer-by-layer one: outputs,
gradients and the weights after three training steps, for networks at the edges of
what it accepts (six layers with 256 columns, whose training kernel takes 66 KB of
LDS; one layer; narrow layers and layers that end inside a block), at row counts
around its tiles and slices.  The loss is summed in another order: n w_L squares in
FP32, added as trees of partial sums on both paths, differ by less than 64
roundings.  The deepest network is also held to the bfloat16 emulator within one
flipped rounding, 2^-8, per product of the chain."""
import ctypes as C

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu

ROWS = 2000
DEEP = [6, 256, 250, 256, 129, 256, 4]


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return torch, qlskum


def _layered(torch, ql, widths):
    """ql.Mlp of a network that runs layer by layer."""
    m = ql.Mlp.__new__(ql.Mlp)
    m.widths, m.h = list(widths), None
    w = np.ascontiguousarray(widths, np.int32)
    h = C.c_void_p()
    rc = ql.lib.ql_mlp_create_layered(
        C.byref(h), C.c_int(0), C.c_void_p(torch.cuda.current_stream().cuda_stream),
        C.c_void_p(w.ctypes.data), C.c_int(len(widths)), C.c_int64(ROWS))
    assert rc == ql.QL_OK
    m.h = h
    return m


@pytest.mark.parametrize("widths", [DEEP, [128] * 7, [6, 128, 128, 4], [5, 3], [2, 2, 2, 1],
                                    [17, 33, 15, 31], [6, 130, 4], [256, 256]])
def test_fused_equals_layered(env, widths):
    torch, ql = env
    rng = np.random.default_rng(sum(widths))
    w = rng.normal(0.0, 0.2, mlp.n_params(widths)).astype(np.float32)
    nets = [ql.Mlp(widths, max_batch=ROWS), _layered(torch, ql, widths)]
    for n in (1, 16, 33, 511, 1024, 1999):
        print(f"same bits widths={widths} n={n}", flush=True)
        X = torch.tensor(rng.normal(0.0, 1.0, (n, widths[0])), dtype=torch.float32, device="cuda")
        T = torch.tensor(rng.normal(0.0, 1.0, (n, widths[-1])), dtype=torch.float32, device="cuda")
        out = []
        for m in nets:
            m.set_weights(w)
            Y = m.forward(X).cpu().numpy()
            loss, g = m.gradient(X, T)
            for _ in range(3):
                m.train_step(X, T, 1e-3)
            out.append((Y, g, m.get_weights(), loss))
        for a, b in zip(*[o[:3] for o in out]):
            assert np.isfinite(a).all()
            np.testing.assert_array_equal(a, b)
        assert abs(out[0][3] - out[1][3]) <= 64 * 2.0 ** -24 * out[1][3]
    for m in nets:
        m.close()


def test_deepest_network_matches_emulator(env):
    torch, ql = env
    rng = np.random.default_rng(7)
    w = rng.normal(0.0, 0.2, mlp.n_params(DEEP)).astype(np.float32)
    m = ql.Mlp(DEEP, max_batch=ROWS)
    m.set_weights(w)
    tol = (len(DEEP) - 1) * 2.0 ** -8
    for n in (31, 1999):
        print(f"deepest network n={n}", flush=True)
        X = rng.normal(0.0, 1.0, (n, DEEP[0])).astype(np.float32)
        T = rng.normal(0.0, 1.0, (n, DEEP[-1])).astype(np.float32)
        Xd, Td = torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda")
        ref = mlp.forward_bf16(w, DEEP, X)
        assert np.abs(m.forward(Xd).cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
        loss, g = m.gradient(Xd, Td)
        lref, gref = mlp.loss_grad_bf16(w, DEEP, X, T)
        assert np.abs(g - gref).max() <= 2 * tol * np.abs(gref).max()
        assert abs(loss - lref) <= 2 * tol * lref
    m.close()
