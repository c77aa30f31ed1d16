"""The residual norms of an iteration are formed by extra workgroups of the
first q-derivative passes of stages 2 to 4 (first order in FP64: of the flux
sweeps); a timed run forms them with launches of their own.  Histories and
states of the two are equal bit for bit: one workgroup and one chunk, a cloud of
one chunk and a remainder, and more cases than the workgroups of one XCD round,
with and without inner iterations, in both precisions and orders."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return qlskum


@pytest.mark.parametrize("precision,n_inner,order",
                         [(0, 3, 2), (1, 3, 2), (0, 0, 2), (1, 0, 2), (0, 3, 1), (1, 3, 1)])
@pytest.mark.parametrize("ns,nr,ncase", [(40, 4, 1), (64, 65, 1), (48, 16, 9)])
def test_norms_equal_launches_of_their_own(ql, ns, nr, ncase, precision, n_inner, order):
    from cloudgen import naca_ocloud
    print(f"residual norms {ns}x{nr} cases={ncase} precision={precision} inner={n_inner} "
          f"order={order}",
          flush=True)
    clouds = [naca_ocloud(ns, nr, jitter=0.1, seed=5 + k) for k in range(ncase)]
    out = []
    for timed in (0, 1):
        s = ql.Solver(limiter=1, precision=precision, n_inner=n_inner, order=order)
        s.upload_batch(clouds, [0.5 + 0.02 * k for k in range(ncase)], [1.0] * ncase)
        s.init_freestream()
        ql.ql_set_timing(s.h, timed)
        hist = [s.step(3), s.step(2)]
        assert (ql.ql_kernel_time(s.h, 3)[1] > 0) == bool(timed)
        out.append(hist + [s.fetch_state()])
        s.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and (a != 0).any()
        np.testing.assert_array_equal(a, b)
