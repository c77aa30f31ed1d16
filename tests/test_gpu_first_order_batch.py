"""First-order batched runs with retirement: a case that reaches the drop keeps the
state and the norms of a solo first-order run of that many iterations bit for bit
(the chunk sums of the norms ride in the flux sweeps, and after a retirement the
sweeps run over the live tiles only), in both precisions, both outer conditions,
eager and replayed."""
import numpy as np
import pytest

from cloudgen import naca_ocloud

pytestmark = pytest.mark.gpu

CASES = [dict(ns=48, nr=16, mach=0.63, alpha=2.0), dict(ns=64, nr=24, mach=0.5, alpha=-1.5),
         dict(ns=40, nr=20, mach=0.75, alpha=4.0)]
DROP, MOST = 0.5, 400


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("precision,outer_bc", [(0, 0), (0, 1), (1, 0)])
def test_first_order_retirement(precision, outer_bc, graph):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum as ql
    print(f"first-order batch precision={precision} outer_bc={outer_bc} graph={graph}", flush=True)
    clouds = [naca_ocloud(c["ns"], c["nr"], jitter=0.05, seed=3 + i) for i, c in enumerate(CASES)]
    prm = dict(order=1, precision=precision, outer_bc=outer_bc)

    def solo(i, n):
        s = ql.Solver(clouds[i], mach=CASES[i]["mach"], alpha_deg=CASES[i]["alpha"], **prm)
        s.init_freestream()
        h = s.step(n)
        U = s.fetch_state()
        s.close()
        return U, h

    for check_every in (1, 40):
        s = ql.Solver(**prm)
        offs = s.upload_batch(clouds, [c["mach"] for c in CASES], [c["alpha"] for c in CASES])
        s.init_freestream()
        iters, res = s.batch_run(DROP, MOST, check_every=check_every, graph=graph)
        U = s.fetch_state()
        assert list(s.batch_status()) == [ql.QL_OK] * len(CASES)
        s.close()
        print(f"  check_every={check_every} iterations {iters}", flush=True)
        assert len(set(iters)) > 1 and min(iters) < MOST
        for i in range(len(CASES)):
            Us, h = solo(i, int(iters[i]))
            if iters[i] < MOST:
                assert h[-1, 0] <= DROP * h[0, 0] and np.all(h[:-1, 0] > DROP * h[0, 0])
            np.testing.assert_array_equal(res[i], h[-1])
            np.testing.assert_array_equal(U[:, offs[i]:offs[i + 1]], Us)
