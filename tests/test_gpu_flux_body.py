"""The FP64 split fluxes on both sides of the line |S| = u_e sqrt(beta) = 1.25
(local Mach about 1.5) where the flux body changes its form of erfc: states
that lie below it, across it and far above it, against the oracle.  Each
component of R within ten times the distance between the oracle's two builds
(with and without FMA contraction), the bound of the full-size parity tests."""
import numpy as np
import pytest

import oracle
from tests._common import cloud, normwise_rel, smooth_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return qlskum


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("limiter", [0, 1])
@pytest.mark.parametrize("mach", [0.4, 1.49, 3.0])
def test_flux_across_the_near_line(ql, mach, limiter, order):
    print(f"flux body mach={mach} limiter={limiter} order={order}", flush=True)
    c = cloud("jitter")
    U = smooth_state(c, mach=mach, alpha_deg=2.0, amp=0.05)
    prm = dict(mach=mach, alpha_deg=2.0, limiter=limiter, order=order, outer_bc=1)
    m2 = U[1] ** 2 + U[2] ** 2
    S = np.sqrt(m2 / (2.0 * U[0] * 0.4 * (U[3] - 0.5 * m2 / U[0])))
    if mach == 1.49:
        assert S.min() < 1.25 < S.max()
    ref = oracle.Oracle(c, oracle.params(**prm)).evaluate(U)["R"]
    fma = oracle.Oracle(c, oracle.params(**prm), lib=oracle.load(oracle.FMA_LIB)).evaluate(U)["R"]
    s = ql.Solver(c, **prm)
    s.set_state(U)
    R = s.evaluate()["R"]
    s.close()
    err, floor = normwise_rel(R, ref), normwise_rel(fma, ref)
    print("  error", err, "floor", floor, flush=True)
    assert err.max() <= 10.0 * floor.max()


@pytest.mark.parametrize("outer_bc", [0, 1])
@pytest.mark.parametrize("gamma", [1.4, 1.3])
def test_first_order_records(ql, gamma, outer_bc):
    """First order: primitive states staged once per point against states
    converted at every entry from memory (flux_lds 16), and a budget between
    them that stages some tiles only, bit for bit, over a cloud that ends
    inside a tile and holds states past the line above."""
    print(f"first order gamma={gamma} outer_bc={outer_bc}", flush=True)
    c = cloud("small") if outer_bc else cloud("jitter")
    U = smooth_state(c, mach=1.49, alpha_deg=2.0, amp=0.05, gamma=gamma)
    out = []
    for b in (0, 16, 160 * 80):
        s = ql.Solver(c, mach=1.49, alpha_deg=2.0, order=1, gamma=gamma, outer_bc=outer_bc,
                      flux_lds=b)
        s.set_state(U)
        R = s.evaluate()["R"]
        s.set_state(U)
        out.append((R, s.step(5), s.fetch_state()))
        s.close()
    for o in out[1:]:
        for a, b in zip(o, out[0]):
            np.testing.assert_array_equal(a, b)


def test_first_order_full_lds(ql):
    """First order with the whole LDS as the budget, on tiles whose images ask
    for more of it than the kernel's own arrays leave (then read from memory)."""
    from cloudgen import random_cloud
    print("first order full LDS", flush=True)
    c = random_cloud(6000, seed=7, k=40)
    src = np.repeat(np.arange(c.n) // 64, np.diff(c.nbr_ptr))
    slots = [len(set(c.nbr_idx[src == t]) | set(range(64 * t, min(64 * t + 64, c.n))))
             for t in range(8)]
    assert any(80 * k <= 160 * 1024 < 80 * k + 8192 for k in slots) and max(slots) * 80 > 152 * 1024
    U = smooth_state(c, mach=0.5, alpha_deg=1.0)
    out = []
    for b in (16, 160 * 1024):
        s = ql.Solver(c, mach=0.5, alpha_deg=1.0, order=1, flux_lds=b, reorder=0)
        s.set_state(U)
        out.append(s.evaluate()["R"])
        s.close()
    np.testing.assert_array_equal(out[0], out[1])
