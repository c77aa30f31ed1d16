"""The inner iteration's entry slots are staged in 16-byte chunks from the
chunk that holds a tile's first entry: tiles whose first entry sits at every
offset in its chunk, and tiles just below, at and above the 2048 slots that the
buffer holds (then read from memory), against sweeps that read every record
from memory (grad_lds 16), bit for bit, for a cloud that ends inside a tile."""
import numpy as np
import pytest

from tests._common import smooth_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum
    return qlskum


def irregular_cloud(k, drop):
    """A random cloud of k neighbours with up to `drop` of each list's last ones left out."""
    from cloudgen import Cloud, random_cloud
    c = random_cloud(2029, seed=11, k=k)
    cnt = np.diff(c.nbr_ptr)
    n = cnt - np.random.RandomState(3).randint(0, drop + 1, c.n)
    keep = np.arange(c.nnz) - np.repeat(c.nbr_ptr[:-1], cnt) < np.repeat(n, cnt)
    return Cloud(x=c.x, y=c.y, nx=c.nx, ny=c.ny, kind=c.kind, nbr_idx=c.nbr_idx[keep],
                 nbr_ptr=np.concatenate([[0], np.cumsum(n)]).astype(np.int32))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("k,drop", [(14, 1), (33, 2)])
def test_entry_chunks(ql, k, drop, precision):
    print(f"entry chunks k={k} precision={precision}", flush=True)
    c = irregular_cloud(k, drop)
    first = np.append(c.nbr_ptr[:-1:64], c.nbr_ptr[-1])
    assert len(set(first % 8)) > 4  # tiles start anywhere in a chunk
    if k == 33:  # and their spans straddle the buffer
        span = first[1:] - (first[:-1] & ~7)
        assert (span[:-1] <= 2048).any() and (span > 2048).any()
    flow = dict(mach=0.5, alpha_deg=1.0, limiter=1, precision=precision, reorder=0)
    U0 = smooth_state(c, mach=0.5, alpha_deg=1.0)
    out = []
    for b in (0, 16, 64 * 1024):
        s = ql.Solver(c, grad_lds=b, **flow)
        s.set_state(U0)
        out.append(s.evaluate()["g"])
        s.close()
    np.testing.assert_array_equal(out[0], out[1])
    np.testing.assert_array_equal(out[2], out[1])
