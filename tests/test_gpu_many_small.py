"""Setup of many small subdomains (Sec. V-B, the exact local solver): copies of
one matrix, one per part, past the counts where the factorisations change their
form, give every copy the bits of the same matrix alone in a handle."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _copies_equal_alone(N, copies, order):
    pr = P.poisson3d(N, 1)
    print(f"[many small] {copies} x {N}^3 order={order}", file=sys.stderr, flush=True)
    opts = dict(local=B.LOCAL_EXACT, exact_order=order, coarse=0)
    r = P.rhs_uniform(pr.n, 8)
    z = []
    for k in (1, copies):
        g = B.Gdsw(sp.block_diag([pr.A] * k, format="csr"), np.repeat(np.arange(k, dtype=np.int32), pr.n), k, 1, **opts)
        z.append(torch.zeros(k * pr.n, dtype=torch.float64, device="cuda"))
        g.apply(torch.from_numpy(np.tile(r, k)).cuda(), z[-1])
        g.close()
    assert torch.equal(z[1].reshape(copies, pr.n), z[0].repeat(copies, 1))


# bands of 4 to 49 (one panel; whole and ragged panels; the last narrow band and
# the first wide one), one more than three matrices per compute unit of 256
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7])
def test_band_cholesky_of_many(N):
    _copies_equal_alone(N, 769, B.ORDER_NATURAL)


# leaves alone up to several heights, with the 128 and the 256 threads that more
# than three and one to three subdomains per compute unit take
@pytest.mark.parametrize("N,copies", [(2, 769), (3, 769), (6, 769), (9, 769), (3, 300), (9, 300), (12, 257)])
def test_supernodal_cholesky_of_many(N, copies):
    _copies_equal_alone(N, copies, B.ORDER_ND)


def test_failing_row_of_one_of_many():
    pr = P.poisson3d(5, 1)
    A = sp.block_diag([pr.A] * 800, format="csr")
    d = A.diagonal()
    d[[700 * pr.n + 77, 700 * pr.n + 90]] = -50.0
    A.setdiag(d)
    with pytest.raises(B.GdswError) as e:
        B.Gdsw(A, np.repeat(np.arange(800, dtype=np.int32), pr.n), 800, 1, local=B.LOCAL_EXACT, coarse=0)
    assert e.value.status == 2 and str(e.value).endswith("in part 700 at row 77"), str(e.value)
