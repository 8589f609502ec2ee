"""Device memory that a handle holds after a numeric re-setup (its setup scratch
stays resident): the coarse inverse by matrix instructions takes no more of it
than the form that read the pivot rows in place, so that a memory budget that was
enough still is."""
import numpy as np
import pytest

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# interiors of one to 27 rows, whose extension is smaller than the pivot rows
@pytest.mark.parametrize("make,bytes_", [
    (lambda: P.poisson3d(9, 3), 933916),
    (lambda: P.poisson3d(24, 8), 148208276),
    (lambda: P.poisson3d(32, 8), 172312900),
    (lambda: P.elasticity_q1(8, 4), 14069520),
    (lambda: P.poisson3d(20, 2), 18939460),
])
def test_memory_after_a_refactor(make, bytes_):
    pr = make()
    free = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, None, local=B.LOCAL_EXACT)
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, None, local=B.LOCAL_EXACT, hbm_budget_bytes=bytes_)
    assert free.info()["n0"] > 32 or pr.n == 8000   # (several blocks of the inverse)
    r = torch.from_numpy(P.rhs_uniform(pr.n, 2)).cuda()
    z0, z1 = torch.zeros_like(r), torch.zeros_like(r)
    free.apply(r, z0)   # (without a cap)
    for _ in range(3):
        g.apply(r, z1)
        assert torch.equal(z0, z1)
        B.gdsw_refactor(g.h, np.ascontiguousarray(pr.A.data))
    assert g.info()["device_bytes"] <= bytes_
    g.close()
    free.close()
