"""Which row a failed supernodal factorisation names (Sec. V-B, the exact
local solver on a matrix that is not positive definite): the first non-positive
pivot in the new numbering, however many panels fail at once."""
import numpy as np
import pytest

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_first_failing_row_is_named():
    pr = P.poisson3d(16, 1)
    opts = dict(local=B.LOCAL_EXACT, exact_order=B.ORDER_ND, coarse=0)
    h = B.gdsw_analyze(pr.A, pr.part, 1, 1, None, B.gdsw_default_options(**opts))
    sn = B.gdsw_copy_map(h, B.MAP_ND_SN).reshape(-1, 4)   # first row, columns, rows, height
    perm = B.gdsw_copy_map(h, B.MAP_ND_PERM)              # old local row of a new one
    idx = B.gdsw_copy_map(h, B.MAP_OV_IDX)
    B.gdsw_destroy(h)
    leaves = sn[sn[:, 3] == 0]
    wide = int(np.argmax(leaves[:, 1] > 16))
    assert leaves[wide, 1] > 16 and len(leaves) > wide + 16
    # the last column of one leaf, past its first 16 (the others' are there
    # sooner), and the first column of every later one
    rows = [int(leaves[wide, 0] + leaves[wide, 1] - 1)] + [int(r) for r in leaves[wide + 1:, 0]]
    d = pr.A.diagonal()
    d[idx[perm[rows]]] = -1e6
    A = pr.A.copy()
    A.setdiag(d)
    for _ in range(3):
        with pytest.raises(B.GdswError) as e:
            B.Gdsw(A, pr.part, 1, 1, **opts)
        assert e.value.status == 2 and str(e.value).endswith(f"at row {min(rows)}"), str(e.value)
