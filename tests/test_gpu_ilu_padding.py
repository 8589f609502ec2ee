"""Padding slots of the ILU sweeps by blocks of rows (Sec. V-B, Jacobi-sweep
triangular solves): an infinity in a right-hand side reaches only the rows that
couple to it.  Rows with fewer factor entries than the widest are padded with
zeros; the block form keeps only the last rows of an iterate at hand, so a
padding column has to be one of them.  Against the streaming form, which keeps
every row: the rows that are finite in it are the same bits."""
import sys

import numpy as np
import pytest

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one part, no coarse space; reach N^2 (ILU(0)), so rings of 1,024 and 2,048
# places with 512 threads, 2,048 with 1,024: infinities in rows that fall on
# place 0, beside it, and in the last row
@pytest.mark.parametrize("N,level", [(18, 0), (21, 0), (18, 2)])
@pytest.mark.parametrize("prec", [B.FP64, B.FP32])
def test_infinite_entries_stay_with_their_rows(N, level, prec):
    pr = P.poisson3d(N, 1)
    print(f"[ilu padding] N={N} level={level} prec={prec}", file=sys.stderr, flush=True)
    g = B.Gdsw(pr.A, pr.part, 1, 1, local=B.LOCAL_ILU0, ilu_level=level, jacobi_sweeps=5, coarse=0,
               local_prec=prec, basis_prec=prec)
    for row in (1024, 2048, 3072, 4096, 2049, pr.n - 1):
        r = torch.from_numpy(P.rhs_uniform(pr.n, 6)).cuda()
        r[row] = float("inf")
        z = {}
        for v in (3, 0, 1):
            B.gdsw_set_launch(g.h, v, 0, 1, 0)
            z[v] = torch.zeros_like(r)
            g.apply(r, z[v])
        finite = torch.isfinite(z[3])
        assert bool(finite.any()) and not bool(finite.all())
        for v in (0, 1):
            assert torch.equal(z[v][finite], z[3][finite]), (row, v, int((~torch.isfinite(z[v][finite])).sum()))
    g.close()
