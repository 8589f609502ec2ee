"""ILU sweeps of rows with many factor entries (Sec. V-B, Jacobi-sweep triangular
solves): the launch forms that read a factor's first or all slots once are
available wherever they were, whatever the number of slots, and give the bits of
the streaming form."""
import sys

import types

import numpy as np
import pytest
import scipy.sparse as sp

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _forms_agree(pr, ns=1, **opts):
    print(f"[ilu forms] n={pr.n} {opts}", file=sys.stderr, flush=True)
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, None, local=B.LOCAL_ILU0, coarse=0, slots=ns, **opts)
    r = torch.from_numpy(np.concatenate([P.rhs_uniform(pr.n, 4 + k) for k in range(ns)])).cuda()
    z = []
    for v in (3, 0, 1, -1):   # streaming, 512 and 1,024 threads, the fixed rule
        B.gdsw_set_launch(g.h, v, 0, 1, 0)
        z.append(torch.zeros_like(r))
        g.apply(r, z[-1])
    assert bool(torch.isfinite(z[0]).all()) and all(torch.equal(x, z[0]) for x in z)
    g.close()


# more slots than the sweeps by blocks of rows take: elasticity (39 and more
# entries a triangle), ILU(4) of the 7-point stencil
@pytest.mark.parametrize("prec", [B.FP64, B.FP32, B.FP16])
@pytest.mark.parametrize("sweeps", [2, 5])
def test_more_than_24_slots(prec, sweeps):
    basis = B.FP64 if prec == B.FP64 else B.FP32
    _forms_agree(P.elasticity_q1(6, 2), local_prec=prec, basis_prec=basis, jacobi_sweeps=sweeps)
    _forms_agree(P.poisson3d(14, 2), local_prec=prec, basis_prec=basis, jacobi_sweeps=sweeps, ilu_level=4)


# ILU(2) and ILU(3), two to four sweeps: subdomains that fill the held form's
# rows (1,694 of 2,048, 4,050 of 4,096) and that do not (324), those with slots
@pytest.mark.parametrize("prec", [B.FP64, B.FP32, B.FP16])
@pytest.mark.parametrize("level,sweeps", [(2, 2), (2, 3), (3, 2), (3, 3), (2, 4)])
@pytest.mark.parametrize("N,boxes,ns", [(22, 2, 1), (30, 2, 1), (12, 2, 3)])
def test_few_sweeps(N, boxes, ns, level, sweeps, prec):
    _forms_agree(P.poisson3d(N, boxes), ns, local_prec=prec, basis_prec=B.FP64 if prec == B.FP64 else B.FP32,
                 jacobi_sweeps=sweeps, ilu_level=level)


def _stencil27(N, boxes):
    """The 27-point stencil on the Poisson problem's grid and boxes."""
    pr = P.poisson3d(N, boxes)
    T = sp.diags([np.ones(N - 1), np.ones(N), np.ones(N - 1)], [-1, 0, 1])
    A = (27.0 * sp.eye(N ** 3) - sp.kron(sp.kron(T, T), T)).tocsr()
    A.sort_indices()
    return types.SimpleNamespace(A=A, part=pr.part, n_parts=pr.n_parts, n=pr.n, dpn=1)


def _red_black(N, boxes):
    """The Poisson problem with the nodes of one colour numbered first (entries
    reach across half of a subdomain)."""
    pr = P.poisson3d(N, boxes)
    i = np.arange(pr.n)
    q = np.argsort((i % N + i // N % N + i // N ** 2) % 2, kind="stable")
    A = pr.A.tocsr()[q][:, q].tocsr()
    A.sort_indices()
    return types.SimpleNamespace(A=A, part=np.asarray(pr.part)[q], n_parts=pr.n_parts, n=pr.n, dpn=1)


# 13 and 15 slots a triangle; three and four sweeps take the held form where
# every thread's rows are full (1,960 rows), five always the blocks
@pytest.mark.parametrize("prec", [B.FP64, B.FP32, B.FP16, B.BF16])
@pytest.mark.parametrize("sweeps", [2, 3, 4, 5])
@pytest.mark.parametrize("make,level", [(lambda: _stencil27(14, 2), 0), (lambda: _red_black(20, (1, 1, 4)), 1)])
def test_13_to_16_slots(make, level, sweeps, prec):
    _forms_agree(make(), local_prec=prec, basis_prec=B.FP64 if prec == B.FP64 else B.FP32, jacobi_sweeps=sweeps,
                 ilu_level=level)
