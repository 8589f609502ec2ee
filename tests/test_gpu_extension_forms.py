"""The extension solves Phi_I = -A_II^{-1} A_IG Phi_G (eq. (2)) in each of their
forms, through an apply against the FP64 oracle: 16 right-hand sides at a time
(interior bands of 63 to 896) and one at a time (narrower and wider bands).
Tolerances as in the other setup tests: FP64 factors of matrices with condition
numbers up to 1e3 (Poisson) and 1e4 (elasticity), 1e-16 times that and a margin
of 10."""
import sys

import numpy as np
import pytest

from oracle import gdsw_oracle as O
from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def interior_bands(pr, is_gamma):
    """(rows, bandwidth) of every part's interior in its natural order."""
    gamma = np.repeat(np.asarray(is_gamma, bool), pr.dpn)
    part = np.repeat(np.asarray(pr.part), pr.dpn)
    pos = np.zeros(pr.n, dtype=np.int64)
    rows = []
    for p in range(pr.n_parts):
        idx = np.flatnonzero((part == p) & ~gamma)
        pos[idx] = np.arange(len(idx))
        rows.append(len(idx))
    A = pr.A.tocoo()
    keep = ~gamma[A.row] & ~gamma[A.col] & (part[A.row] == part[A.col])
    band = np.zeros(pr.n_parts, dtype=np.int64)
    np.maximum.at(band, part[A.row[keep]], np.abs(pos[A.row[keep]] - pos[A.col[keep]]))
    return np.array(rows), band


# elasticity with rotations: several groups of 16 right-hand sides, ragged last
# blocks of 64 rows; slabs of 29^2 and 30^2 planes: bands of 841, where the
# solved blocks fill the 160 KiB of LDS exactly, and of 900, past them
@pytest.mark.parametrize("case,bmin,bmax", [("elasticity10", 63, 896), ("slabs29", 833, 896), ("slabs30", 897, 1187)])
def test_extension_form_matches_oracle(case, bmin, bmax):
    pr = P.elasticity_q1(10, 2) if case == "elasticity10" else P.poisson3d(int(case[-2:]), (1, 1, 4))
    Z = P.rigid_body_modes(pr) if pr.dpn == 3 else None
    print(f"[extension] {case} n={pr.n}", file=sys.stderr, flush=True)
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, Z)
    rows, band = interior_bands(pr, B.gdsw_copy_map(g.h, B.MAP_IS_GAMMA))
    assert bmin <= band.min() and band.max() <= bmax and (rows % 64 != 0).any(), (rows, band)
    M = O.GDSW(pr.A, pr.part, pr.dpn, pr.n_parts, Z=Z, local="exact")
    r = P.rhs_uniform(pr.n, 3)
    z = torch.zeros(pr.n, dtype=torch.float64, device="cuda")
    g.apply(torch.from_numpy(r).cuda(), z)
    zr = M.apply(r)
    tol = 1e-11 if pr.dpn == 3 else 1e-12
    assert np.abs(z.cpu().numpy() - zr).max() <= tol * np.abs(zr).max()
    g.close()
