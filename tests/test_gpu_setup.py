"""Numerical setup kernels at the edges of their tiles, through the applies
they feed, against the FP64 oracle."""
import sys

import numpy as np
import pytest

from oracle import gdsw_oracle as O
from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu


def _apply_matches(pr, tol=1e-12, Z=None, oracle_local="exact", coarse=None, **options):
    """M^{-1} r to `tol` of the oracle's max-norm: FP64 factors of matrices
    with condition numbers below 1e3 (1e-16 x 1e3, and a margin of 10)."""
    import torch
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, Z, **options)
    M = O.GDSW(pr.A, pr.part, pr.dpn, pr.n_parts, Z=Z, local=oracle_local)
    r = P.rhs_uniform(pr.n, 3)
    z = torch.zeros(pr.n, dtype=torch.float64, device="cuda")
    g.apply(torch.from_numpy(r).cuda(), z)
    zr = M.apply(r)
    g.close()
    assert np.abs(z.cpu().numpy() - zr).max() <= tol * np.abs(zr).max()


# one part: rows N^3 and band N^2 on both sides of the 16- and 32-wide panels
# (8 rows, 27, 64 = two panels, 125, 216, 512 = whole blocks of 64); several:
# interiors of every size down to one row, bands narrower than a panel
@pytest.mark.parametrize("N,boxes", [(2, 1), (3, 1), (4, 1), (5, 1), (6, 1), (8, 1), (4, 2), (7, 3), (9, 2), (17, 2)])
def test_band_cholesky(N, boxes):
    _apply_matches(P.poisson3d(N, boxes))


# supernodes of one column up to separators of several blocks of 16 columns and
# panels past the 64 rows one wavefront eliminates (17^3 and 20^3 in one part:
# separators of more than 200 columns); leaves alone (3^3)
@pytest.mark.parametrize("N,boxes", [(3, 1), (5, 1), (9, 1), (13, 1), (17, 1), (20, 1), (9, 2), (16, 2)])
def test_supernodal_cholesky(N, boxes):
    _apply_matches(P.poisson3d(N, boxes), exact_order=B.ORDER_ND)


# right-hand sides of the extension on both sides of 16 (24 and more columns per
# interior with rotations), interiors of less and more than one 64-row block
@pytest.mark.parametrize("Ne,boxes,tol", [(6, 2, 1e-11), (8, 2, 1e-11), (9, 3, 1e-11)])
def test_extension_many_columns(Ne, boxes, tol):
    pr = P.elasticity_q1(Ne, boxes)
    _apply_matches(pr, tol=tol, Z=P.rigid_body_modes(pr))   # (condition numbers up to 1e4)


# sweeps by blocks of rows: blocks of 512 and 1,024 rows with a ragged last
# one, more rows than the register-resident forms take (one part of 18^3, 21^3
# rows; ILU(0) and ILU(1)), more slots (ILU(2), ILU(3)), two sweeps (no iterate
# between the first and the last); the streaming sweeps give the same bits
@pytest.mark.parametrize("N,level,sweeps", [(18, 0, 5), (21, 1, 5), (18, 2, 5), (9, 2, 2), (18, 3, 3), (3, 2, 5)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_ilu_block_sweeps(N, level, sweeps, prec):
    import torch
    pr = P.poisson3d(N, 1)
    g = B.Gdsw(pr.A, pr.part, 1, 1, local=B.LOCAL_ILU0, ilu_level=level, jacobi_sweeps=sweeps,
               local_prec=B.FP64 if prec == "fp64" else B.FP32)
    r = torch.from_numpy(P.rhs_uniform(pr.n, 4)).cuda()
    out = []
    for v in range(4):
        try:
            B.gdsw_set_launch(g.h, v, 0, 1, 0)
        except B.GdswError as e:
            assert e.status == 1 and "fit" in str(e)
            continue
        out.append(torch.zeros_like(r))
        g.apply(r, out[-1])
    assert len(out) >= 3 and all(torch.equal(z, out[0]) for z in out)
    if prec == "fp64":
        M = O.GDSW(pr.A, pr.part, 1, 1, local="ilu0", ilu_level=level, sweeps=sweeps)
        zr = M.apply(r.cpu().numpy())
        assert np.abs(out[0].cpu().numpy() - zr).max() <= 1e-12 * np.abs(zr).max()
    g.close()


# The look-ahead band solve (1,024 threads) reads its entries through a window
# that gives zero outside the band and past the subdomain; the 256-thread form
# tests each load.  Same sums in the same order, so the same bits: subdomains of
# one block, bands of 49 (substituted triangles), 64 and 81, ragged last blocks.
@pytest.mark.parametrize("prec", [B.FP64, B.FP32, B.FP16, B.BF16])
@pytest.mark.parametrize("N,boxes", [(6, 2), (7, (1, 1, 2)), (8, (1, 1, 2)), (8, (1, 1, 4)), (9, (1, 1, 3)), (21, 2)])
def test_band_look_ahead(N, boxes, prec):
    import torch
    pr = P.poisson3d(N, boxes)
    print(f"[band look-ahead] {N} {boxes} prec={prec}", file=sys.stderr, flush=True)
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, 1, local=B.LOCAL_EXACT, exact_order=B.ORDER_NATURAL, local_prec=prec,
               basis_prec=B.FP64 if prec == B.FP64 else B.FP32)
    r = torch.from_numpy(P.rhs_uniform(pr.n, 3)).cuda()
    zs = []
    for v in (0, 2):
        B.gdsw_set_launch(g.h, v, 0, 1, 0)
        z = torch.zeros_like(r)
        g.apply(r, z)
        zs.append(z)
    assert bool(torch.isfinite(zs[0]).all())
    assert torch.equal(zs[0], zs[1])
    g.close()
