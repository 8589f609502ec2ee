"""The streaming ILU sweeps with their iterates in global memory (subdomains
whose three vectors do not fit LDS, Sec. V-B): pinned, since the fixed rule takes
the sweeps by blocks of rows there.  Several right-hand-side slots give each
slot's bits alone, the allocation-free apply (which carves the iterates out of
the library's static array) gives gdsw_apply's, and both give the fixed rule's."""
import sys

import numpy as np
import pytest

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_streaming_sweeps_in_global_memory():
    pr, ns = P.poisson3d(40, 2), 3
    print(f"[ilu streaming] n={pr.n}", file=sys.stderr, flush=True)
    one = B.Gdsw(pr.A, pr.part, pr.n_parts, 1, local=B.LOCAL_ILU0)
    many = B.Gdsw(pr.A, pr.part, pr.n_parts, 1, local=B.LOCAL_ILU0, slots=ns)
    # three FP64 vectors of the largest subdomain against 160 KiB
    assert 24 * int(np.diff(B.gdsw_copy_map(one.h, B.MAP_OV_PTR)).max()) > 160 * 1024
    r = torch.from_numpy(np.concatenate([P.rhs_uniform(pr.n, 30 + k) for k in range(ns)])).cuda()
    rule = torch.zeros_like(r)
    many.apply(r, rule)
    for v in (2, 3):
        for g in (one, many):
            B.gdsw_set_launch(g.h, v)
        z = torch.zeros_like(r)
        many.apply(r, z)
        assert torch.equal(z, rule)
        for k in range(ns):
            rk = r[k * pr.n:(k + 1) * pr.n].clone()
            zk, zs = torch.zeros_like(rk), torch.full_like(rk, float("nan"))
            one.apply(rk, zk)
            assert torch.equal(zk, z[k * pr.n:(k + 1) * pr.n]), (v, k)
            B.gdsw_apply_static(one.h, rk, zs)
            assert torch.equal(zs, zk), (v, k)
    one.close()
    many.close()
