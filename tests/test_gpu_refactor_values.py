"""The values of a numeric re-setup (Sec. V-A): a non-finite one, wherever it
stands, is refused and leaves the handle as it was; and a process that can start
no further thread can still re-set a handle up."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("N", [5, 40])   # fewer values than one workgroup's threads take, and 438,400
def test_non_finite_values_are_refused(N):
    pr = P.poisson3d(N, 2)
    g = B.Gdsw(pr.A, pr.part, pr.n_parts, 1, local=B.LOCAL_ILU0)
    r = torch.from_numpy(P.rhs_uniform(pr.n, 2)).cuda()
    z0, z1, z2 = torch.zeros_like(r), torch.zeros_like(r), torch.zeros_like(r)
    g.apply(r, z0)
    for at in (0, 1, pr.A.nnz // 2, pr.A.nnz - 1):
        for x in (np.nan, np.inf, -np.inf):
            v = pr.A.data.copy()
            v[at] = x
            with pytest.raises(B.GdswError) as e:
                B.gdsw_refactor(g.h, v)
            assert e.value.status == 1 and "non-finite" in str(e.value)
    g.apply(r, z1)
    assert torch.equal(z1, z0)
    B.gdsw_refactor(g.h, 2.0 * pr.A.data)
    g.apply(r, z2)
    assert float((2.0 * z2 - z0).abs().max()) <= 1e-12 * float(z0.abs().max())
    # a handle whose re-setup failed (a zero row) is unfactored, and checks too
    bad = pr.A.data.copy()
    bad[pr.A.indptr[5]:pr.A.indptr[6]] = 0.0
    with pytest.raises(B.GdswError):
        B.gdsw_refactor(g.h, bad)
    v = pr.A.data.copy()
    v[-1] = np.nan
    with pytest.raises(B.GdswError) as e:
        B.gdsw_refactor(g.h, v)
    assert e.value.status == 1 and "non-finite" in str(e.value)
    B.gdsw_refactor(g.h, pr.A.data)
    g.apply(r, z1)
    assert torch.equal(z1, z0)
    g.close()


AT_LIMIT = """
import resource, sys, threading
sys.path.insert(0, {root!r})
import torch
from paper_2304_04876_amd import binding as B, problems as P
pr = P.poisson3d(40, 2)
g = B.Gdsw(pr.A, pr.part, pr.n_parts, 1, local=B.LOCAL_ILU0)
go, done = threading.Event(), []
def work():
    go.wait()
    B.gdsw_refactor(g.h, 2.0 * pr.A.data)
    done.append(True)
t = threading.Thread(target=work)
t.start()
B.gdsw_refactor(g.h, pr.A.data)
torch.cuda.synchronize()
soft, hard = resource.getrlimit(resource.RLIMIT_NPROC)
resource.setrlimit(resource.RLIMIT_NPROC, (1, hard))
go.set()
t.join()
assert done
print("re-set up", flush=True)
"""


def test_refactor_without_further_threads():
    """(In a process of its own; a user thread started before the limit calls
    gdsw_refactor.)"""
    out = subprocess.run([sys.executable, "-c", AT_LIMIT.format(root=ROOT)], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and "re-set up" in out.stdout, (out.returncode, out.stderr[-600:])
