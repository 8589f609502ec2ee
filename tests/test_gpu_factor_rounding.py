"""The Cholesky factorisations' square roots, reciprocals and quotients are
correctly rounded (Sec. V-B, the exact local solver): one 2x2 matrix [[d, c],
[c, 2^60]] per subdomain, so that two applies show 1 / sqrt(d) and c / sqrt(d)
to the last bit through products that numpy rounds the same way.

With L = [[s, 0], [l, 2^30]], i = 1 / s: r = (0, 2^60) gives z_0 = -l i (every
other product is by a power of two), r = (1, 0) gives z_0 = i^2 (what l adds is
below half a unit in the last place).  The band divides by s, the supernodal
panel multiplies by 1 / s."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2304_04876_amd import binding as B

pytestmark = pytest.mark.gpu

# 1 / s next to the middle of two doubles: s with all mantissa bits set, and
# divisors of 2^106 - 2 and 2^106 - 4, the other s whose reciprocal a single
# correction of an estimate two units off can miss
HARD = ["0x1.fffffffffffffp+0", "0x1.fffffffffffffp-1", "0x1.fffffffffffffp+1", "0x1.fffffffffffffp-20",
        "0x1.024a3bd98da02p+0", "0x1.0699d36aec84ep+0", "0x1.3a324a526d5eep+0", "0x1.99e1b447e99c2p+0",
        "0x1.ef7930608393ep+0", "0x1.72f10bf899124p+0", "0x1.c928b5b9dc714p+0", "0x1.ffb8a8b628dbcp+0"]


def _hard_quotients(rng, count):
    """(c, s), c < s, with c / s within 2^-106 of the middle of two doubles."""
    out = []
    while len(out) < count:
        s = int(rng.integers(2 ** 52, 2 ** 53)) | 1
        for N in (1, -1):
            M = N * pow(s, -1, 2 ** 54) % 2 ** 54
            c = (s * M - N) // 2 ** 54
            if M & 1 and 2 ** 52 <= c < s:
                out.append((c / 2.0 ** 52, s / 2.0 ** 52))
    return out[:count]


@pytest.mark.parametrize("order", [B.ORDER_NATURAL, B.ORDER_ND])
def test_roots_reciprocals_and_quotients(order):
    import torch
    rng = np.random.default_rng(5)
    pairs = [(c, float.fromhex(h)) for h in HARD for c in (0.0, 1.0, 0.75, float(rng.uniform(0.1, 1)))]
    pairs += _hard_quotients(rng, 200)
    pairs += [(float(c), float(s)) for c, s in zip(rng.uniform(-1, 1, 200), rng.uniform(0.5, 4, 200))]
    c, s = np.array(pairs).T
    c = c * np.exp2(np.floor(np.log2(s)))   # (|c / s| below 4)
    # every d whose rounded root is s: the rounded square, and neighbours of it
    d = np.concatenate([s * s, np.nextafter(s * s, np.inf), np.nextafter(s * s, 0)])
    c, s = np.tile(c, 3), np.tile(s, 3)
    keep = np.sqrt(d) == s
    assert keep[:len(pairs)].all()
    c, s, d = c[keep], s[keep], d[keep]
    m = len(d)
    A = sp.block_diag([np.array([[d[k], c[k]], [c[k], 2.0 ** 60]]) for k in range(m)], format="csr")
    g = B.Gdsw(A, np.repeat(np.arange(m, dtype=np.int32), 2), m, 1, local=B.LOCAL_EXACT, exact_order=order, coarse=0)
    z = torch.zeros(2 * m, dtype=torch.float64, device="cuda")
    inv = 1.0 / s
    g.apply(torch.tensor([1.0, 0.0], dtype=torch.float64, device="cuda").repeat(m), z)
    wrong = s[z.cpu().numpy()[::2] != inv * inv]
    assert not len(wrong), [x.hex() for x in wrong[:4]]
    g.apply(torch.tensor([0.0, 2.0 ** 60], dtype=torch.float64, device="cuda").repeat(m), z)
    l = c / s if order == B.ORDER_NATURAL else c * inv
    wrong = s[z.cpu().numpy()[::2] != -(l * inv)]
    assert not len(wrong), [x.hex() for x in wrong[:4]]
    assert np.array_equal(z.cpu().numpy()[1::2], np.ones(m))
    g.close()
