"""GPU: dense fp64 products large enough that sums are carried from row to row
(terms sorted by code, 2^27 pairs or more), against the oracle: long runs of
codes, short ones and none, equal codes, buckets too full to sort, tile and item
remainders, infinities and NaN."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from tests.helpers import assert_tolerance

pytestmark = pytest.mark.gpu
TOL = 1e-13


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _exps(rng, shape, n):
    if shape == "line":         # one run
        return np.arange(n, dtype=np.int32)[:, None]
    if shape == "even":         # no two consecutive codes, equal gaps
        return 2 * np.arange(n, dtype=np.int32)[:, None]
    if shape == "scattered":    # runs of one to three
        return np.sort(rng.choice(6 * n, n, replace=False)).astype(np.int32)[:, None]
    if shape == "crowded":      # buckets of thousands of terms: one far term
        e = np.arange(n, dtype=np.int32) // 2
        e[0] = 40000000
        return e[:, None]
    if shape == "twice":        # every term twice
        return np.repeat(np.arange((n + 1) // 2, dtype=np.int32), 2)[:n, None]
    out = [(i, j, k) for i in range(41) for j in range(41 - i) for k in range(41 - i - j)]
    return np.array(out, np.int32)[:n]   # simplex: runs of 1 to 41


@pytest.mark.parametrize("shape,na,nb", [("line", 11601, 11603), ("even", 11600, 11593),
                                         ("scattered", 11611, 11600), ("twice", 11601, 11601),
                                         ("simplex", 11480, 11701), ("crowded", 11600, 11600)])
def test_matches_oracle(shape, na, nb):
    print("[case] chain", shape, na, "x", nb, flush=True)
    rng = np.random.default_rng([na, nb])
    a, b = (_exps(rng, shape, n) for n in (na, nb))
    assert len(a) * len(b) >= 1 << 27
    a, b = a[rng.permutation(len(a))], b[rng.permutation(len(b))]
    ca, cb = rng.standard_normal(len(a)), rng.standard_normal(len(b))
    r, _ = kp.mul_laurent(kp.Poly(dev(a), dev(ca)), kp.Poly(dev(b), dev(cb)), mode="dense")
    oe, oc, oab = O.laurent_mul(a, ca, b, cb, threads=8)
    assert_tolerance([r.exps.cpu().numpy()], r.coef.cpu().numpy(), [oe], oc, oab, TOL, shape)


def test_infinities_stay_in_their_slots():
    """An infinite and a NaN coefficient reach exactly the sums they are in."""
    rng = np.random.default_rng(7)
    n = 11600
    e = np.arange(n, dtype=np.int32)[:, None]
    ca, cb = rng.standard_normal(n), np.zeros(n)
    cb[:3] = rng.standard_normal(3)
    ca[5000], ca[9000] = np.inf, np.nan
    cb[3:] = 1e-300 * rng.standard_normal(n - 3)
    r, _ = kp.mul_laurent(kp.Poly(dev(e), dev(ca)), kp.Poly(dev(e), dev(cb)), mode="dense")
    x, c = r.exps.cpu().numpy()[:, 0], r.coef.cpu().numpy()
    low = x < 5000
    assert np.isfinite(c[low]).all() and not np.isfinite(c[(x >= 5000) & (x < 5000 + n)]).any()
    assert np.isnan(c[(x >= 9000) & (x < 9000 + n)]).all()
    assert np.isfinite(c[x >= 9000 + n]).all()
