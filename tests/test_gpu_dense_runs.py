"""GPU: dense fp64 products of two variables large enough that sums are carried
from row to row (terms sorted by code, 2^27 pairs or more), against the oracle:
long runs of codes, short ones and none, equal codes, buckets too full to sort,
tile and item remainders, infinities and NaN; and a dense Poisson product."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from paper_1004_4548_amd import inputs as I
from tests.helpers import assert_tolerance

pytestmark = pytest.mark.gpu
TOL = 1e-13


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _exps(rng, shape, n):
    x = np.zeros((n, 2), np.int32)   # the second variable splits the line in two
    x[n // 2:, 1] = 1
    if shape == "line":         # two runs
        x[:, 0] = np.arange(n)
    elif shape == "even":       # no two consecutive codes, equal gaps
        x[:, 0] = 2 * np.arange(n)
    elif shape == "scattered":  # runs of one to three
        x[:, 0] = np.sort(rng.choice(6 * n, n, replace=False))
    elif shape == "crowded":    # buckets of thousands of terms: one far term
        x[:, 0] = np.arange(n) // 2
        x[0, 0] = 12000000
    else:                       # every term twice
        x[:, 0] = np.arange(n) // 2
    return x


@pytest.mark.parametrize("shape,na,nb", [("line", 11601, 11603), ("even", 11600, 11593),
                                         ("scattered", 11611, 11600), ("twice", 11601, 11601),
                                         ("crowded", 11600, 11600)])
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
    e = np.zeros((n + 1, 2), np.int32)   # (the last term only makes a second variable)
    e[:n, 0] = np.arange(n)
    e[n, 1] = 1
    ca, cb = rng.standard_normal(n + 1), np.zeros(n + 1)
    cb[:3] = rng.standard_normal(3)
    ca[5000], ca[9000] = np.inf, np.nan
    cb[3:] = 1e-300 * rng.standard_normal(n - 2)
    r, _ = kp.mul_laurent(kp.Poly(dev(e), dev(ca)), kp.Poly(dev(e), dev(cb)), mode="dense")
    line = r.exps.cpu().numpy()[:, 1] == 0
    x, c = r.exps.cpu().numpy()[line, 0], r.coef.cpu().numpy()[line]
    low = x < 5000
    assert np.isfinite(c[low]).all() and not np.isfinite(c[(x >= 5000) & (x < 5000 + n)]).any()
    assert np.isnan(c[(x >= 9000) & (x < 9000 + n)]).all()
    assert np.isfinite(c[x >= 9000 + n]).all()


def test_dense_poisson_matches_oracle():
    """A dense Poisson product of 2^27 segmented pairs takes the same steps."""
    n = 8200
    print("[case] dense Poisson", n, "x", n, flush=True)
    a, b = (I.poisson_random(nx=1, ny=2, n=n, xlo=0, xhi=4, jmax=30, cfg=9, factor=k) for k in (0, 1))
    assert 2 * n * n >= 1 << 27
    dts = (np.int32, np.int32, np.uint8, np.float64)
    s = [kp.PoissonSeries(*(dev(np.asarray(f[k], dts[k])) for k in range(4))) for f in (a, b)]
    r, _ = kp.mul_poisson(s[0], s[1], mode="dense")
    ox, oy, ot, oc, oab = O.poisson_mul(a, b, 1, 2, threads=8)
    got = [t.cpu().numpy() for t in (r.x, r.y, r.is_sin[:, None])]
    assert_tolerance(got, r.coef.cpu().numpy(), [ox, oy, np.asarray(ot)[:, None]], oc, oab, TOL,
                     "dense Poisson")
