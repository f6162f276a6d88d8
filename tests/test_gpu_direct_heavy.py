"""GPU: crowded sparse products whose intervals hold far too many products in
one code or in few: one term many times, and terms at an even gap, where an
interval's samples may all be one code.  Their cuts have to end."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from tests.helpers import assert_exact, assert_tolerance

pytestmark = pytest.mark.gpu
TOL = 1e-13


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _mul(a, b, kind):
    r, lay = kp.mul_laurent(kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1])),
                            mode="hash", exact=kind == "exact")
    assert lay.nkeys >= 64 * len(a[1]) * len(b[1])
    return r.exps.cpu().numpy(), r.coef.cpu().numpy()


@pytest.mark.parametrize("kind", ["i64", "f64", "exact"])
@pytest.mark.parametrize("copies,terms", [(200, 1), (200, 2), (120, 70), (3000, 1)])
def test_terms_many_times(copies, terms, kind):
    print("[case] heavy codes:", copies, "copies of", terms, kind, flush=True)
    rng = np.random.default_rng([copies, terms])
    e = np.repeat(rng.integers(0, 100, (terms, 2)), copies, 0).astype(np.int32)
    e = np.concatenate([e, [[150000, 160000]]]).astype(np.int32)
    c = rng.standard_normal(len(e)) if kind == "f64" else rng.integers(-999, 1000, len(e))
    a = (e, c if kind == "f64" else c.astype(np.int64))
    ge, gc = _mul(a, a, kind)
    oe, oc, oab = O.laurent_mul(*a, *a, threads=8, **({"exact": True} if kind == "exact" else {}))
    if kind == "f64":
        assert_tolerance([ge], gc, [oe], oc, oab, TOL, "heavy")
    elif kind == "exact":
        for w in (0, 1):
            assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"heavy, word {w}")
    else:
        assert_exact([ge], gc, [oe], oc, "heavy")


@pytest.mark.parametrize("kind", ["i64", "f64"])
@pytest.mark.parametrize("n,gap", [(1500, 64), (1500, 1000), (20000, 100)])
def test_even_gaps(n, gap, kind):
    """(sum of c_j t^(gap j) + d u^far)^2, its sums whole numbers in fp64 too."""
    print("[case] even gaps:", n, gap, kind, flush=True)
    rng = np.random.default_rng([n, gap])
    far, d = 60000, 7
    c = rng.integers(1, 1000, n)
    e = np.zeros((n + 1, 2), np.int32)
    e[:n, 0] = gap * np.arange(n)
    e[n] = (0, far)
    both = np.concatenate([c, [d]])
    order = rng.permutation(n + 1)
    a = (e[order], both[order].astype(np.float64 if kind == "f64" else np.int64))
    ge, gc = _mul(a, a, kind)
    want = np.concatenate([np.convolve(c, c), 2 * d * c, [d * d]])
    at = np.zeros((len(want), 2), np.int64)
    at[:2 * n - 1, 0] = gap * np.arange(2 * n - 1)
    at[2 * n - 1:3 * n - 1, 0] = gap * np.arange(n)
    at[2 * n - 1:, 1] = far
    at[-1] = (0, 2 * far)
    got, exp = np.lexsort(ge.T), np.lexsort(at.T)
    assert len(gc) == len(want)
    assert (ge[got] == at[exp]).all() and (gc[got] == want[exp]).all()


@pytest.mark.parametrize("kind", ["i64", "f64", "exact"])
@pytest.mark.parametrize("terms,copies,hi", [(60, 20, 400), (700, 3, 400), (2300, 2, 2000),
                                             (90, 25, 2000)])
def test_several_products_per_code(terms, copies, hi, kind):
    """Spread terms that repeat: an interval's codes fit its table though its
    products are many times more, fill it, or take several stretches."""
    print("[case] repeated, spread:", terms, "x", copies, kind, flush=True)
    rng = np.random.default_rng([terms, copies])
    e = np.repeat(rng.integers(0, hi, (terms, 5)), copies, 0).astype(np.int32)
    c = rng.standard_normal(len(e)) if kind == "f64" else rng.integers(-999, 1000, len(e))
    order = rng.permutation(len(e))
    a, b = (e, c), (e[order], c[order])
    ge, gc = _mul(a, b, kind)
    oe, oc, oab = O.laurent_mul(*a, *b, threads=8, **({"exact": True} if kind == "exact" else {}))
    if kind == "f64":
        assert_tolerance([ge], gc, [oe], oc, oab, TOL, "repeated")
    elif kind == "exact":
        for w in (0, 1):
            assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"repeated, word {w}")
    else:
        assert_exact([ge], gc, [oe], oc, "repeated")
