"""GPU: hash products accumulated straight from the sorted factors (the
default for products spread thinly over the code space) against the oracle:
batch and lane remainders, small and large intervals, 32- and 64-bit offsets,
every way the digits are written, crowded and repeated codes, zero products,
and the errors of a codes call."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from paper_1004_4548_amd import inputs as I
from tests.helpers import assert_exact, assert_tolerance

pytestmark = pytest.mark.gpu
TOL = 1e-13


def say(*a):
    print("[case]", *a, flush=True)


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _factor(rng, n, nv, lo, hi, kind):
    e = I._distinct_uniform(rng, nv, n, lo, hi)
    if kind == "f64":
        return e, rng.standard_normal(n)
    c = rng.integers(-(1 << 61), 1 << 61, n) if kind == "exact" else rng.integers(1, 1000, n)
    return e, c.astype(np.int64)


def _check(a, b, what, kind="i64"):
    say(what, kind, len(a[1]), "x", len(b[1]), a[0].shape[1], "variables")
    exact = kind == "exact"
    r, lay = kp.mul_laurent(kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1])),
                            mode="hash", exact=exact)
    assert lay.nkeys >= 64 * len(a[1]) * len(b[1])   # thin: the route under test
    oe, oc, oab = O.laurent_mul(a[0], a[1], b[0], b[1], threads=8, **({"exact": True} if exact else {}))
    ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
    if kind == "f64":
        assert_tolerance([ge], gc, [oe], oc, oab, TOL, what)
    elif exact:
        for w in (0, 1):
            assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"{what}, word {w}")
    else:
        assert_exact([ge], gc, [oe], oc, what)


@pytest.mark.parametrize("kind", ["i64", "f64", "exact"])
@pytest.mark.parametrize("na,nb,nv,hi", [
    (2, 2, 4, 300), (2, 65, 4, 300), (63, 64, 4, 300), (65, 257, 4, 300),   # lane remainders
    (2049, 2100, 5, 120),                # rows past the small intervals
    (300, 4097, 5, 120), (4097, 300, 5, 120),   # columns placed by a launch of their own; swapped
    (500, 611, 6, 80), (2100, 700, 6, 80), (333, 400, 5, 900),   # 64-bit offsets
    (333, 400, 2, 400000),               # digits past two bytes
    (200, 300, 8, 20), (150, 170, 16, 3),   # more digits than the unrolled copy takes
])
def test_matches_oracle(na, nb, nv, hi, kind):
    rng = np.random.default_rng([na, nb, nv])
    a, b = _factor(rng, na, nv, -hi // 2, hi // 2, kind), _factor(rng, nb, nv, 0, hi, kind)
    _check(a, b, "sparse", kind)


@pytest.mark.parametrize("kind", ["i64", "f64", "exact"])
@pytest.mark.parametrize("rows", [700, 2200])
def test_crowded_codes(rows, kind):
    """Terms crowded in one corner of a box that one outlier makes huge: the
    products fall into a few intervals, which are cut before anything is
    written, and share their cells, so that the table is filled in parts."""
    rng = np.random.default_rng(rows)
    a, b = (_factor(rng, n, 3, 0, 23, kind) for n in (rows, 900))
    for e, _ in (a, b):
        e[0] = (50000, 60000, 70000)
    _check(a, b, "crowded", kind)


def test_repeated_terms():
    """Every term twice: four products in each code, all of them shared."""
    rng = np.random.default_rng(5)
    a, b = _factor(rng, 900, 5, 0, 150, "i64"), _factor(rng, 1100, 5, 0, 150, "i64")
    a, b = ((np.concatenate([e, e]), np.concatenate([c, 3 * c])) for e, c in (a, b))
    _check(a, b, "repeated terms")
    back = (a[0], np.concatenate([a[1][:900], -a[1][:900]]))
    r, _ = kp.mul_laurent(kp.Poly(dev(back[0]), dev(back[1])), kp.Poly(dev(b[0]), dev(b[1])),
                          mode="hash")
    assert r.coef.shape[0] == 0   # every sum cancels


@pytest.mark.parametrize("kind", ["zero terms", "wraps to zero", "underflows"])
def test_zero_products(kind):
    rng = np.random.default_rng(11)
    a, b = _factor(rng, 700, 5, 0, 150, "i64"), _factor(rng, 600, 5, 0, 150, "i64")
    if kind == "zero terms":
        a[1][::3] = 0
    elif kind == "wraps to zero":
        a[1][::3] = 1 << 40
        b[1][::2] = 3 << 24
    else:
        a, b = (a[0], a[1] * 1e-300), (b[0], b[1] * 1.0)
        b[1][::2] = 1e-300
    _check(a, b, kind, "f64" if kind == "underflows" else "i64")


def test_codes_call_and_its_errors():
    import torch
    ctx = kp.context()
    rng = np.random.default_rng(3)
    a, b = _factor(rng, 500, 5, 0, 150, "i64"), _factor(rng, 700, 5, 0, 150, "i64")
    pa, pb = kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1]))
    lay = kp.laurent_layout(pa, pb, ctx)
    ka, kb = kp.encode(lay, 0, pa.exps, ctx=ctx)[0], kp.encode(lay, 1, pb.exps, ctx=ctx)[0]
    codes, coef, _ = kp.mul_laurent_codes(lay, ka, pa.coef, kb, pb.coef, "hash", ctx)
    oe, oc, _ = O.laurent_mul(a[0], a[1], b[0], b[1], threads=4)
    assert_exact([kp.decode(lay, codes, ctx=ctx).cpu().numpy()], coef.cpu().numpy(), [oe], oc,
                 "codes")
    small = (torch.empty(1000, dtype=torch.int64, device="cuda"),
             torch.full((1001,), -7, dtype=torch.int64, device="cuda")[:1000],
             torch.empty(1, dtype=torch.int64, device="cuda"))
    guard = small[1]._base
    with pytest.raises(kp.KPError) as e:
        kp.mul_laurent_codes(lay, ka, pa.coef, kb, pb.coef, "hash", ctx, out=small)
    assert e.value.status == kp.KP_E_CAPACITY
    assert int(guard[1000].item()) == -7
    for which, k in ((0, ka), (1, kb)):
        bad = k.clone()
        bad[7] = lay.nkeys + 5
        args = (bad, pa.coef, kb, pb.coef) if which == 0 else (ka, pa.coef, bad, pb.coef)
        with pytest.raises(kp.KPError) as e:
            kp.mul_laurent_codes(lay, *args, "hash", ctx)
        assert e.value.status == kp.KP_E_RANGE
