"""GPU: sparse products whose columns one outlier crowds into few buckets,
against the oracle: columns sorted by one workgroup and by many, small and
large intervals, 32- and 64-bit offsets, codes that crowd on several scales,
equal codes, one row, the roles swapped."""
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


def _factor(rng, n, nv, hi, far, kind):
    e = rng.integers(0, hi, (n, nv)).astype(np.int32)   # terms may repeat
    e[rng.integers(0, n)] = far
    c = rng.standard_normal(n) if kind == "f64" else rng.integers(-999, 1000, n)
    return e, c if kind == "f64" else c.astype(np.int64)


@pytest.mark.parametrize("kind", ["i64", "f64", "exact"])
@pytest.mark.parametrize("na,nb,nv,hi,far", [
    (1, 700, 3, 24, 50000), (64, 65, 5, 30, 1500), (600, 900, 3, 24, 50000),
    (600, 900, 5, 30, 1500), (900, 600, 2, 400, 500000),
    (200, 4097, 4, 40, 9000), (2100, 2300, 3, 90, 60000), (2060, 4200, 5, 25, 300),
])
def test_matches_oracle(na, nb, nv, hi, far, kind):
    print("[case] crowded", na, "x", nb, nv, "variables", kind, flush=True)
    rng = np.random.default_rng([na, nb, nv])
    a, b = _factor(rng, na, nv, hi, far, kind), _factor(rng, nb, nv, hi, far, kind)
    exact = kind == "exact"
    r, lay = kp.mul_laurent(kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1])),
                            mode="hash", exact=exact)
    assert lay.nkeys >= 64 * na * nb
    oe, oc, oab = O.laurent_mul(a[0], a[1], b[0], b[1], threads=8, **({"exact": True} if exact else {}))
    ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
    if kind == "f64":
        assert_tolerance([ge], gc, [oe], oc, oab, TOL, "crowded")
    elif exact:
        for w in (0, 1):
            assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"crowded, word {w}")
    else:
        assert_exact([ge], gc, [oe], oc, "crowded")
