"""GPU: sparse products whose columns span little of the code space, so that
few rows meet an interval, each with many columns: batches of few rows and of
parts of their columns.  Against the oracle: one to hundreds of rows, fewer
columns than parts, small and large intervals, 32- and 64-bit offsets."""
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


@pytest.mark.parametrize("rows,cols,nv,hi,last,kinds", [
    (2, 3, 3, 500, 1, "i64"), (40, 41, 3, 900, 1, "i64 f64 exact"), (255, 300, 3, 3000, 3, "i64 f64"),
    (257, 900, 5, 1500, 1, "exact i64"),      # 64-bit offsets
    (1200, 1300, 3, 5000, 1, "i64"), (2060, 2100, 3, 9000, 1, "f64"),
    (2060, 2100, 3, 9000, 40, "i64"), (2060, 2100, 5, 1500, 1, "exact"),
    (300, 4200, 3, 6000, 2, "i64"),           # columns placed by a launch of their own
])
def test_matches_oracle(rows, cols, nv, hi, last, kinds):
    rng = np.random.default_rng([rows, cols, nv, last])
    a = rng.integers(0, hi, (rows, nv)).astype(np.int32)
    b = rng.integers(0, hi, (cols, nv)).astype(np.int32)
    b[:, nv - 1] %= last
    for kind in kinds.split():
        print("[case] few rows meet:", rows, "x", cols, nv, "variables", last, kind, flush=True)
        coef = lambda n: rng.standard_normal(n) if kind == "f64" else rng.integers(-999, 1000, n)
        ca, cb = coef(rows), coef(cols)
        exact = kind == "exact"
        r, lay = kp.mul_laurent(kp.Poly(dev(a), dev(ca)), kp.Poly(dev(b), dev(cb)), mode="hash",
                                exact=exact)
        assert lay.nkeys >= 64 * rows * cols
        oe, oc, oab = O.laurent_mul(a, ca, b, cb, threads=8, **({"exact": True} if exact else {}))
        ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
        if kind == "f64":
            assert_tolerance([ge], gc, [oe], oc, oab, TOL, "few rows")
        elif exact:
            for w in (0, 1):
                assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"few rows, word {w}")
        else:
            assert_exact([ge], gc, [oe], oc, "few rows")
