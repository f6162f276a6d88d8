"""GPU: sparse products whose rows crowd in a small box while the columns are
spread and only some of them lie in clumps: a sample of the products tells that
intervals would be too full, and the columns are then sorted and the intervals
bounded by the sample.  Against the oracle: clumps that are and are not found,
small and large intervals, 32- and 64-bit offsets, both roles, repeated rows."""
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


def _box(rng, n, nv, w, repeat):
    flat = rng.choice(w ** nv, n, replace=repeat)
    return np.stack([flat // w ** v % w for v in range(nv)], axis=1).astype(np.int32)


@pytest.mark.parametrize("rows,cols,nv,hi,clumps,size,repeat,kinds", [
    (500, 600, 3, 5000, 1, 100, False, "i64 f64 exact"), (500, 600, 3, 5000, 0, 0, False, "i64"),
    (700, 500, 5, 2000, 2, 90, False, "i64 f64"),       # 64-bit offsets, the box among the columns
    (1500, 1600, 3, 9000, 1, 400, False, "i64"), (2060, 2100, 3, 9000, 1, 400, False, "f64 exact"),
    (2060, 2100, 3, 9000, 250, 8, False, "i64"), (2060, 2100, 3, 9000, 1, 400, True, "i64"),
    (700, 4200, 5, 2000, 2, 300, False, "exact i64"),   # columns placed by a launch of their own
])
def test_matches_oracle(rows, cols, nv, hi, clumps, size, repeat, kinds):
    for kind in kinds.split():
        _check(rows, cols, nv, hi, clumps, size, repeat, kind)


def _check(rows, cols, nv, hi, clumps, size, repeat, kind):
    print("[case] rows in a box:", rows, "x", cols, nv, "variables", clumps, "of", size, kind, flush=True)
    rng = np.random.default_rng([rows, cols, nv, clumps])
    a = _box(rng, rows, nv, int(np.ceil((1.3 * rows) ** (1 / nv))) + 1, repeat)
    b = rng.integers(0, hi, (cols, nv)).astype(np.int32)
    for k in range(clumps):
        b[k * size:(k + 1) * size] = rng.integers(0, hi - 8, nv) + rng.integers(0, 8, (size, nv))
    coef = lambda n: rng.standard_normal(n) if kind == "f64" else rng.integers(-999, 1000, n)
    ca, cb = coef(rows), coef(cols)
    exact = kind == "exact"
    r, lay = kp.mul_laurent(kp.Poly(dev(a), dev(ca)), kp.Poly(dev(b), dev(cb)), mode="hash",
                            exact=exact)
    assert lay.nkeys >= 64 * rows * cols
    oe, oc, oab = O.laurent_mul(a, ca, b, cb, threads=8, **({"exact": True} if exact else {}))
    ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
    if kind == "f64":
        assert_tolerance([ge], gc, [oe], oc, oab, TOL, "rows in a box")
    elif exact:
        for w in (0, 1):
            assert_exact([ge], gc[:, w], [oe], np.asarray(oc)[:, w], f"rows in a box, word {w}")
    else:
        assert_exact([ge], gc, [oe], oc, "rows in a box")
