"""GPU: crowded columns in the order that their codes need: one workgroup's
worth, one chunk and many, remainders, buckets inside a chunk and over several,
few codes that repeat,
buckets counted and sorted."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from tests.helpers import assert_exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols,hi", [(2, 2), (65, 4), (4095, 60), (4096, 3), (4097, 60), (8192, 2),
                                     (12289, 25), (60001, 3), (70000, 300),
                                     (900, 25), (20000, 400)])
@pytest.mark.parametrize("rows", [2, 40])
def test_matches_oracle(rows, cols, hi):
    import torch
    rows = min(rows, cols)   # (the columns are the factor of more terms)
    print("[case] crowded order", rows, "x", cols, "in", hi, flush=True)
    rng = np.random.default_rng([rows, cols, hi])
    e = [rng.integers(0, hi, (n, 3)).astype(np.int32) for n in (rows, cols)]
    for x in e:
        x[rng.integers(0, len(x))] = 200000
    c = [rng.integers(-999, 1000, n) for n in (rows, cols)]
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    r, lay = kp.mul_laurent(kp.Poly(dev(e[0]), dev(c[0])), kp.Poly(dev(e[1]), dev(c[1])), mode="hash")
    assert lay.nkeys >= 64 * rows * cols
    oe, oc, _ = O.laurent_mul(e[0], c[0], e[1], c[1], threads=8)
    assert_exact([r.exps.cpu().numpy()], r.coef.cpu().numpy(), [oe], oc, "crowded order")
