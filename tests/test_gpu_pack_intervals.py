"""GPU: the intervals of packed batches against the oracle: directly indexed
and hashed ones, roles swapped, tables that overflow, columns crowded in one
bucket (cells bounded by a sample), one code in one interval, and a graph that
replays batches of different shapes."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from paper_1004_4548_amd import inputs as I
from tests.helpers import assert_exact, assert_tolerance

pytestmark = pytest.mark.gpu
TOL = 1e-13


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _factor(rng, n, nv, hi, f64, far=None):
    e = I._distinct_uniform(rng, nv, n, 0, hi)
    if far is not None:
        e[0] = far
    c = rng.standard_normal(n) if f64 else rng.integers(-999, 1000, n).astype(np.int64)
    return e, c


def _tasks(seed):
    rng = np.random.default_rng(seed)
    out = []
    for f64 in (False, True):
        for na, nb, nv, hi, far in (
                (40, 700, 1, 5000, None),               # directly indexed
                (700, 41, 1, 100000, None),             # roles swapped
                (257, 300, 4, 90, None),                # hashed
                (600, 500, 3, 11, (2**18,) * 3),    # crowded: 23^3 codes, many shared
                (600, 640, 5, 30, (2**11,) * 5),        # crowded: few codes shared
                (1, 900, 5, 30, (2**11,) * 5),          # one row
                (3, 2, 6, 300, None), (1, 1, 2, 9, None)):
            out.append((_factor(rng, na, nv, hi, f64, far), _factor(rng, nb, nv, hi, f64, far)))
    e = np.repeat(np.arange(12, dtype=np.int32)[:, None], 90, 0)   # every code 90 times
    out.append(((e, rng.integers(1, 9, len(e))), (e, rng.integers(1, 9, len(e)))))
    order = rng.permutation(len(out))
    return [out[i] for i in order]


@pytest.mark.parametrize("graph", [False, True])
def test_matches_oracle(graph):
    p = kp.Pack(20)
    for seed in (1, 2, 3):
        tasks = _tasks(seed)[:17 - 4 * (seed == 2)]
        print("[case] pack of", len(tasks), "seed", seed, "graph", graph, flush=True)
        p.launch([(kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1])))
                  for a, b in tasks], graph=graph)
        for (a, b), r in zip(tasks, p.wait()):
            oe, oc, oab = O.laurent_mul(a[0], a[1], b[0], b[1], threads=4)
            ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
            what = f"{len(a[1])} x {len(b[1])}, seed {seed}"
            if gc.dtype == np.float64:
                assert_tolerance([ge], gc, [oe], oc, oab, TOL, what)
            else:
                assert_exact([ge], gc, [oe], oc, what)


@pytest.mark.parametrize("na,nb", [(1, 1), (2, 3), (60, 70), (1, 4000), (300, 2000)])
def test_serving_bound_covers_the_arena(na, nb):
    """The bytes that a server sets aside for products of a pack hold their
    results and the pack's arena."""
    from types import SimpleNamespace
    from paper_1004_4548_amd import serve
    rng = np.random.default_rng([na, nb])
    (ea, ca), (eb, cb) = _factor(rng, na, 4, 500, False), _factor(rng, nb, 4, 500, False)
    prods = [(kp.Poly(dev(ea), dev(ca)), kp.Poly(dev(eb), dev(cb))) for _ in range(7)]
    _, nbytes = kp.Pack(8).plan(prods)
    s = SimpleNamespace(a=prods[0][0], b=prods[0][1], pairs=na * nb)
    assert nbytes <= 7 * serve.pack_bytes(s)
