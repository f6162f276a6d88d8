"""GPU: packed products whose intervals are cut many times over.  One factor's
terms are x^(20 i), the other's clumps of x^0 .. x^9 at far powers of y: every
product is a term of its own, an interval holds those of a whole clump, and the
table fills from the first rows alone, so that each cut leaves nearly all of
the interval in its last piece."""
import numpy as np
import pytest

import paper_1004_4548_amd as kp

pytestmark = pytest.mark.gpu


def _task(na, clumps, f64, seed):
    import torch
    rng = np.random.default_rng([na, clumps, seed])
    a = np.zeros((na, 2), np.int32)
    a[:, 0] = 20 * np.arange(na)
    y = np.sort(rng.choice(10 ** 9, clumps, replace=False)).astype(np.int32)
    b = np.stack([np.tile(np.arange(10, dtype=np.int32), clumps), np.repeat(y, 10)], axis=1)
    ca, cb = rng.integers(1, 1 << 20, na), rng.integers(1, 1 << 20, len(b))
    t = torch.float64 if f64 else torch.int64
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return (kp.Poly(dev(a), dev(ca).to(t)), kp.Poly(dev(b), dev(cb).to(t))), dev(y)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("na,clumps", [(2000, 210), (6000, 610), (8000, 820)])
def test_every_product_once(na, clumps, f64):
    """Both factors as the rows; whole-number sums, exact in fp64 too."""
    import torch
    print("[case] pack cuts", na, "x", 10 * clumps, "f64" if f64 else "i64", flush=True)
    (a, b), y = _task(na, clumps, f64, 1)
    few = b.exps.shape[0] - na + 1    # the clumps' factor with fewer terms: its terms are the rows
    b2 = kp.Poly(b.exps[few:].contiguous(), b.coef[few:].contiguous())
    p = kp.Pack(4)
    p.launch([(a, b), (a, b2), (b2, a)])
    for r, (u, first) in zip(p.wait(), ((b, 0), (b2, few), (b2, few))):
        x, c = r.exps[:, 0].long(), r.coef
        i, j = x // 20, x % 20
        k = 10 * torch.searchsorted(y, r.exps[:, 1].contiguous()) + j - first
        assert int(j.max()) < 10 and int(k.min()) >= 0 and int(k.max()) < len(u.coef)
        assert len(c) == na * len(u.coef)
        assert bool((torch.bincount(i * len(u.coef) + k, minlength=len(c)) == 1).all())
        assert bool((r.exps[:, 1] == u.exps[k, 1]).all())
        assert bool((c == a.coef[i] * u.coef[k]).all())


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", ["box rows, clumped columns", "box rows, spread columns",
                                   "copies and a far term", "copies of one term, far"])
def test_crowds_match_oracle(shape, f64):
    """Products that crowd though the columns do not, and codes that many
    products share: sampled cells, some taken together, some of one code."""
    import torch
    import oracle as O
    from tests.helpers import assert_exact, assert_tolerance
    print("[case] pack", shape, "f64" if f64 else "i64", flush=True)
    rng = np.random.default_rng([len(shape), f64])
    coef = lambda n: rng.standard_normal(n) if f64 else rng.integers(-999, 1000, n)
    tasks = []
    for n in (300, 1700):
        if shape.startswith("box"):
            flat = rng.choice(15 ** 3, n, replace=False)
            a = np.stack([flat // 15 ** v % 15 for v in range(3)], axis=1)
            b = rng.integers(0, 5000, (n + 100, 3))
            if "clumped" in shape:
                b[:100] = rng.integers(0, 4990, 3) + rng.integers(0, 8, (100, 3))
        else:
            terms = 1 if "one" in shape else 30
            a = np.repeat(rng.integers(0, 20, (terms, 4)), n // terms, 0)
            a[0] = 6000
            b = a[rng.permutation(len(a))]
        a, b = a.astype(np.int32), b.astype(np.int32)
        tasks.append((a, coef(len(a)), b, coef(len(b))))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    p = kp.Pack(4)
    p.launch([(kp.Poly(dev(a), dev(ca)), kp.Poly(dev(b), dev(cb))) for a, ca, b, cb in tasks])
    for (a, ca, b, cb), r in zip(tasks, p.wait()):
        oe, oc, oab = O.laurent_mul(a, ca, b, cb, threads=8)
        ge, gc = r.exps.cpu().numpy(), r.coef.cpu().numpy()
        if f64:
            assert_tolerance([ge], gc, [oe], oc, oab, 1e-13, shape)
        else:
            assert_exact([ge], gc, [oe], oc, shape)
