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
