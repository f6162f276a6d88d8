"""GPU: products found from the sorted factors, and packs, against the grouped
layout over many forms of factors: spread terms, boxes, clumps, far terms,
repeated terms, even gaps and flat factors on either side, of every size class,
whole-number sums (exact in fp64 too) in every type."""
import numpy as np
import pytest

import paper_1004_4548_amd as kp

pytestmark = pytest.mark.gpu


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.fixture(scope="module")
def contexts():
    """The default knobs, and groups by two levels of hash bits."""
    groups = kp.Context(0)
    groups.set_tune(hash_grouping=1)
    return kp.Context(0), groups


def _factor(rng, n, nv, hi):
    e = rng.integers(0, hi, (n, nv))
    kind = rng.integers(0, 8)
    if kind == 1:      # a small box
        e %= max(2, int(np.ceil((1.5 * n) ** (1 / nv))))
    elif kind == 2:    # one clump
        m = int(rng.integers(1, n + 1))
        e[:m] = rng.integers(0, hi, nv) // 2 + rng.integers(0, 6, (m, nv))
    elif kind == 3:    # clumps everywhere
        w = int(rng.integers(2, 12))
        e = (e // w * w)[np.arange(n) // w] + rng.integers(0, 4, (n, nv))
    elif kind == 4:    # repeated terms
        e = e[rng.integers(0, max(1, n // int(rng.integers(2, 40))), n)]
    elif kind == 5:    # an even gap in one variable
        e[:, 1:] = 0
        e[:, 0] = int(rng.integers(1, 200)) * np.arange(n)
    elif kind == 6:    # flat in the last variable
        e[:, -1] %= int(rng.integers(1, 4))
    elif kind == 7:    # crowded on several scales
        e = e >> rng.integers(0, max(1, int(hi).bit_length()), (n, 1))
    if rng.random() < 0.4:
        e[int(rng.integers(0, n))] = hi * int(rng.integers(2, 40))
    return e.astype(np.int32), int(kind)


def _sorted(exps, coef):
    import torch
    key = torch.zeros(len(exps), dtype=torch.int64, device="cuda")
    for v in range(exps.shape[1]):
        x = exps[:, v].long()
        key = key * (int(x.max()) - int(x.min()) + 1) + (x - x.min())
    at = torch.argsort(key)
    return exps[at], coef[at]


def _case(seed):
    rng = np.random.default_rng([seed, 71])
    nv = int(rng.integers(2, 7))
    least = 1 if seed % 4 == 0 else 60
    na, nb = (int(np.exp(rng.uniform(np.log(least), np.log(m)))) for m in rng.permutation([4000, 12000]))
    hi = int(np.ceil((400.0 * max(na, nb) ** 2) ** (1 / nv)))
    while True:   # (until the codes fit)
        (a, ka), (b, kb) = _factor(rng, na, nv, hi), _factor(rng, nb, nv, hi)
        spans = np.ptp(a, axis=0) + np.ptp(b, axis=0) + 1
        if np.log2(spans.astype(np.float64)).sum() < 61.5:
            break
    c = [rng.integers(-500, 501, n) for n in (na, nb)]
    return rng, a, c[0], b, c[1], (ka, kb)


@pytest.mark.parametrize("part", range(6))
def test_single_products_equal_the_groups(contexts, part):
    import torch
    for seed in range(part * 25, part * 25 + 25):
        rng, a, ca, b, cb, kinds = _case(seed)
        kind = ("i64", "f64", "exact")[int(rng.integers(0, 3))]
        print("[case] forms", seed, kinds, len(a), "x", len(b), a.shape[1], kind, flush=True)
        t = torch.float64 if kind == "f64" else torch.int64
        pa, pb = kp.Poly(dev(a), dev(ca).to(t)), kp.Poly(dev(b), dev(cb).to(t))
        got, want = (_sorted(r.exps, r.coef) if len(r.coef) else None for r in
                     (kp.mul_laurent(pa, pb, mode="hash", exact=kind == "exact", ctx=c)[0]
                      for c in contexts))
        assert (got is None) == (want is None)
        if got is not None:
            assert got[0].shape == want[0].shape
            assert bool((got[0] == want[0]).all()) and bool((got[1] == want[1]).all())


@pytest.mark.parametrize("part", range(3))
def test_packs_equal_the_groups(contexts, part):
    import torch
    tasks = []
    for seed in range(1000 + part * 20, 1000 + part * 20 + 20):
        rng, a, ca, b, cb, kinds = _case(seed)
        t = torch.float64 if seed % 2 else torch.int64
        tasks.append((kp.Poly(dev(a[:3000]), dev(ca[:3000]).to(t)), kp.Poly(dev(b[:3000]), dev(cb[:3000]).to(t))))
        print("[case] pack forms", seed, kinds, len(tasks[-1][0].coef), "x", len(tasks[-1][1].coef), flush=True)
    p = kp.Pack(len(tasks), contexts[0])
    p.launch(tasks)
    for (u, v), r in zip(tasks, p.wait()):
        w = kp.mul_laurent(u, v, mode="hash", ctx=contexts[1])[0]
        assert r.coef.shape == w.coef.shape
        if len(w.coef):
            got, want = _sorted(r.exps, r.coef), _sorted(w.exps, w.coef)
            assert bool((got[0] == want[0]).all()) and bool((got[1] == want[1]).all())
