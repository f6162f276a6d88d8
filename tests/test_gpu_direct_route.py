"""GPU: which products are accumulated straight from the sorted factors.  Hash
statistics tell: only products that share a hash cell enter a table there, so
there is hardly a probe beyond the home slots; the groups' tables take them all."""
import numpy as np
import pytest

import oracle as O
import paper_1004_4548_amd as kp
from paper_1004_4548_amd import inputs as I
from tests.helpers import assert_exact

pytestmark = pytest.mark.gpu


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.fixture
def ctx():
    """A context of its own, at the default knobs."""
    c = kp.Context(0)
    c.hash_stats(True)
    yield c
    c.hash_stats(False)


def _probes(ctx, a, b):
    """Extra probes per product of a checked product."""
    r, lay = kp.mul_laurent(kp.Poly(dev(a[0]), dev(a[1])), kp.Poly(dev(b[0]), dev(b[1])),
                            mode="hash", ctx=ctx)
    ins, extra, _ = ctx.hash_stats_read()
    oe, oc, _ = O.laurent_mul(a[0], a[1], b[0], b[1], threads=4)
    assert_exact([r.exps.cpu().numpy()], r.coef.cpu().numpy(), [oe], oc, "route")
    return extra / ins


@pytest.mark.parametrize("knobs,direct", [
    ({}, True), (dict(hash_bin_fill=55), True), (dict(hash_bin_slots=8192), True),
    (dict(hash_bin_slots=2048, hash_bin_fill=30, hash_rows=32, hash_load=0.35), True),
    (dict(hash_grouping=1), False), (dict(hash_grouping=2), False),
    (dict(hash_grouping=2, hash_bin_slots=2048, hash_max_bin_bits=0), False),
    (dict(hash_partitioned=2, hash_bin_slots=2048), False)])
def test_only_a_grouping_asks_for_groups(ctx, knobs, direct):
    """A tuner's size and fill of the bins leave the route as it is."""
    print("[case] route", knobs, flush=True)
    a, b = I.config(3, scale=0.04)
    ctx.set_tune(**knobs)
    assert (_probes(ctx, a, b) < 0.02) == direct


@pytest.mark.parametrize("exact", [False, True])
def test_codes_outside_a_factors_box(ctx, exact):
    """The factors of a codes call the other way round: one's codes lie outside
    the other's box.  Refused for 8-byte types, a product of 128-bit sums."""
    print("[case] swapped codes", "exact" if exact else "i64", flush=True)
    rng = np.random.default_rng(17)
    a = (rng.integers(0, 40, (300, 5)).astype(np.int32), rng.integers(-999, 1000, 300))
    b = (rng.integers(0, 200, (400, 5)).astype(np.int32), rng.integers(-999, 1000, 400))
    pa, pb = (kp.Poly(dev(e), dev(c)) for e, c in (a, b))
    lay = kp.laurent_layout(pa, pb, ctx)
    assert lay.nkeys >= 64 * 300 * 400
    ka, kb = kp.encode(lay, 0, pa.exps, ctx=ctx)[0], kp.encode(lay, 1, pb.exps, ctx=ctx)[0]
    if not exact:
        with pytest.raises(kp.KPError) as e:
            kp.mul_laurent_codes(lay, kb, pb.coef, ka, pa.coef, "hash", ctx)
        assert e.value.status == kp.KP_E_RANGE
        return
    codes, coef, _ = kp.mul_laurent_codes(lay, kb, pb.coef, ka, pa.coef, "hash", ctx, exact=True)
    oe, oc, _ = O.laurent_mul(a[0], a[1], b[0], b[1], threads=4, exact=True)
    got = kp.decode(lay, codes, ctx=ctx).cpu().numpy()
    for w in (0, 1):
        assert_exact([got], coef.cpu().numpy()[:, w], [oe], np.asarray(oc)[:, w], f"word {w}")
