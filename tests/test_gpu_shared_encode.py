"""A batch whose products share plaintext buffers and bring their matrices: each
plaintext holds what encoding the products one after the other leaves there,
at every ring size.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, torch

pytestmark = pytest.mark.gpu


def _bufs(plans, what):
    return [dev_f64(p.bytes(what) // 8) for p in plans]


@pytest.mark.parametrize("same_matrix", [True, False])
@pytest.mark.parametrize("name,m,n,count", [("C1", 16, 1000, 5), ("C3", 60, 2048, 9), ("C5", 50, 8000, 16)])
def test_one_buffer_for_all_products(name, m, n, count, same_matrix):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    plans = [plan] * count
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(7)
    X = [t.from_numpy(rng.standard_normal((m, n))).cuda() for _ in range(1 if same_matrix else count)]
    X = X * count if same_matrix else X
    v = [t.from_numpy(rng.uniform(-1, 1, n)).cuda() for _ in range(count)]
    want = dev_f64(plan.bytes("pt") // 8)
    plan.encode_pt(X[-1], want)
    pt = dev_f64(want.numel())
    b = pvfl.Batch(ctx, plans, X=X, v=v, pt=[pt] * count, ct=_bufs(plans, "ct_in"), out=_bufs(plans, "ct_out"),
                   y=[dev_f64(m) for _ in plans], keys=keys)
    for go in (b.encode, b.encode, lambda: b.run(sk, 20), lambda: b.run(sk, 20, graph=True), lambda: b.run(sk, 20, graph=True)):
        pt.fill_(float("nan"))
        go()
        t.cuda.synchronize()
        assert t.equal(pt, want)


@pytest.mark.parametrize("name,big,small", [("C1", (16, 1000), (8, 1000)), ("C5", (50, 8000), (20, 5000))])
def test_a_buffer_inside_another(name, big, small):
    """the second product's plaintexts lie two plaintexts into the first one's"""
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plans = [ctx.plan(pvfl.PLAN_HYBRID, *s, lazy=True) for s in (big, small, big)]
    keys = ctx.rotkeys(sk, plans[0].galois(), 4)
    rng = np.random.default_rng(8)
    X = [t.from_numpy(rng.standard_normal(s)).cuda() for s in (big, small, big)]
    one = plans[0].info["pt_limbs"] * ctx.N
    n_small = plans[1].info["n_pts"]
    assert 2 + n_small <= plans[0].info["n_pts"]

    def bufs():
        a, c = dev_f64(plans[0].bytes("pt") // 8), dev_f64(plans[0].bytes("pt") // 8)
        return [a, a[2 * one: (2 + n_small) * one], c]
    want, got = bufs(), bufs()
    for p, x, o in zip(plans, X, want):
        p.encode_pt(x, o)
    b = pvfl.Batch(ctx, plans, X=X, pt=got, ct=_bufs(plans, "ct_in"), out=_bufs(plans, "ct_out"), keys=keys)
    for _ in range(3):
        got[0].fill_(float("nan"))
        got[2].fill_(float("nan"))
        b.encode()
        t.cuda.synchronize()
        assert t.equal(got[0], want[0]) and t.equal(got[2], want[2])
