"""Workspaces between the smallest and the recommended size through the
binding: accepted from the smallest on, refused below it, the result the same.
Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


# more: whether the recommended size is larger than the smallest (giant steps: where the spent partial sums do not
# hold all rotations)
@pytest.mark.parametrize("name,m,n,opts,more", [
    ("C2", 60, 1024, dict(lazy=False), True),
    ("C2", 60, 1024, dict(lazy=False, unhoisted=True), True),
    ("C2", 60, 1024, dict(bsgs=4), False),
    ("C3", 128, 4096, dict(bsgs=4), True),
    ("C2", 60, 1024, dict(lazy=True), False),
])
def test_smallest_workspace(name, m, n, opts, more):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, **opts)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(4)
    i, L1 = plan.info, ctx.L + 1
    ct = dev_f64(plan.bytes("ct_in") // 8)
    ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8, ct)
    pt = dev_f64(plan.bytes("pt") // 8)
    ctx.pt_import(ctx.L, i["pt_limbs"] > L1, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (i["n_pts"], ctx.N))), pt)
    want, got = (dev_f64(plan.bytes("ct_out") // 8) for _ in range(2))
    plan.matmul(ct, pt, keys, want)
    least = plan.workspace_min_bytes()
    assert 0 < least and (least < plan.bytes("workspace") if more else least == plan.bytes("workspace"))
    for size in (least, (least + plan.bytes("workspace")) // 16 * 8, plan.bytes("workspace")):
        got.fill_(float("nan"))
        plan.matmul(ct, pt, keys, got, ws=t.full((size // 8,), float("nan"), dtype=t.float64, device="cuda"))
        t.cuda.synchronize()
        assert t.equal(got, want), size
    with pytest.raises(pvfl.PvflError) as e:
        plan.matmul(ct, pt, keys, got, ws=dev_f64(least // 8 - 1))
    assert e.value.status == pvfl.E_SHAPE


def test_smallest_workspace_of_a_sum():
    t = torch()
    ctx = context("C1")
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, 40, 512, lazy=True)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(4)
    cts, pts = [], []
    for k in range(3):
        ct = dev_f64(plan.bytes("ct_in") // 8)
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8 + k, ct)
        pt = dev_f64(plan.bytes("pt") // 8)
        ctx.pt_import(ctx.L, True, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (plan.info["n_pts"], ctx.N))), pt)
        cts.append(ct)
        pts.append(pt)
    want, got = (dev_f64(plan.bytes("ct_out") // 8) for _ in range(2))
    plan.matmul_sum(cts, pts, keys, want)
    least = plan.workspace_min_bytes(3)
    assert plan.workspace_min_bytes(1) < least <= plan.workspace_sum_bytes(3)
    plan.matmul_sum(cts, pts, keys, got, ws=dev_f64(least // 8))
    t.cuda.synchronize()
    assert t.equal(got, want)
    with pytest.raises(pvfl.PvflError):
        plan.matmul_sum(cts, pts, keys, got, ws=dev_f64(least // 8 - 1))
