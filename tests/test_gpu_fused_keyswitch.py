"""Key switching with both transforms of a step in one launch (few target
limbs, one special prime) against the two-launch form that many targets take:
the same residues bit for bit.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,m,n", [("C1", 16, 256), ("C2", 5, 700), ("C3", 9, 1000), ("C4", 9, 1000), ("C5", 3, 900)])
def test_few_and_many_targets(name, m, n):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    L1, N = ctx.L + 1, ctx.N
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(8)
    pt = dev_f64(plan.bytes("pt") // 8)
    ctx.pt_import(ctx.L, True, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (plan.info["n_pts"], N))), pt)
    beta = -(-L1 // ctx.alpha)
    tasks = beta * (L1 + ctx.alpha)
    for count in (1, 256 // tasks, 256 // tasks + 1, 256 // (2 * L1) + 1):   # each side of 256 targets, both steps
        cts, outs, want = [], [], []
        for k in range(count):
            ct = dev_f64(plan.bytes("ct_in") // 8)
            ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, N)), 60 + k, ct)
            w = dev_f64(plan.bytes("ct_out") // 8)
            plan.matmul(ct, pt, keys, w)
            cts.append(ct)
            want.append(w)
            outs.append(dev_f64(w.numel()).fill_(float("nan")))
        b = pvfl.Batch(ctx, [plan] * count, pt=[pt] * count, ct=cts, out=outs, keys=keys)
        b.matmul()
        t.cuda.synchronize()
        for o, w in zip(outs, want):
            assert t.equal(o, w), count
