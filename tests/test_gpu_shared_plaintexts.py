"""Products that share their plaintexts (many encrypted columns of one matrix)
against the per-call product, bit for bit: full and ragged groups, chunk
lengths on both sides of the fixed stage row.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,m,n", [("C2", 100, 700), ("C3", 129, 1024), ("C4", 40, 2048)])
def test_columns_give_the_per_call_residues(name, m, n):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(6)
    pt = dev_f64(plan.bytes("pt") // 8)
    ctx.pt_import(ctx.L, True, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (plan.info["n_pts"], ctx.N))), pt)
    cts, want = [], []
    for k in range(9):
        ct = dev_f64(plan.bytes("ct_in") // 8)
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 60 + k, ct)
        o = dev_f64(plan.bytes("ct_out") // 8)
        plan.matmul(ct, pt, keys, o)
        cts.append(ct)
        want.append(o)
    for count, group, chunk, vec in [(9, 2, 64, 2), (9, 4, 64, 1), (8, 2, 65, 2), (3, 2, 7, 1), (2, 1, 32, 1)]:
        outs = [dev_f64(want[0].numel()).fill_(float("nan")) for _ in range(count)]
        b = pvfl.Batch(ctx, [plan] * count, pt=[pt] * count, ct=cts[:count], out=outs, keys=keys, group=group, chunk=chunk,
                       vec=vec)
        b.matmul()
        t.cuda.synchronize()
        for k in range(count):
            assert t.equal(outs[k], want[k]), (count, group, chunk, vec, k)
