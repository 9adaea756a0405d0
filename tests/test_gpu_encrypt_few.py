"""Encryption of many ciphertexts in one call (one workgroup per limb) against
the same ciphertexts one at a time (their transforms side by side): the same
residues bit for bit, under the secret and the public key.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,m,n", [("C1", 16, 16), ("C1", 128, 128), ("C2", 64, 64), ("C4", 16, 16), ("C4", 32, 32),
                                      ("C5", 8, 8), ("C5", 32, 32)])
def test_many_and_single_ciphertexts(name, m, n):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(5)
    pk = ctx.pk_gen(sk, 6)
    L1, N = ctx.L + 1, ctx.N
    plan = ctx.plan(pvfl.PLAN_CTMAT, m, n, n_out=8)
    count = plan.info["ct_in"]
    zero = dev_i64(np.zeros(N))
    H = dev_f64(m * n).view(m, n)
    for many, single in ((lambda o: plan.encrypt(sk, H, 40, o), lambda s, o: ctx.encrypt_coeffs(sk, ctx.L, zero, s, o)),
                         (lambda o: plan.encrypt_pk(pk, H, 40, o), lambda s, o: ctx.encrypt_coeffs_pk(pk, ctx.L, zero, s, o))):
        got = dev_f64(plan.bytes("ct_in") // 8).fill_(float("nan"))
        many(got)
        got = got.view(count, -1)
        for c in range(count):
            want = dev_f64(2 * L1 * N).fill_(float("nan"))
            single(40 + c, want)
            t.cuda.synchronize()
            assert t.equal(got[c], want), c


@pytest.mark.parametrize("name,count", [("C1", 2), ("C2", 50), ("C3", 31), ("C3", 40)])
def test_batch_and_single_vectors(name, count):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(5)
    plan = ctx.plan(pvfl.PLAN_HYBRID, 4, 300, lazy=True)
    g = np.random.default_rng(count)
    r = [t.from_numpy(g.standard_normal(300)).cuda() for _ in range(count)]
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    cts = [dev_f64(plan.bytes("ct_in") // 8).fill_(float("nan")) for _ in range(count)]
    b = pvfl.Batch(ctx, [plan] * count, v=r, pt=[dev_f64(plan.bytes("pt") // 8)] * count, ct=cts,
                   out=[dev_f64(plan.bytes("ct_out") // 8) for _ in range(count)], keys=keys)
    b.encrypt(sk, 90)
    for c in range(count):
        want = dev_f64(plan.bytes("ct_in") // 8)
        plan.encrypt(sk, r[c], 90 + c, want)
        t.cuda.synchronize()
        assert t.equal(cts[c], want), c
