"""The batched fused kernel against the per-call product, bit for bit: every
way its options choose group sizes and chunk lengths, and residues at the ends
of their ranges, where its exact sums of products are largest.  Needs an
MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu

SHAPES = [(256, 700), (40, 2048), (3, 8), (129, 1024), (64, 300)]   # m' from 1 up, one product in the last group


def _setup(name, extreme):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plans = [ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True) for m, n in SHAPES]
    keys = ctx.rotkeys(sk, sorted({g for p in plans for g in p.galois()}), 4)
    rng = np.random.default_rng(5)
    L1, N = ctx.L + 1, ctx.N
    cts, pts = [], []
    for k, p in enumerate(plans):
        ct = dev_f64(p.bytes("ct_in") // 8)
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, N)), 60 + k, ct)
        pt = dev_f64(p.bytes("pt") // 8)
        ctx.pt_import(ctx.L, True, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (p.info["n_pts"], N))), pt)
        cts.append(ct)
        pts.append(pt)
    if extreme:
        # ciphertexts and plaintexts at +-q (the largest residues a caller may pass), keys at +-(q - 1) / 2 (the
        # largest the generator makes); one sign for half of the indices, so that the sums grow in one direction
        q = t.tensor([float(x) for x in ctx.q + ctx.p], dtype=t.float64, device="cuda")
        sign = t.ones(N, dtype=t.float64, device="cuda")
        sign[1::2] = -1.0
        for ct in cts:
            ct.view(2, L1, N).copy_(q[:L1, None].expand(2, L1, N))
        for pt in pts:
            v = pt.view(-1, L1 + ctx.alpha, N)
            v.copy_((q[:, None] * sign).expand_as(v))
        beta = -(-L1 // ctx.alpha)
        n = len(keys.galois) * beta * 2 * (L1 + ctx.alpha) * N
        kv = keys._keep[1][: 8 * n].view(t.float64).view(-1, L1 + ctx.alpha, N)
        kv.copy_(((q - 1) / 2)[:, None].expand_as(kv))
    want = []
    for p, ct, pt in zip(plans, cts, pts):
        o = dev_f64(p.bytes("ct_out") // 8)
        p.matmul(ct, pt, keys, o)
        want.append(o)
    return ctx, plans, keys, cts, pts, want


@pytest.mark.parametrize("name,extreme", [("C1", False), ("C2", True), ("C3", False), ("C3", True), ("C4", True),
                                          ("C5", False)])
def test_batch_options_give_the_per_call_residues(name, extreme):
    t = torch()
    ctx, plans, keys, cts, pts, want = _setup(name, extreme)
    for group, chunk, vec in [(1, 8, 1), (2, 64, 2), (2, 65, 2), (4, 7, 2), (1, 1024, 2), (2, 1024, 2), (4, 64, 1),
                              (2, 1, 1)]:
        outs = [dev_f64(w.numel()).fill_(float("nan")) for w in want]
        b = pvfl.Batch(ctx, plans, pt=pts, ct=cts, out=outs, keys=keys, group=group, chunk=chunk, vec=vec)
        b.matmul()
        t.cuda.synchronize()
        for k, (o, w) in enumerate(zip(outs, want)):
            assert t.equal(o, w), (group, chunk, vec, SHAPES[k])


def test_chunk_too_long_for_the_group_is_refused():
    ctx, plans, keys, cts, pts, want = _setup("C3", False)
    b = pvfl.Batch(ctx, plans, pt=pts, ct=cts, out=[dev_f64(w.numel()) for w in want], keys=keys, group=4, chunk=1024, vec=1)
    with pytest.raises(pvfl.PvflError):
        b.matmul()
