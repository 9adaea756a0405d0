"""The products' exact sums on large residues that are not multiples of the
primes: the ciphertext's, the plaintexts' and the keys' evaluation-domain values
lie near the ends of their ranges, half of the indices with one sign
throughout.  Per-call, batched and giant-step products, every output residue
against the oracle's integers.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import plans as PL
from paper_2405_00482_amd import pvfl
from paper_2405_00482_amd import workloads as W

from gpu_util import context, dev_f64, dev_u64, export, export_ct, host_u64, torch

pytestmark = pytest.mark.gpu


def _near_ends(shape, top, N, seed, first_sign):
    """whole numbers of magnitude top - (0 .. 999), random signs on the odd indices and one sign on the even ones;
    top broadcasts over the last axis (N indices)"""
    t = torch()
    g = t.Generator(device="cuda").manual_seed(seed)
    mag = top - t.floor(t.rand(*shape, N, generator=g, dtype=t.float64, device="cuda") * 1000)
    sign = t.where(t.rand(*shape, N, generator=g, dtype=t.float64, device="cuda") < 0.5, -1.0, 1.0)
    sign[..., ::2] = first_sign
    return mag * sign


def _residue_terms(prm, plan, ct, keys, pts):
    """sum_i pt_i RotL(ct, i) over Q u P, then ModDown, with plaintexts as residues [i][limb][N]"""
    QP = prm.qp(prm.L)
    digits = O.modup(prm, prm.L, ct.c1)

    def term(i):
        t0, t1 = PL.lazy_term(prm, ct, digits, keys, i)
        return [[O.poly_mul(pts[i][r], x[r], q) for r, q in enumerate(QP)] for x in (t0, t1)]
    acc = None
    for t in PL._pmap(term, range(plan.info["mprime"]), 8):
        acc = t if acc is None else [[O.poly_add(a, b, q) for a, b, q in zip(x, y, QP)] for x, y in zip(acc, t)]
    return [O.moddown(prm, prm.L, np.stack(x)) for x in acc]


@pytest.mark.parametrize("name,m,n", [("C2", 256, 4096), ("C3", 128, 4096), ("C4", 64, 2048)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_products_on_large_residues(name, m, n, sign):
    t = torch()
    prm, ctx = O.Params.from_dict(W.params_dict(name)), context(name)
    L1, N, K = ctx.L + 1, ctx.N, ctx.L + 1 + ctx.alpha
    beta = -(-L1 // ctx.alpha)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    mp = plan.info["mprime"]
    assert mp >= 16 and plan.info["n_pts"] == mp
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    q = t.tensor([float(x) for x in ctx.q + ctx.p], dtype=t.float64, device="cuda")[:, None]
    ct = _near_ends((2, L1), q[:L1] - 1, N, 1, sign)
    pt = _near_ends((mp, K), q - 1, N, 2, 1.0)
    n_key = len(keys.galois) * beta * 2 * K * N
    kv = keys._keep[1][: 8 * n_key].view(t.float64).view(-1, K, N)
    kv.copy_(_near_ends((kv.shape[0], K), (q - 1) / 2, N, 3, 1.0))
    # the same numbers as the oracle holds them: canonical residues of the coefficients
    c = export_ct(ctx, ctx.L, ct.view(-1))[0]
    oct_ = O.Ciphertext(c[0], c[1], ctx.L)
    opts = export(ctx, ctx.L, True, pt.view(-1), mp)
    okeys = {}
    for k, g in enumerate(keys.galois):
        out = dev_u64(beta * 2 * K * N)
        keys.export(k, out)
        kk = host_u64(out).reshape(beta, 2, K, N)
        okeys[g] = O.SwitchKey(g, list(kk[:, 0]), list(kk[:, 1]))
    want = _residue_terms(prm, plan, oct_, okeys, opts)
    assert min(np.count_nonzero(w) for w in want) > L1 * N // 2
    got = {"call": dev_f64(2 * L1 * N).fill_(float("nan"))}
    plan.matmul(ct.view(-1), pt.view(-1), keys, got["call"])
    for group, chunk, vec in ((1, 8, 1), (2, 64, 2), (4, 7, 1), (1, 100, 2)):
        outs = [dev_f64(2 * L1 * N).fill_(float("nan")) for _ in range(3)]
        b = pvfl.Batch(ctx, [plan] * 3, pt=[pt.view(-1), pt.clone().view(-1), pt.view(-1)], ct=[ct.view(-1)] * 3, out=outs,
                       keys=keys, group=group, chunk=chunk, vec=vec)
        b.matmul()
        for k, o in enumerate(outs):
            got[f"batch {group} {chunk} {vec} product {k}"] = o
    for what, o in got.items():
        r = export_ct(ctx, ctx.L, o)[0]
        for h in range(2):
            assert np.array_equal(r[h], want[h]), (what, h)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_giant_steps_on_large_residues(sign):
    """giant step 0 alone carries plaintexts (the others' are zero), so that the result is the baby steps' sum"""
    t = torch()
    prm, ctx = O.Params.from_dict(W.params_dict("C2")), context("C2")
    L1, N, K, bs = ctx.L + 1, ctx.N, ctx.L + 1 + ctx.alpha, 128
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, 256, 4096, lazy=True, bsgs=bs)
    mp = plan.info["mprime"]
    assert mp >= 2 * bs
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    q = t.tensor([float(x) for x in ctx.q + ctx.p], dtype=t.float64, device="cuda")[:, None]
    ct = _near_ends((2, L1), q[:L1] - 1, N, 1, sign)
    pt = t.zeros(plan.info["n_pts"], K, N, dtype=t.float64, device="cuda")
    pt[:bs] = _near_ends((bs, K), q - 1, N, 2, 1.0)
    beta = -(-L1 // ctx.alpha)
    kv = keys._keep[1][: 8 * len(keys.galois) * beta * 2 * K * N].view(t.float64).view(-1, K, N)
    kv.copy_(_near_ends((kv.shape[0], K), (q - 1) / 2, N, 3, 1.0))
    c = export_ct(ctx, ctx.L, ct.view(-1))[0]
    opts = export(ctx, ctx.L, True, pt[:bs].view(-1), bs)
    okeys = {}
    for k, g in enumerate(keys.galois):
        out = dev_u64(beta * 2 * K * N)
        keys.export(k, out)
        kk = host_u64(out).reshape(beta, 2, K, N)
        okeys[g] = O.SwitchKey(g, list(kk[:, 0]), list(kk[:, 1]))

    class Babies:
        info = {"mprime": bs}
    want = _residue_terms(prm, Babies, O.Ciphertext(c[0], c[1], ctx.L), okeys, opts)
    assert min(np.count_nonzero(w) for w in want) > L1 * N // 2
    out = dev_f64(2 * L1 * N).fill_(float("nan"))
    plan.matmul(ct.view(-1), pt.view(-1), keys, out)
    got = export_ct(ctx, ctx.L, out)[0]
    for h in range(2):
        assert np.array_equal(got[h], want[h]), h
