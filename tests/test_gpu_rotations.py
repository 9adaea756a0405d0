"""Rotations run side by side against the same rotations one at a time: more
rotations than one launch takes, workspaces and scratch for one rotation only,
in-place single rotations, and a captured stream that may not allocate.  Bit
equality throughout (residues are exact integers).  Needs an MI355X."""
import ctypes

import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


def _random(ctx, sk, plan, seed):
    rng = np.random.default_rng(seed)
    L1, i = ctx.L + 1, plan.info
    ct = dev_f64(plan.bytes("ct_in") // 8)
    Q2 = 2 * L1 * ctx.N
    for c in range(i["ct_in"]):
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), seed + c, ct[c * Q2:(c + 1) * Q2])
    pt = dev_f64(plan.bytes("pt") // 8)
    ctx.pt_import(ctx.L, i["pt_limbs"] > L1, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (i["n_pts"], ctx.N))), pt)
    return ct, pt


def _smallest_ws(ctx):
    """bytes for one rotation at a time: digits, ModUp and ModDown buffers, one ciphertext and a half, temporaries"""
    L1, a = ctx.L + 1, ctx.alpha
    K, beta = L1 + a, -(-L1 // a)
    return 8 * ctx.N * (beta * K + L1 + 2 * K + 2 * a + 7 * L1)


@pytest.mark.parametrize("unhoisted", [False, True])
@pytest.mark.parametrize("name,m,n", [("C1", 2, 2048), ("C1", 256, 1024), ("C4", 20, 2000), ("C2", 3000, 5000)])
def test_per_rotation_moddown_on_any_workspace(name, m, n, unhoisted):
    t = torch()
    ctx = context(name)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=False, unhoisted=unhoisted)
    if plan.info["n_pts"] > 300:
        plan = ctx.plan(pvfl.PLAN_HYBRID, 8, n, lazy=False, unhoisted=unhoisted)   # two column blocks
        assert plan.info["col_blocks"] > 1
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    ct, pt = _random(ctx, sk, plan, 50)
    want = dev_f64(plan.bytes("ct_out") // 8)
    plan.matmul(ct, pt, keys, want)
    nb = _smallest_ws(ctx)
    assert nb <= plan.bytes("workspace")
    ws = t.full((nb // 8,), float("nan"), dtype=t.float64, device="cuda")
    got = dev_f64(plan.bytes("ct_out") // 8).fill_(float("nan"))
    call = lambda size: pvfl.lib().pvfl_matmul_ct_pt(plan.h, pvfl._ptr(ct), pvfl._ptr(pt), keys.h, pvfl._ptr(got),  # noqa: E731
                                                     pvfl._ptr(ws), ctypes.c_size_t(size), pvfl._stream())
    assert call(nb - 8) == -2                       # as before: smaller is refused
    assert call(nb) == 0
    t.cuda.synchronize()
    assert t.equal(got, want)


@pytest.mark.parametrize("hoisted", [False, True])
@pytest.mark.parametrize("name", ["C1", "C3", "C4", "C5"])
def test_rotation_in_place(name, hoisted):
    ctx = context(name)
    sk = ctx.keygen(3)
    g = pow(5, 3, 2 * ctx.N)
    keys = ctx.rotkeys(sk, [g], 4)
    rng = np.random.default_rng(9)
    ct = dev_f64(2 * (ctx.L + 1) * ctx.N)
    ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8, ct)
    out = dev_f64(ct.numel())
    ctx.rotate(keys, ctx.L, ct, g, hoisted, out)
    ctx.rotate(keys, ctx.L, ct, g, hoisted, ct)
    torch().cuda.synchronize()
    assert torch().equal(ct, out)


@pytest.mark.parametrize("name,m,n,count", [("C2", 128, 256, 127), ("C4", 64, 16, 15), ("C3", 16, 64, 15)])
def test_conversion_equals_single_rotations(name, m, n, count):
    """diagonal i of A^T is diagonal k of A rotated by r (see pvfl_ctmat_transpose)"""
    ctx = context(name)
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_CTMAT, m, n, n_out=1, pack=(ctx.N // 2) // max(m, n))
    gal = plan.transpose_galois()
    assert len(gal) == count
    keys = ctx.rotkeys(sk, gal, 4)
    ct, _ = _random(ctx, sk, plan, 70)
    got = dev_f64(ct.numel())
    plan.transpose(ct, keys, got)
    lo, hi, Q2 = min(m, n), max(m, n), 2 * (ctx.L + 1) * ctx.N
    one = dev_f64(Q2)
    for i in range(lo):
        k = (lo - i) % lo
        r = i if m >= n else (hi - lo + i if i else 0)
        src = ct[k * Q2:(k + 1) * Q2]
        if r:
            ctx.rotate(keys, ctx.L, src, pow(5, r, 2 * ctx.N), False, one)
        assert torch().equal(got[i * Q2:(i + 1) * Q2], one if r else src), i


@pytest.mark.parametrize("kind", ["row", "transpose"])
def test_captured_without_growing_scratch(kind):
    """a context whose scratch holds one rotation: the captured call runs its
    items one at a time and every replay gives the uncaptured result"""
    t = torch()
    ctx, big = context("C2"), context("C2")
    res = []
    for c, capture in ((big, False), (ctx, True)):
        sk = c.keygen(3)
        if kind == "row":
            plan = c.plan(pvfl.PLAN_ROW, 5, 16)
            gal = plan.galois()
        else:
            plan = c.plan(pvfl.PLAN_CTMAT, 16, 8, n_out=1, pack=c.N // 32)
            gal = plan.transpose_galois()
        keys = c.rotkeys(sk, gal, 4)
        ct, pt = _random(c, sk, plan, 90)
        out = dev_f64(plan.bytes("ct_out" if kind == "row" else "ct_in") // 8)
        run = (lambda: plan.matmul(ct, pt, keys, out)) if kind == "row" else (lambda: plan.transpose(ct, keys, out))
        if not capture:
            run()
            res.append(out.clone())
            continue
        one = dev_f64(2 * (c.L + 1) * c.N)
        c.rotate(keys, c.L, ct[: one.numel()], gal[0], False, one)   # the single-operation scratch exists
        plan.workspace()
        t.cuda.synchronize()
        g = t.cuda.CUDAGraph()
        with t.cuda.graph(g):
            run()
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            t.cuda.synchronize()
            assert t.equal(out, res[0])
