"""The context's scratch of single rotations: which calls leave it large enough
for a captured rotation, and that later calls which fit it leave it where a
captured graph reads it.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


def _capture_and_check(ctx, keys, level, ct, g, hoisted, between=lambda: None):
    """the rotation captured without a warm-up of its own; every replay gives the uncaptured result"""
    t = torch()
    out, want = dev_f64(ct.numel()), dev_f64(ct.numel())
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph):
        ctx.rotate(keys, level, ct, g, hoisted, out)
    ctx.rotate(keys, level, ct, g, hoisted, want)
    for _ in range(3):
        between()
        out.fill_(float("nan"))
        graph.replay()
        t.cuda.synchronize()
        assert t.equal(out, want)


@pytest.mark.parametrize("hoisted", [False, True])
@pytest.mark.parametrize("warm", ["transpose", "row", "rotate_and_sum"])
def test_rotation_captured_after(warm, hoisted):
    t = torch()
    ctx = context("C2")
    sk = ctx.keygen(3)
    rng = np.random.default_rng(5)
    if warm == "transpose":
        plan = ctx.plan(pvfl.PLAN_CTMAT, 16, 8, n_out=1, pack=ctx.N // 32)
        gal, level = plan.transpose_galois(), ctx.L
    elif warm == "row":
        plan = ctx.plan(pvfl.PLAN_ROW, 5, 16)
        gal, level = plan.galois(), ctx.L - 1          # the level ROW's rotate-and-sum runs at
    else:
        plan = ctx.plan(pvfl.PLAN_DIAG, 16, 64, lazy=True, ras_in_ct=True)
        gal, level = plan.galois(), ctx.L
    keys = ctx.rotkeys(sk, gal, 4)
    ct = dev_f64(plan.bytes("ct_in") // 8)
    Q2 = 2 * (ctx.L + 1) * ctx.N
    for c in range(plan.info["ct_in"]):
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8 + c, ct[c * Q2:(c + 1) * Q2])
    if warm == "transpose":
        plan.transpose(ct, keys, dev_f64(ct.numel()))
    else:
        pt = dev_f64(plan.bytes("pt") // 8)
        i = plan.info
        ctx.pt_import(ctx.L, i["pt_limbs"] > ctx.L + 1, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (i["n_pts"], ctx.N))), pt)
        plan.matmul(ct, pt, keys, dev_f64(plan.bytes("ct_out") // 8))
    one = dev_f64(2 * (level + 1) * ctx.N)
    ctx.encrypt_coeffs(sk, level, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 90, one)
    _capture_and_check(ctx, keys, level, one, gal[0], hoisted)
    t.cuda.synchronize()


def test_scratch_of_a_captured_rotation_stays():
    """decoding whose residues and slots fit the rotation's scratch (digits, ModUp, key products, ModDown and two
    ciphertexts) must not replace it"""
    ctx = context("C1")
    L1, a, N = ctx.L + 1, ctx.alpha, ctx.N
    K, beta = L1 + a, -(-L1 // a)
    room = beta * K + L1 + 2 * K + 2 * a + 4 * L1                # limbs
    nct = int(room // (L1 + 0.5))                                 # residues and half a limb of slots per ciphertext
    assert (room - 2 * L1) < nct * (L1 + 0.5) <= room             # more than the rotation alone
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_CTMAT, 1, 1, n_out=nct, pack=1)
    assert plan.info["ct_out"] == nct
    rng = np.random.default_rng(6)
    g = pow(5, 3, 2 * N)
    keys = ctx.rotkeys(sk, [g], 4)
    ct = dev_f64(2 * L1 * N)
    ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, N)), 8, ct)
    ctx.rotate(keys, ctx.L, ct, g, False, dev_f64(ct.numel()))
    outs = dev_f64(plan.bytes("ct_out") // 8)
    y = dev_f64(nct)
    _capture_and_check(ctx, keys, ctx.L, ct, g, False, between=lambda: plan.decrypt_decode(sk, outs, y))
