"""Rotations whose scratch grows while another stream is being captured: the
capture stays valid and both results are right.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


def test_conversion_beside_a_capture():
    t = torch()
    ctx, other = context("C2"), context("C2")
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_CTMAT, 64, 32, n_out=1, pack=ctx.N // 128)
    keys = ctx.rotkeys(sk, plan.transpose_galois(), 4)
    rng = np.random.default_rng(9)
    ct = dev_f64(plan.bytes("ct_in") // 8)
    Q2 = 2 * (ctx.L + 1) * ctx.N
    for c in range(plan.info["ct_in"]):
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8 + c, ct[c * Q2:(c + 1) * Q2])
    ctx.rotate(keys, ctx.L, ct[:Q2], plan.transpose_galois()[0], False, dev_f64(Q2))  # one rotation's scratch only
    got, want = dev_f64(ct.numel()), dev_f64(ct.numel())
    a, b = ct[:Q2], ct[Q2:2 * Q2]
    total, total_want = dev_f64(Q2), dev_f64(Q2)
    other.ct_add(other.L, a, b, total_want)
    side = t.cuda.Stream()
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph):
        other.ct_add(other.L, a, b, total)
        with t.cuda.stream(side):
            plan.transpose(ct, keys, got)
    plan.transpose(ct, keys, want)
    t.cuda.synchronize()
    assert t.equal(got, want)
    for _ in range(3):
        total.fill_(float("nan"))
        graph.replay()
        t.cuda.synchronize()
        assert t.equal(total, total_want)
