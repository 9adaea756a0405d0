"""The per-call lazy product's kernels where they branch: more digits than one
exact sum takes, few and many diagonals for a workgroup's waves, slices of the
diagonals, giant steps in more than one group, and outputs over the inputs.
Bit-exact against the oracle.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch
from test_gpu_parity import run_hybrid_both

pytestmark = pytest.mark.gpu


def _xy(m, n):
    g = np.random.default_rng(m * 31 + n)
    return g.uniform(-1, 1, (m, n)), g.uniform(-1, 1, n)


@pytest.mark.parametrize("name,m,n,bs", [
    ("C4a1", 9, 1000, 0),     # six digits: folded four and two
    ("C4a1", 33, 1000, 4),    # the same under giant steps
    ("C4a2", 17, 600, 0),     # three digits
    ("C1", 5, 2048, 0),       # m' = 8: fewer diagonals than waves
    ("C1", 130, 2048, 0),     # m' = 256: two slices of the diagonals
    ("C1", 128, 2048, 4),     # 32 giant steps of 4
    ("C1", 90, 300, 8),       # m' = 32: 4 giant steps, half a group
])
def test_bit_exact(name, m, n, bs):
    X, y = _xy(m, n)
    run_hybrid_both(name, X, y, True, bsgs=bs)


@pytest.mark.parametrize("m,n", [(64, 256), (4096, 64), (4096, 4096)])
def test_output_over_the_input(m, n):
    """one and two row blocks, one and two column blocks: the output may be the input's own buffer"""
    t = torch()
    ctx = context("C1")
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(2)
    size = max(plan.bytes("ct_in"), plan.bytes("ct_out")) // 8
    ct = dev_f64(size)
    Q2 = 2 * (ctx.L + 1) * ctx.N
    for c in range(plan.info["ct_in"]):
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8 + c, ct[c * Q2:(c + 1) * Q2])
    pt = dev_f64(plan.bytes("pt") // 8)
    coeffs = dev_i64(rng.integers(-2 ** 40, 2 ** 40, (8, ctx.N)))
    one = dev_f64(8 * 3 * ctx.N)
    ctx.pt_import(ctx.L, True, coeffs, one)
    reps = pt.numel() // one.numel()
    if reps:
        pt.copy_(one.repeat(reps + 1)[: pt.numel()])
    else:
        pt.copy_(one[: pt.numel()])
    want = dev_f64(plan.bytes("ct_out") // 8)
    plan.matmul(ct, pt, keys, want)
    plan.matmul(ct, pt, keys, ct)
    t.cuda.synchronize()
    assert t.equal(ct[: want.numel()], want)
