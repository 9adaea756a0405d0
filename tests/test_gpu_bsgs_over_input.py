"""Giant-step products whose output lies over their input, whole or in part:
two row blocks (the second reads the inputs after the first is written) and
two column blocks (the second input is read after the first one's sums are).
Bit equality with the product into a buffer of its own.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, dev_i64, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,bs,shift", [
    (64, 256, 4, 0),       # one row block, one column block
    (4096, 64, 8, 0),      # two row blocks
    (64, 4096, 4, 0),      # two column blocks, the output over the first input
    (64, 4096, 4, 1),      # ... over the second
    (4096, 4096, 32, 0),   # two of each
    (4096, 4096, 32, 1),   # ... the outputs from the second input on
])
def test_output_over_the_input(m, n, bs, shift):
    t = torch()
    ctx = context("C1")
    sk = ctx.keygen(3)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True, bsgs=bs)
    keys = ctx.rotkeys(sk, plan.galois(), 4)
    rng = np.random.default_rng(2)
    Q2 = 2 * (ctx.L + 1) * ctx.N
    n_in, n_out = plan.bytes("ct_in") // 8, plan.bytes("ct_out") // 8
    buf = dev_f64(max(n_in, shift * Q2 + n_out))
    ct = buf[:n_in]
    for c in range(plan.info["ct_in"]):
        ctx.encrypt_coeffs(sk, ctx.L, dev_i64(rng.integers(-2 ** 40, 2 ** 40, ctx.N)), 8 + c, ct[c * Q2:(c + 1) * Q2])
    one = dev_f64(8 * 3 * ctx.N)
    ctx.pt_import(ctx.L, True, dev_i64(rng.integers(-2 ** 40, 2 ** 40, (8, ctx.N))), one)
    n_pt = plan.bytes("pt") // 8
    pt = one.repeat(-(-n_pt // one.numel()))[:n_pt].contiguous()
    want = dev_f64(n_out)
    plan.matmul(ct, pt, keys, want)
    got = buf[shift * Q2: shift * Q2 + n_out]
    plan.matmul(ct, pt, keys, got)
    t.cuda.synchronize()
    assert t.equal(got, want)
