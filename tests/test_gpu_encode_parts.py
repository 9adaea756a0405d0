"""Plaintexts whose limbs several workgroups share (few plaintexts) against the
batched encoder, which always gives a plaintext one workgroup: the same
residues bit for bit, for every number of parts that limb counts allow.  Needs
an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, dev_f64, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,m,n", [
    ("C1", 16, 256), ("C1", 700, 2048),                # 2 plaintexts in 3 parts; 1024 in one
    ("C2", 256, 1024), ("C2", 500, 2048),              # 64 in 4, 256 in 2
    ("C3", 2, 5), ("C3", 300, 2048), ("C3", 300, 4096),  # 1 in 5, 128 in 2, 256 in 1
    ("C4", 60, 4096), ("C4a2", 30, 2000),              # 32 of 9 limbs, 8 of 8
    ("C5", 4, 100), ("C5", 120, 4096), ("C5", 300, 4096)])  # 1 of 10 limbs, 32, 128
def test_shared_limbs(name, m, n):
    t = torch()
    ctx = context(name)
    plan = ctx.plan(pvfl.PLAN_HYBRID, m, n, lazy=True)
    g = np.random.default_rng(m + n)
    X = t.from_numpy(g.standard_normal((m, n))).cuda()
    got, want = (dev_f64(plan.bytes("pt") // 8).fill_(float("nan")) for _ in range(2))
    plan.encode_pt(X, got)
    keys = None if plan.info["mprime"] == 1 else ctx.rotkeys(ctx.keygen(1), plan.galois(), 2)
    b = pvfl.Batch(ctx, [plan], X=[X], pt=[want], ct=[dev_f64(plan.bytes("ct_in") // 8)],
                   out=[dev_f64(plan.bytes("ct_out") // 8)], keys=keys)
    b.encode()
    t.cuda.synchronize()
    assert t.equal(got, want) and bool(t.isfinite(got).all())
