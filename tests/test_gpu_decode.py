"""Decode and read-out against an independent CRT lift and transform, for limb
counts with and without a register-resident variant and every plan kind's
read-out.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl
from paper_2405_00482_amd import workloads as W

from gpu_util import dev_f64, torch

pytestmark = pytest.mark.gpu


def _primes(logN, count):
    """NTT-friendly primes below 2^40 (probable primes; the context checks them)"""
    out, step = [], 2 << logN
    x = (1 << 40) // step * step + 1
    while len(out) < count:
        if all(x % p for p in (3, 5, 7, 11, 13)) and pow(2, x - 1, x) == 1 and pow(3, x - 1, x) == 1:
            out.append(x)
        x -= step
    return out


@pytest.mark.parametrize("logN,limbs", [(12, 1), (12, 7), (12, 9), (13, 8), (14, 7), (15, 2), (15, 8), (15, 9)])
def test_every_limb_count(logN, limbs):
    """a plan with one diagonal: y = x * r through encrypt, product and decode;
    the precision is the encoding's, 2^-30 of the largest value or better with scale 2^30 per operand
    (fresh noise below 2^14 of coefficients against 2^60)"""
    t = torch()
    pr = _primes(logN, limbs + 1)
    scale = 18.0 if limbs == 1 else 30.0            # one 40-bit limb holds a 2^36 product
    ctx = pvfl.Context(logN, pr[:limbs], pr[limbs:], scale)
    sk = ctx.keygen(5)
    plan = ctx.plan(pvfl.PLAN_HYBRID, 1, 8, lazy=True) if limbs > 1 else ctx.plan(pvfl.PLAN_HYBRID, 1, 1, lazy=True)
    n = plan.info["n"]
    g = np.random.default_rng(limbs)
    x, r = g.uniform(-1, 1, (1, n)), g.uniform(-1, 1, n)
    keys = ctx.rotkeys(sk, plan.galois(), 6)
    pt, ct, out, y = (dev_f64(plan.bytes(w) // 8) for w in ("pt", "ct_in", "ct_out", "pt"))
    y = dev_f64(1)
    plan.encode_pt(t.from_numpy(x).cuda(), pt)
    plan.encrypt(sk, t.from_numpy(r).cuda(), 7, ct)
    plan.matmul(ct, pt, keys, out)
    plan.decrypt_decode(sk, out, y)
    # noise: CBD(21) errors (sigma 3.3) and roundings of N coefficients, sqrt(N) < 2^8, over the scale; times n terms
    tol = n * 2.0 ** (8 + 4 + 3 - scale)
    assert abs(float(y.item()) - float((x @ r)[0])) < tol


@pytest.mark.parametrize("kind,m,n,n_out,pack,ras", [
    ("HYBRID", 5, 8, 0, 1, False), ("HYBRID", 300, 2048, 0, 1, False), ("HYBRID", 5000, 3, 0, 1, False),
    ("DIAG", 6, 100, 0, 1, False), ("DIAG", 6, 100, 0, 1, True), ("DIAG", 100, 6, 0, 1, False),
    ("CTMAT", 10, 40, 7, 3, False), ("CTMAT", 40, 10, 5, 2, False), ("COL", 5000, 2, 0, 1, False), ("ROW", 4, 10, 0, 1, False)])
def test_read_out_of_every_plan(kind, m, n, n_out, pack, ras):
    """the fused read-out against the slot-by-slot one (pvfl_lazy_ras) on the same decoded slots, bit for bit"""
    t = torch()
    ctx = pvfl.Context.from_dict(W.params_dict("C3"), device=0)
    sk = ctx.keygen(5)
    plan = ctx.plan(getattr(pvfl, "PLAN_" + kind), m, n, n_out=n_out, pack=pack, ras_in_ct=ras)
    i = plan.info
    lv, N = i["out_level"], ctx.N
    ct = t.zeros(i["ct_out"], 2, lv + 1, N, dtype=t.float64, device="cuda")
    one = t.zeros(2 * (lv + 1) * N, dtype=t.float64, device="cuda")
    g = t.Generator(device="cuda").manual_seed(3)
    for c in range(i["ct_out"]):
        msg = t.randint(-2 ** 30, 2 ** 30, (N,), dtype=t.int64, device="cuda", generator=g)
        ctx.encrypt_coeffs(sk, lv, msg, 40 + c, one)
        ct[c] = one.view(2, lv + 1, N)
    count = m * n_out if kind == "CTMAT" else m
    y, y2 = dev_f64(count), dev_f64(count)
    plan.decrypt_decode(sk, ct.view(-1), y)
    # the slots themselves: a plan of the same level and scale whose outputs are all the slots of one ciphertext
    slots = t.zeros(i["ct_out"], N // 2, dtype=t.float64, device="cuda")
    flat = ctx.plan(pvfl.PLAN_COL, N // 2, 1, level=lv, pt_log2_scale=i["out_log2_scale"] - ctx.log2_scale)
    for c in range(i["ct_out"]):
        o = dev_f64(N // 2)
        flat.decrypt_decode(sk, ct[c].contiguous().view(-1), o)
        slots[c] = o
    plan.lazy_ras(slots.view(-1), y2)
    assert t.equal(y, y2)
