"""The ciphertext-matrix product over every count of outputs and ciphertexts
that its workgroups treat apart, at residues up to the ends of their range,
against exact integer sums at sampled places.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["C1", "C4"])
@pytest.mark.parametrize("m,n,n_out", [(1, 1, 1), (2, 4, 2), (3, 9, 3), (16, 8, 4), (8, 16, 5), (64, 128, 8), (32, 16, 9), (128, 128, 17)])
def test_sums_of_products(name, m, n, n_out):
    t = torch()
    ctx = context(name)
    plan = ctx.plan(pvfl.PLAN_CTMAT, m, n, n_out=n_out, pack=1)
    i = plan.info
    L1, N, nct, nout = ctx.L + 1, ctx.N, i["ct_in"], i["ct_out"]
    g = t.Generator(device="cuda").manual_seed(m + n)
    q = t.tensor([float(x) for x in ctx.q], dtype=t.float64, device="cuda")[:, None]

    def residues(*shape):
        r = t.floor((t.rand(*shape, L1, N, generator=g, dtype=t.float64, device="cuda") * 2 - 1) * q)
        r[..., : N // 4] = q               # the largest a caller may pass
        r[..., N // 4: N // 2] = -q
        return r
    ct, pt = residues(nct, 2), residues(nct, nout)
    out = t.full((nout, 2, L1, N), float("nan"), dtype=t.float64, device="cuda")
    plan.matmul(ct.view(-1), pt.view(-1), None, out.view(-1))
    idx = [0, 63, 64, N // 4 - 1, N // 4, N // 2, N // 2 + 1, N - 1]
    c, p, o = (x[..., idx].cpu().numpy().astype(object) for x in (ct, pt, out))
    for l, prime in enumerate(ctx.q):
        for k in range(nout):
            for h in range(2):
                for s in range(len(idx)):
                    want = sum(int(c[a, h, l, s]) * int(p[a, k, l, s]) for a in range(nct)) % prime
                    got = int(o[k, h, l, s])
                    assert got % prime == want and 2 * abs(got) <= prime + 1
