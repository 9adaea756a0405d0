"""The ciphertext-matrix and column-order products where the split of their
work changes: every number of outputs that a workgroup holds, one to eight
waves, one ciphertext, ciphertexts that the waves do not share evenly.  Exact
integer sums at sampled places.  Needs an MI355X."""
import pytest

from paper_2405_00482_amd import pvfl

from gpu_util import context, torch

pytestmark = pytest.mark.gpu


def _check(ctx, plan):
    t = torch()
    i = plan.info
    L1, N, nct, nout = ctx.L + 1, ctx.N, i["ct_in"], i["ct_out"]
    g = t.Generator(device="cuda").manual_seed(nct + nout)
    q = t.tensor([float(x) for x in ctx.q], dtype=t.float64, device="cuda")[:, None]

    def residues(*shape):
        r = t.floor((t.rand(*shape, L1, N, generator=g, dtype=t.float64, device="cuda") * 2 - 1) * q)
        r[..., : N // 4] = q - 1
        r[..., N // 4: N // 2] = 2 - q
        return r
    ct, pt = residues(nct, 2), residues(nct, nout)
    out = t.full((nout, 2, L1, N), float("nan"), dtype=t.float64, device="cuda")
    plan.matmul(ct.view(-1), pt.view(-1), None, out.view(-1))
    idx = [0, 63, 64, 255, 256, N // 4, N // 2, N // 2 + 1, N - 1]
    c, p, o = (x[..., idx].cpu().numpy().astype(object) for x in (ct, pt, out))
    for l, prime in enumerate(ctx.q):
        for k in range(nout):
            for h in range(2):
                for s in range(len(idx)):
                    want = sum(int(c[a, h, l, s]) * int(p[a, k, l, s]) for a in range(nct)) % prime
                    got = int(o[k, h, l, s])
                    assert got % prime == want and 2 * abs(got) <= prime + 1
    assert not t.isnan(out).any()


@pytest.mark.parametrize("n_out", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 17])
@pytest.mark.parametrize("name,m,n", [("C1", 1, 4), ("C1", 2, 2), ("C1", 64, 32), ("C2", 16, 16), ("C4", 8, 4)])
def test_matrix(name, m, n, n_out):
    ctx = context(name)
    _check(ctx, ctx.plan(pvfl.PLAN_CTMAT, m, n, n_out=n_out, pack=1))


@pytest.mark.parametrize("name,n", [("C1", 1), ("C1", 3), ("C1", 17), ("C1", 67), ("C5", 5)])
@pytest.mark.parametrize("blocks", [1, 2])
def test_columns(name, n, blocks):
    ctx = context(name)
    plan = ctx.plan(pvfl.PLAN_COL, blocks * ctx.N // 2, n)
    assert plan.info["ct_in"] == n and plan.info["ct_out"] == blocks
    _check(ctx, plan)
