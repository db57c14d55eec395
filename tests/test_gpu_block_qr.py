"""The stabilized sweeps' norm-sorted blocked QR at the sizes where it can go
wrong: one tile to eight and the gangs above, full and ragged, last blocks shorter than k, against the oracle's column-pivoted chains; and
blocks whose columns are nearly dependent, where the order by norm is not
good enough and the sort is repeated or the pivoted QR takes over.  Bar: the
suite's relative 1e-10 per matrix; where B is scaled to norm 1/2, 1 + B has
condition at most 3 and the bar is 1e-12 (n <= 128 times eps, two orders)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl
from _gpu import DEV, relF, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return sdq.Context(0)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 65, 79, 80, 81, 95, 97, 112, 113, 127, 128])
def test_sizes(ctx, n):
    m, k = 23, 5
    E, Ei = wl.expk_pair(wl.chain_hopping_matrix(n) if n > 2 else -np.ones((n, n)) + np.eye(n), 0.1)
    rng = np.random.default_rng(wl.BASE_SEED + n)
    f = 2.0 * rng.integers(0, 2, (m, n)) - 1.0
    lam = wl.hirsch_lambda(4.0, 0.1)
    ch = [sdq.Chain(torch.from_numpy(E).to(DEV), torch.from_numpy(f).to(DEV), a, k, torch.from_numpy(Ei).to(DEV))
          for a in (lam, -lam)]
    ls = [0, 3, 5, 20, 22, 23]
    say(f"[gpu] sizes: n = {n}")
    gts, gs, ld, sg, st = ctx.greens_tdisp(ch, ls)
    g2, ld2, sg2, st2 = ctx.greens(ch)
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all() and (st2.cpu().numpy() == 0).all()
    for i, a in enumerate((lam, -lam)):
        G, ldo, sgo = oracle.greens(E, f, a, k)
        for g, l, s in ((gs, ld, sg), (g2, ld2, sg2)):
            assert relF(g[i].cpu().numpy(), G) <= 1e-10
            assert abs(l[i].item() - ldo) <= 1e-12 * max(1.0, abs(ldo)) and s[i].item() == sgo
        for q, l in enumerate(ls):
            assert relF(gts[i][q].cpu().numpy(), oracle.greens_tdisp(E, Ei, f, a, k, l)) <= 1e-10, l


@pytest.mark.parametrize("n", [130, 145, 160, 161, 177, 241, 257, 272, 321, 336, 400])
def test_gang_sizes(ctx, n):
    """Chains over several workgroups: every split of a panel's rows and of a
    column slab into tiles, ragged sizes; the second call reuses the scratch."""
    m, k = 8, 3
    E, Ei = wl.expk_pair(wl.chain_hopping_matrix(n), 0.1)
    rng = np.random.default_rng(wl.BASE_SEED + n)
    f = 2.0 * rng.integers(0, 2, (m, n)) - 1.0
    lam = wl.hirsch_lambda(4.0, 0.1)
    ch = [sdq.Chain(torch.from_numpy(E).to(DEV), torch.from_numpy(f).to(DEV), lam, k, torch.from_numpy(Ei).to(DEV))]
    say(f"[gpu] gang sizes: n = {n}")
    gts, gs, ld, sg, st = ctx.greens_tdisp(ch, [2, 6])
    g2, ld2, sg2, st2 = ctx.greens(ch)
    grads, ld3, sg3, st3 = ctx.logdet_grad(ch)
    torch.cuda.synchronize()
    assert st.item() == 0 and st2.item() == 0 and st3.item() == 0
    G, ldo, sgo = oracle.greens(E, f, lam, k)
    for g, l, s in ((gs[0], ld, sg), (g2[0], ld2, sg2), (None, ld3, sg3)):
        if g is not None:
            assert relF(g.cpu().numpy(), G) <= 1e-10
        assert abs(l.item() - ldo) <= 1e-12 * max(1.0, abs(ldo)) and s.item() == sgo
    for q, l in enumerate((2, 6)):
        assert relF(gts[0][q].cpu().numpy(), oracle.greens_tdisp(E, Ei, f, lam, k, l)) <= 1e-10, l
    assert relF(grads[0][3].cpu().numpy(), oracle.logdet_grad(E, f, lam, k, [4])[0]) <= 1e-10


@pytest.mark.parametrize("n,noise", [(36, 1e-3), (64, 1e-3), (64, 1e-6), (64, 1e-9), (100, 1e-6), (128, 1e-3)])
def test_nearly_dependent_columns(ctx, n, noise):
    m, k = 6, 2
    slices = []
    for seed in range(12):
        rng = np.random.default_rng(seed)
        w = rng.normal(size=(n, n // 2)) @ rng.normal(size=(n // 2, n)) + noise * rng.normal(size=(n, n))
        b = np.stack([w] + [np.linalg.qr(rng.normal(size=(n, n)))[0] for _ in range(m - 1)])
        b[0] *= 0.5 / np.linalg.norm(w, 2)
        slices.append(b)
    say(f"[gpu] nearly dependent columns: n = {n}, noise {noise}")
    gs, ld, sg, st = ctx.greens_dense([torch.from_numpy(b).to(DEV) for b in slices], k)
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all()
    for i, b in enumerate(slices):
        G, ldo, sgo = oracle.greens_dense(b, k)
        assert relF(gs[i].cpu().numpy(), G) <= 1e-12
        assert abs(ld[i].item() - ldo) <= 1e-12 * max(1.0, abs(ldo)) and sg[i].item() == sgo
