"""Values at the ends of the range in the blocked QR: middle matrices that are
exactly zero (log|det(1 + B)| = -inf, range status, the batch's other chains as
ever) or far from one in size (columns whose squares underflow).  Bar where the
oracle has a result: the suite's relative 1e-10."""
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


@pytest.mark.parametrize("n", [1, 5, 16, 40, 64, 81, 100, 128, 140, 150, 260, 520])
def test_singular(ctx, n):
    """B = -1 beside B = 1 / 2 (E = -1 and 1 / 2, a field of zeros)."""
    f = torch.zeros(1, n, dtype=torch.float64, device=DEV)
    es = [s * torch.eye(n, dtype=torch.float64, device=DEV) for s in (-1.0, 0.5)]
    ch = [sdq.Chain(e, f, 1.0, 1) for e in es]
    say(f"[gpu] singular 1 + B: n = {n}")
    gs, ld, sg, st = ctx.greens(ch)
    torch.cuda.synchronize()
    assert ld[0].item() == -np.inf and abs(sg[0].item()) == 1.0 and st[0].item() != 0
    assert relF(gs[1].cpu().numpy(), np.eye(n) / 1.5) <= 1e-14
    assert abs(ld[1].item() - n * np.log(1.5)) <= 1e-14 * n and sg[1].item() == 1.0 and st[1].item() == 0
    if n <= 128:
        gs, ld, sg, st = ctx.greens_dense([e[None].clone() for e in es], 1)
        assert ld[0].item() == -np.inf and st[0].item() != 0 and st[1].item() == 0
        assert relF(gs[1].cpu().numpy(), np.eye(n) / 1.5) <= 1e-14
    if n <= 64:
        gs, ld, ph, st = ctx.greens_complex([e[None].to(torch.complex128) for e in es], 1)
        assert ld[0].item() == -np.inf and st[0].item() != 0 and st[1].item() == 0
        assert relF(gs[1].cpu().numpy(), np.eye(n) / 1.5) <= 1e-14


@pytest.mark.parametrize("n", [9, 16, 33, 64, 81, 100, 128, 140, 150, 260])
@pytest.mark.parametrize("shift", [23.0, -23.0])
def test_scaled_middle_matrices(ctx, n, shift):
    """Slices times exp(23) = 1e10 in one half of the chain and over it in the
    other: B(tau,0) is of the size 1e180 or 1e-180 in the middle, the middle
    matrix of G(tau,0) of the size 1e-180 either way."""
    m, k = 36, 3
    E, Ei = wl.expk_pair(wl.chain_hopping_matrix(n), 0.1)
    rng = np.random.default_rng(wl.BASE_SEED + 9000 + n)
    f = 0.3 * rng.standard_normal((m, n))
    f[: m // 2] += shift
    f[m // 2 :] -= shift
    ls = [3, 17, 18, 20, 33]
    say(f"[gpu] scaled slices: n = {n}, shift {shift}")
    gts, gs, ld, sg, st = ctx.greens_tdisp([sdq.Chain(torch.from_numpy(E).to(DEV), torch.from_numpy(f).to(DEV), 1.0, k,
                                                      torch.from_numpy(Ei).to(DEV))], ls)
    torch.cuda.synchronize()
    assert st.item() == 0
    G, ldo, sgo = oracle.greens(E, f, 1.0, k)
    refs = [oracle.greens_tdisp(E, Ei, f, 1.0, k, l) for l in ls]
    got = [(gs, ld, sg, gts[0])]
    if n <= 128:
        b = E[None] * np.exp(f)[:, None, :]
        g2, gd, ld2, sg2, st2 = ctx.greens_tdisp_dense([torch.from_numpy(b).to(DEV)], k, ls)
        assert st2.item() == 0
        got.append((gd, ld2, sg2, g2[0]))
    for g, l1, s1, gt in got:
        assert relF(g[0].cpu().numpy(), G) <= 1e-10
        assert abs(l1.item() - ldo) <= 1e-12 * max(1.0, abs(ldo)) and s1.item() == sgo
        for q, ref in enumerate(refs):
            top = np.abs(ref).max()
            assert relF(gt[q].cpu().numpy() / top, ref / top) <= 1e-10, ls[q]
