"""Blocks in the middle of a chain whose columns are nearly dependent, so that the
norm-sorted QR repeats its sort or gives up and pivots: a model of the
acceptance rule on the CPU picks such chains (fields that suppress some of the
sites of one slice of an orthogonal chain, E scaled to 0.8), forward and backward,
and they run beside one ordinary chain each.  Every slice is a contraction
and 1 + B has condition below 2, so the reference is the plain product, and the bar
1e-12 (n <= 272 times eps, an order and more).
T in registers (n <= 80), in scratch (<= 128), R's upper tiles too (<= 144), gangs above."""
import numpy as np
import pytest
import torch

from paper_2003_05286_amd import binding as sdq
from _gpu import DEV, relF, say

pytestmark = pytest.mark.gpu

M, K, AT = 6, 2, 2  # slices, block length, the suppressing slice (block 1 of 0 .. 2 both ways)
PASSES = 6


def passes(w, bound):
    """(factorizations, accepted, the smallest margin by which one failed) of a
    block's columns w by the sorted QR's rule."""
    key, margin = np.linalg.norm(w, axis=0), np.inf
    for p in range(PASSES):
        w = w[:, np.argsort(-key, kind="stable")]
        r = np.abs(np.linalg.qr(w, mode="r"))
        d = np.diag(r)
        grown = np.triu(r, 1) > bound * d[:, None]
        if not grown.any():
            return p + 1, True, margin
        margin = min(margin, (np.triu(r, 1) / (bound * d[:, None])).max())
        key = np.maximum(d, np.where(grown, r, 0.0).max(0))
    return PASSES, False, margin


def chain(n, seed):
    rng = np.random.default_rng(seed)
    E = 0.8 * np.linalg.qr(rng.normal(size=(n, n)))[0]
    f = np.zeros((M, n))
    f[AT, rng.permutation(n)[: rng.integers(n // 4, 7 * n // 8)]] = np.log(rng.choice([1e-3, 1e-6, 1e-9]))
    return E, f


def outcomes(n, E, f, bound):
    v, q = np.exp(f[AT]), E / 0.8
    fw = q @ (q @ (v[:, None] * (q @ q)))  # the orthogonal blocks beside it only permute and flip columns
    bw = v[:, None] * (q.T @ q.T @ q.T @ q.T)
    return passes(fw, bound), passes(bw, bound)


def pick(n, bound):
    """Chains whose block repeats the sort at least twice, and that give up, each
    way, by a margin that rounding does not decide."""
    repeat, gave_up = [set(), set()], [set(), set()]
    for seed in range(600):
        for way, (p, ok, margin) in enumerate(outcomes(n, *chain(n, seed), bound)):
            if ok and p >= 3 and len(repeat[way]) < 2:
                repeat[way].add(seed)
            if not ok and margin > 1.05 and len(gave_up[way]) < 2:
                gave_up[way].add(seed)
        if all(repeat) and all(gave_up):
            break
    return repeat, gave_up


@pytest.mark.parametrize("n", [20, 36, 48, 64, 80, 96, 128, 140, 160, 272])
def test_repeated_and_given_up(n):
    repeat, gave_up = pick(n, 2.0 if n <= 144 else 4.0)
    assert all(repeat) and (all(gave_up) or n < 64), "the model takes every branch (small blocks never give up)"
    seeds = sorted(set().union(*repeat, *gave_up))
    say(f"[gpu] n = {n}: chains {seeds}, given up {gave_up}")
    data = [chain(n, s) for s in seeds]
    rng = np.random.default_rng(n)
    data += [(E, 0.1 * rng.standard_normal((M, n))) for E, _ in data]  # ordinary ones among them
    ch = [sdq.Chain(torch.from_numpy(E).to(DEV), torch.from_numpy(f).to(DEV), 1.0, K,
                    torch.from_numpy(np.ascontiguousarray(E.T / 0.64)).to(DEV)) for E, f in data]
    ls = [2, 3, 4, 5]
    ctx = sdq.Context(0)
    gts, gs, ld, sg, st = ctx.greens_tdisp(ch, ls)
    g2, ld2, sg2, st2 = ctx.greens(ch)
    got = [(gs, gts, ld, sg), (g2, None, ld2, sg2)]
    assert (st.cpu().numpy() == 0).all() and (st2.cpu().numpy() == 0).all()
    if n <= 128:
        sl = [torch.from_numpy(E[None] * np.exp(f)[:, None, :]).to(DEV) for E, f in data]
        gds, gd, ld3, sg3, st3 = ctx.greens_tdisp_dense(sl, K, ls)
        assert (st3.cpu().numpy() == 0).all()
        got.append((gd, gds, ld3, sg3))
    torch.cuda.synchronize()
    for i, (E, f) in enumerate(data):
        prod = [np.eye(n)]
        for x in f:
            prod.append(E @ (np.exp(x)[:, None] * prod[-1]))
        G = np.linalg.inv(np.eye(n) + prod[M])
        sgo, ldo = np.linalg.slogdet(np.eye(n) + prod[M])
        for g, gt, l1, s1 in got:
            errs = [relF(g[i].cpu().numpy(), G)]
            if gt is not None:
                errs += [relF(gt[i][q].cpu().numpy(), prod[l] @ G) for q, l in enumerate(ls)]
            assert max(errs) <= 1e-12, (i, errs)
            assert abs(l1[i].item() - ldo) <= 1e-12 * max(1.0, abs(ldo)) and s1[i].item() == sgo
