"""Complex UDT of columns that lose most of their norm in many steps, so that
remaining norms are recomputed again and again (by every wave, from partial sums
that the waves exchange), with as many workgroups on a compute unit as fit:
U D T = W and U^H U = 1 to 1e-12 (n <= 64 times eps, two orders), |diag R|
not increasing beyond rounding, and every copy of a matrix factored to the same bits."""
import numpy as np
import pytest
import torch

from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl
from _gpu import DEV, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return sdq.Context(0)


@pytest.mark.parametrize("n", [3, 7, 15, 16, 17, 24, 32, 33, 47, 48, 49, 63, 64])
def test_norms_recomputed(ctx, n):
    rng = np.random.default_rng(wl.BASE_SEED + 6300 + n)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    W = np.zeros((4, n, n), dtype=complex)
    for b in range(4):  # ranks added at falling sizes: 1e-3, 1e-5, .. of the first
        r = max(1, n // (2 * (b + 1)))
        for lvl in range(0, n, r):
            W[b] += 10.0 ** (-(2 + b) * (lvl // r)) * cn(n, min(r, n - lvl)) @ cn(min(r, n - lvl), n)
    say(f"[gpu] sdq_udt_complex n={n}, falling norms")
    count = 2048
    u, d, t = ctx.udt_complex(torch.from_numpy(W).to(DEV).repeat(count // 4, 1, 1))
    for x in (u, d, t):
        y = x.reshape(count // 4, 4, *x.shape[1:])
        assert torch.equal(y, y[:1].expand_as(y))
    u, d, t = (x[:4].cpu().numpy() for x in (u, d, t))
    for b in range(4):
        back = (u[b] * d[b]) @ t[b]
        assert np.all(np.linalg.norm(back - W[b], axis=0) <= 1e-12 * np.linalg.norm(W[b], axis=0))
        assert np.linalg.norm(u[b].conj().T @ u[b] - np.eye(n)) <= 1e-12 * np.sqrt(n)
        assert np.all(d[b][1:] <= d[b][:-1] * (1 + 1e-6))
