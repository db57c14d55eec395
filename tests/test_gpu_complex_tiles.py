"""The complex kernels at the edges of their tiles: one variant for each 16
rows (n = 1 .. 64), a chain of each size and a batch that mixes them, against
the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl
from _gpu import DEV, relF, say

pytestmark = pytest.mark.gpu

SIZES = (1, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64)


@pytest.fixture(scope="module")
def ctx():
    return sdq.Context(0)


def cnormal(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def slices(n, m):
    """1 + a small dense part: chains of a condition that the oracle's own
    rounding resolves."""
    rng = np.random.default_rng(wl.BASE_SEED + 6100 + n)
    return np.eye(n) + 0.1 / np.sqrt(n) * cnormal(rng, m, n, n)


@pytest.mark.parametrize("n", SIZES)
def test_udt_at_tile_edges(ctx, n):
    """U and D of a graded matrix, columns over 20 decades; U D T = W."""
    rng = np.random.default_rng(wl.BASE_SEED + 6000 + n)
    W = cnormal(rng, 2, n, n) * 10.0 ** rng.uniform(-10, 10, (2, 1, n))
    say(f"[gpu] sdq_udt_complex n={n}, graded")
    u, d, t = (x.cpu().numpy() for x in ctx.udt_complex(torch.from_numpy(W).to(DEV)))
    for b in range(2):
        Uo, Do, To = oracle.udt_complex(W[b])
        assert relF(u[b], Uo) <= 1e-10 and np.allclose(d[b], Do, rtol=1e-10, atol=0)
        back = (u[b] * d[b]) @ t[b]
        assert np.all(np.linalg.norm(back - W[b], axis=0) <= 1e-12 * np.linalg.norm(W[b], axis=0))


@pytest.mark.parametrize("sizes", [(n,) for n in SIZES] + [SIZES])
def test_chain_at_tile_edges(ctx, sizes):
    say(f"[gpu] sdq_greens_complex n={sizes}")
    sls = [slices(n, 9) for n in sizes]
    gs, ld, ph, st = ctx.greens_complex([torch.from_numpy(s).to(DEV) for s in sls], [4] * len(sls))
    assert st.cpu().tolist() == [0] * len(sls)
    for i, s in enumerate(sls):
        G, ldo, pho = oracle.greens_complex(s, 4)
        assert relF(gs[i].cpu().numpy(), G) <= 1e-10
        assert abs(ld[i].item() - ldo) <= 1e-12 * max(1.0, abs(ldo))
        assert abs(ph[i].item() - pho) <= 1e-10
