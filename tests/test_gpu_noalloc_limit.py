"""sdq_greens_noalloc near the end of its fixed scratch: batches that leave no
room for the blocked QR's copies of a block's columns (150 chains of n = 128,
800 of n = 64) run with the pivoted sweeps and are not refused."""
import numpy as np
import pytest
import torch

from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl
from _gpu import DEV, relF, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count", [(128, 100), (128, 150), (64, 800)])
def test_batches_that_fill_the_scratch(n, count):
    m, k = 4, 2
    E, Ei = wl.expk_pair(wl.chain_hopping_matrix(n), 0.1)
    rng = np.random.default_rng(wl.BASE_SEED + 9700 + n)
    f = 2.0 * rng.integers(0, 2, (count, m, n)) - 1.0
    e, ei, fd = (torch.from_numpy(x).to(DEV) for x in (E, Ei, f))
    ch = [sdq.Chain(e, x, wl.hirsch_lambda(4.0, 0.1), k, ei) for x in fd]
    ctx = sdq.Context(0)
    ref, ld0, sg0, st0 = ctx.greens(ch)
    gs = [torch.full((n, n), float("nan"), dtype=torch.float64, device=DEV) for _ in ch]
    ld, sg = (torch.zeros(count, dtype=torch.float64, device=DEV) for _ in range(2))
    st = torch.full((count,), 7, dtype=torch.int32, device=DEV)
    say(f"[gpu] sdq_greens_noalloc: {count} chains of n = {n}")
    ctx.greens_noalloc(ch, gs, ld, sg, st)
    torch.cuda.synchronize()
    assert (st.cpu() == 0).all() and (st0.cpu() == 0).all() and torch.equal(sg, sg0)
    assert torch.allclose(ld, ld0, rtol=1e-12, atol=1e-12)
    assert max(relF(a.cpu().numpy(), b.cpu().numpy()) for a, b in zip(gs, ref)) <= 1e-10
    ctx.close()
