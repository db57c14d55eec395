"""A gang (n > 144) takes many stage pairs and many equal-time inversions in a
row out of one scratch area: what it computes for each equals, bit for bit,
what a gang computes that has nothing else to do, and no member waits for ever."""
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


# 128, 42, 19 and 4 gangs on the 256 compute units: several items for each
@pytest.mark.parametrize("n,m,k,count", [(160, 24, 2, 40), (272, 24, 2, 16), (400, 24, 3, 10), (1000, 4, 2, 10)])
def test_items_of_a_gang(ctx, n, m, k, count):
    E, Ei = wl.expk_pair(wl.chain_hopping_matrix(n), 0.1)
    rng = np.random.default_rng(wl.BASE_SEED + 8000 + n)
    f = 2.0 * rng.integers(0, 2, (count, m, n)) - 1.0
    e, ei = torch.from_numpy(E).to(DEV), torch.from_numpy(Ei).to(DEV)
    lam = wl.hirsch_lambda(4.0, 0.1)
    ch = [sdq.Chain(e, torch.from_numpy(x).to(DEV), lam, k, ei) for x in f]
    ls = list(range(k, m, k))
    say(f"[gpu] gang items: n = {n}, {count} chains, {len(ls)} pairs each")
    gts, gs, ld, sg, st = ctx.greens_tdisp(ch, ls)
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all()
    for i in range(0, count, 3):
        say(f"[gpu] chain {i} alone")
        for q, l in enumerate(ls):
            gt1, g1, ld1, sg1, st1 = ctx.greens_tdisp([ch[i]], [l])
            assert torch.equal(gt1[0][0], gts[i][q]), (i, l)
        assert torch.equal(g1[0], gs[i]) and ld1.item() == ld[i].item() and sg1.item() == sg[i].item()
        assert st1.item() == 0
