"""Complex UDT of matrices whose rows span hundreds of decades, so that what
remains of a column is far below its largest entry in every later step: D and U
against the oracle, which squares nothing unscaled.  Rows in falling order and
column pivoting make the factorization stable row by row: the bar 1e-8 is n eps
(1.4e-14) times the growth and condition of the scaled random part (1e3 .. 1e4
at n = 64), one order wider.  log|det| by n times that, relative to one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl
from _gpu import DEV, relF, say

pytestmark = pytest.mark.gpu


def graded(n, top, bottom):
    rng = np.random.default_rng(wl.BASE_SEED + 6400 + n)
    g = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    ex = np.linspace(top, bottom, n) if n > 1 else np.array([float(bottom)])
    return 10.0 ** ex[:, None] * g, np.linalg.slogdet(g)[1] + np.log(10.0) * ex.sum()


@pytest.mark.parametrize("top,bottom", [(0, -160), (0, -290), (150, -150)])
@pytest.mark.parametrize("n", [2, 5, 16, 17, 33, 48, 64])
def test_rows_over_hundreds_of_decades(n, top, bottom):
    W, ld = graded(n, top, bottom)
    say(f"[gpu] sdq_udt_complex n={n}, rows from 1e{top} to 1e{bottom}")
    u, d, t = (x[0].cpu().numpy() for x in sdq.context().udt_complex(torch.from_numpy(W[None]).to(DEV)))
    Uo, Do, To = oracle.udt_complex(W)
    assert np.all(np.abs(d / Do - 1.0) <= 1e-8)
    assert relF(u, Uo) <= 1e-8
    assert abs(np.log(d).sum() - ld) <= n * 1e-8
    back = (u * d) @ t
    assert np.all(np.linalg.norm(back - W, axis=0) <= 1e-12 * np.linalg.norm(W, axis=0))
