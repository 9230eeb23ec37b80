"""The one-kernel CG iteration of periodic grids against the oracle's textbook
CG: the iterate after a fixed number of iterations (odd and even counts: the
update of x lags by none or one), on grids at the edges of its tiles (60 x 2, 6
or 14 stored cells, cells that are their own neighbours) and with more blocks
than the launches sum directly."""
import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1311_7477_amd import dg as m
    return m


def iterate(dg, n, nx, ny, cw, k, w):
    import torch
    grid = dg.Grid(n, nx, ny)
    grid.set_tiles(cw, 8)
    psi = torch.zeros(grid.shape, dtype=torch.float64, device="cuda")
    res = dg.cg_solve_poisson(grid, torch.from_numpy(w).cuda(), psi, dg.Workspace(grid),
                              dg.cg_opts(rtol=1e-14, max_iter=k))
    return res, psi.cpu().numpy()


# The iterates of both sides are the same Krylov vectors, alpha and beta from
# the same sums up to rounding.  After k <= 7 iterations a relative error of
# about 1e-15 per operation (sums of one sign; the operator's entries spread
# by at most about 1e2 within a cell at n = 5) has passed k dependent scalars:
# k * 1e2 * 1e-15 < 1e-12, taken with a factor of 10.
@pytest.mark.parametrize("n,nx,ny,cw", [
    (1, 61, 5, 8), (2, 60, 6, 8), (2, 120, 7, 4), (3, 59, 13, 16), (3, 62, 3, 8), (3, 1, 9, 4),
    (4, 64, 1, 8), (4, 121, 12, 8), (4, 2, 2, 16), (5, 63, 8, 4), (5, 60, 15, 8),
    (1, 610, 96, 4),      # 11 x 48 blocks
])
@pytest.mark.parametrize("k", [1, 2, 7])
def test_iterate_matches_textbook_cg(dg, n, nx, ny, cw, k):
    print(f"cg step n={n} nx={nx} ny={ny} cw={cw} k={k}", flush=True)
    w = I.white_noise(n, nx, ny, seed=nx + ny)
    ref = O.cg_poisson(O.Grid2D(n, nx, ny), w, rtol=1e-14, max_iter=k)
    res, psi = iterate(dg, n, nx, ny, cw, k, w)
    assert res.iters == ref.iters
    assert np.max(np.abs(psi - ref.x)) <= 1e-11 * np.max(np.abs(ref.x))
