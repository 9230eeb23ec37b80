"""The matrix products of the fast-diagonalisation inverse, at the edges of the
product kernel's 32 x 32 tiles and 64-long chunks, with an empty half, on long
thin grids and on both sides of the sizes where rocBLAS takes over, in FP64 and
as the FP32 preconditioner of a mixed solve, against the oracle."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# halves of (N + 1) / 2 and (N - 1) / 2 cells: 1/0, 2/1, 16/15, 17/16, 32/31,
# 33/32, 64/63, 65/64; n^2 nx ny max(nx, ny) operations below and above 6e8
PERIODIC = [(2, 1, 33), (3, 31, 1), (5, 3, 31), (4, 33, 63), (3, 63, 65), (2, 65, 127),
            (4, 127, 33), (2, 129, 131), (3, 2001, 9), (2, 17, 1501), (1, 841, 843),
            (1, 845, 847)]
# 2 (n N)^3 operations below and above 2e8; n N = 31 .. 129 beside the tiles
WALLS = [(1, 31, 33), (1, 65, 63), (3, 43, 11), (4, 32, 16), (1, 464, 464), (1, 465, 465)]


def _wn(g, u):
    return math.sqrt(O.inner(g, u, u))


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n,nx,ny,walls", [c + (False,) for c in PERIODIC]
                         + [c + (True,) for c in WALLS])
def test_products(n, nx, ny, walls, mixed):
    from paper_1311_7477_amd import dg
    print(f"fd products n={n} {nx}x{ny} walls={walls} mixed={mixed}", flush=True)
    bc = "dirichlet" if walls else "periodic"
    g = O.Grid2D(n, nx, ny, 0.0, 2.0, -1.0, 1.5, bc, bc)
    grid = dg.Grid(n, nx, ny, 0.0, 2.0, -1.0, 1.5, int(walls), int(walls))
    ws = dg.Workspace(grid, dg.DG_WS_FD)
    r = I.white_noise(n, nx, ny, seed=3 * n + nx) + 0.7
    fd = O.FastDiagonalisation(g)
    ref = fd.apply(r)
    b = r if walls else r - O.wmean(g, r)
    floor = _wn(g, b + O.laplacian(g, ref))
    if mixed:
        # the FP32 inverse under the FP64 iteration: the solve's own target
        psi = torch.zeros(r.shape, dtype=torch.float64, device="cuda")
        opts = dg.cg_opts(rtol=1e-9, precond=dg.DG_PRECOND_FD, precision=dg.DG_PREC_MIXED)
        res = dg.cg_solve_poisson(grid, torch.from_numpy(r).cuda(), psi, ws, opts)
        assert res.converged
        got = psi.cpu().numpy()
        assert _wn(g, b + O.laplacian(g, got)) <= max(2e-9 * _wn(g, b), 4.0 * floor)
        return
    got = dg.precond_apply(grid, torch.from_numpy(r).cuda(), ws).cpu().numpy()
    inv = np.abs(fd.inv_mu[fd.inv_mu != 0])
    kappa = inv.max() / inv.min()
    d = got - ref
    if not walls:
        d -= O.wmean(g, d)
    assert np.max(np.abs(d)) <= 2e-14 * kappa * np.max(np.abs(ref))
    assert _wn(g, b + O.laplacian(g, got)) <= max(1e-11 * _wn(g, b), 4.0 * floor)
