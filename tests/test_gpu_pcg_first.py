"""The kernel that takes the first step of a preconditioned solve and writes the
solution: every way a solve can leave it, at the edges of its 64-cell rows and
tile heights, on periodic grids and with walls, against the oracle."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(1, 65, 3, 8), (2, 64, 9, 4), (2, 5, 17, 16), (3, 63, 8, 8), (3, 129, 5, 16),
         (4, 64, 17, 8), (4, 1, 4, 4), (4, 66, 33, 16), (5, 65, 6, 8), (5, 36, 5, 16)]


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("n,nx,ny,cw", SIZES)
def test_first_step(n, nx, ny, cw, walls):
    from paper_1311_7477_amd import dg
    print(f"pcg first n={n} {nx}x{ny} cw={cw} walls={walls}", flush=True)
    bc = "dirichlet" if walls else "periodic"
    g = O.Grid2D(n, nx, ny, 0.0, 2.0, -1.0, 1.5, bc, bc)
    grid = dg.Grid(n, nx, ny, 0.0, 2.0, -1.0, 1.5, int(walls), int(walls))
    if not walls:
        grid.set_tiles(cw, 8)
    ws = dg.Workspace(grid, dg.DG_WS_FD)
    w, guess = I.white_noise(n, nx, ny, seed=n) + 0.5, I.white_noise(n, nx, ny, seed=nx + 1)

    def less_mean(a):
        return a if walls else a - O.wmean(g, a)

    def norm(a):
        return math.sqrt(O.inner(g, a, a))

    def solve(omega, x0, **opts):
        psi = torch.from_numpy(np.ascontiguousarray(x0)).cuda()
        res = dg.cg_solve_poisson(grid, torch.from_numpy(np.ascontiguousarray(omega)).cuda(), psi,
                                  ws, dg.cg_opts(precond=dg.DG_PRECOND_FD, **opts))
        return res, psi.cpu().numpy()

    b = less_mean(w)
    r0 = b + O.laplacian(g, guess)
    # one step, then no more: x0 + M r0, as exact as the inverse (1e-11 of the
    # residual it is applied to, as for the inverse alone) or as the oracle's
    exact = O.FastDiagonalisation(g).apply(r0)
    bound = max(1e-11 * norm(r0), 4.0 * norm(r0 + O.laplacian(g, exact)))
    res, psi = solve(w, guess, rtol=1e-30, max_iter=1)
    assert not res.converged and res.iters == 1
    r = b + O.laplacian(g, psi)
    assert norm(r) <= bound
    assert abs(res.rel_residual - norm(r) / norm(b)) <= 0.5 * bound / norm(b) + 1e-15
    if not walls:
        assert abs(O.wmean(g, psi)) <= 1e-13 * np.max(np.abs(guess))
    # that solution is within a tolerance above its residual: the setup ends
    # the solve and the guess comes back (less its mean)
    res, again = solve(w, psi + (0.0 if walls else 3.0), rtol=2.0 * bound / norm(b) + 1e-9)
    assert res.converged and res.iters == 0
    assert np.max(np.abs(again - psi)) <= 1e-14 * (3.0 + np.max(np.abs(psi)))
    # no iteration allowed, b = 0, non-finite data
    res, same = solve(w, guess, rtol=1e-12, max_iter=0)
    assert not res.converged and res.iters == 0
    assert np.max(np.abs(same - less_mean(guess))) <= 1e-14 * np.max(np.abs(guess))
    res, zero = solve(np.zeros_like(w) if walls else np.full_like(w, 2.0), guess, rtol=1e-12)
    assert res.converged and res.iters == 0 and np.all(zero == 0)
    bad = w.copy()
    bad.flat[w.size // 2] = np.nan
    res, same = solve(bad, guess, rtol=1e-12)
    assert not res.converged and res.iters == 0
    assert np.max(np.abs(same - less_mean(guess))) <= 1e-14 * np.max(np.abs(guess))
    # and a solve to the tolerance, in FP64 and with the FP32 inverse
    for precision in (dg.DG_PREC_FP64, dg.DG_PREC_MIXED):
        rtol = 1e-10 + 4.0 * bound / norm(b)
        res, psi = solve(w, guess, rtol=rtol, precision=precision)
        assert res.converged and 1 <= res.iters <= 4
        assert norm(b + O.laplacian(g, psi)) <= 1.5 * rtol * norm(b)
