"""Live timing counts launches that ran a whole iteration, and no others."""
import math

import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_only_iterations_are_sampled():
    from paper_1311_7477_amd import dg
    print("profile", flush=True)
    grid = dg.Grid(3, 24, 20)
    ws = dg.Workspace(grid)
    ws.profile(True)
    w = torch.from_numpy(I.white_noise(3, 24, 20, seed=1)).cuda()
    psi = torch.zeros_like(w)
    # nothing to solve, no iteration allowed, one iteration (the launch that only
    # makes the first direction is not one)
    assert dg.cg_solve_poisson(grid, torch.zeros_like(w), psi, ws).iters == 0
    assert ws.read_profile()[1] == 0
    dg.cg_solve_poisson(grid, w, psi, ws, dg.cg_opts(rtol=1e-12, max_iter=0))
    assert ws.read_profile()[1] == 0
    # the last launch finds the solve stopped; of k iterations launches 1 .. k count
    for k, every in ((1, 2), (5, 2), (64, 0)):
        psi.zero_()
        assert dg.cg_solve_poisson(grid, w, psi, ws, dg.cg_opts(
            rtol=1e-14, max_iter=k, check_every=every)).iters == k
        ms, count, _, residual = ws.read_profile()
        # launches 1, chunk, 2 chunk + 1, 3 chunk, ...
        chunk = every or 32
        want = sum(1 for r in range(k // chunk + 2) if 1 <= r * chunk + (~r & 1) <= k)
        assert count == want and residual == 0 and 0.0 < ms < 1.0
    psi.zero_()
    assert dg.cg_solve_poisson(grid, w, psi, ws).converged
    ws.read_profile()
    dg.cg_solve_poisson(grid, w, psi, ws, dg.cg_opts(rtol=1e-10))      # already solved
    assert ws.read_profile()[1] == 0 and math.isnan(ws.read_profile()[0])
