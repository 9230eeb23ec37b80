"""The CG iteration kernel at the edges of its tiles, against the oracle's textbook
CG: rows of 61 to 64 cells, which one wave takes whole, and their neighbours; grids
large enough for tiles of 8 rows (6 stored) and those whose tiles of 4 it keeps; and
grids on which the last tiles hold little.  The cell tile height does not matter."""
import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# the bound of the other test of these iterates: after k <= 7 iterations a relative
# error of about 1e-15 per operation, the operator's entries spread by at most 1e2,
# k dependent scalars, and a factor of 10
@pytest.mark.parametrize("n,nx,ny", [
    (1, 60, 14), (1, 61, 14), (2, 62, 15), (3, 63, 16), (4, 64, 17), (5, 61, 3), (5, 64, 1),
    (5, 65, 4), (3, 64, 2),                                   # tiles of 4
    (1, 64, 519), (2, 63, 523), (3, 61, 517), (4, 65, 260), (5, 62, 521), (5, 122, 173),
    (2, 3, 1000),                                             # tiles of 8
    (4, 180, 1030), (5, 63, 3088),                            # 8 would be 2 to 3.5 a CU: 4
])
@pytest.mark.parametrize("k", [1, 2, 7])
def test_iterate_matches_textbook_cg(n, nx, ny, k):
    from paper_1311_7477_amd import dg
    print(f"cg step tiles n={n} nx={nx} ny={ny} k={k}", flush=True)
    w = I.white_noise(n, nx, ny, seed=nx + ny)
    ref = O.cg_poisson(O.Grid2D(n, nx, ny), w, rtol=1e-14, max_iter=k)
    got = []
    for cw in (4, 8, 16):
        grid = dg.Grid(n, nx, ny)
        grid.set_tiles(cw, 8)
        psi = torch.zeros(grid.shape, dtype=torch.float64, device="cuda")
        res = dg.cg_solve_poisson(grid, torch.from_numpy(w).cuda(), psi, dg.Workspace(grid),
                                  dg.cg_opts(rtol=1e-14, max_iter=k))
        assert res.iters == ref.iters
        got.append(psi.cpu().numpy())
        assert np.max(np.abs(got[-1] - ref.x)) <= 1e-11 * np.max(np.abs(ref.x))


# a batch cuts its members as a solve alone does
def test_batch_members():
    from paper_1311_7477_amd import dg
    print("cg step tiles batch", flush=True)
    opts, dt, D = dg.cg_opts(rtol=1e-9), 1e-4, 1e-4
    batch, inst = dg.Batch(5), []
    for n, nx, ny, cw in ((3, 64, 20, 8), (3, 61, 22, 16), (3, 62, 519, 4), (5, 63, 12, 4),
                          (3, 120, 21, 8)):
        grid = dg.Grid(n, nx, ny)
        grid.set_tiles(cw, 8)
        w0 = torch.from_numpy(I.random_modes(n, nx, ny, seed=nx)).cuda()
        w = w0.clone()
        inst.append((batch.attach(grid, w, dt, D), grid, w0, w))
    assert batch.rk_step(opts)[1]
    for slot, grid, w0, w in inst:
        st = dg.State(grid)
        dg.rk_step(grid, w0, st, dg.Workspace(grid), dt, D, opts)
        assert torch.equal(w, w0)
        assert torch.equal(batch.psi(slot), st.psi())


# members whose rows end within a wave in one launch group with others
def test_batch_group_of_both():
    from paper_1311_7477_amd import dg
    print("cg step tiles batch, one group", flush=True)
    opts, dt, D = dg.cg_opts(rtol=1e-9), 1e-4, 1e-4
    batch, inst = dg.Batch(9), []
    for n, nx, ny in ((2, 61, 9), (2, 33, 30), (3, 62, 18), (3, 64, 17), (3, 60, 20), (3, 130, 5),
                      (4, 63, 7), (5, 1, 40), (5, 63, 12)):
        grid = dg.Grid(n, nx, ny)
        w0 = torch.from_numpy(I.random_modes(n, nx, ny, seed=nx)).cuda()
        w = w0.clone()
        inst.append((batch.attach(grid, w, dt, D), grid, w0, w))
    for _ in range(2):
        assert batch.rk_step(opts)[1]
    for slot, grid, w0, w in inst:
        st, ws = dg.State(grid), dg.Workspace(grid)
        for _ in range(2):
            dg.rk_step(grid, w0, st, ws, dt, D, opts)
        assert torch.equal(w, w0)
        assert torch.equal(batch.psi(slot), st.psi())
