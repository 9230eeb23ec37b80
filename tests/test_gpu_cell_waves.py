"""At n = 5 cell tiles of 16 rows run as tiles of 8: every solve that takes cell tiles
gives the same bits for both, on a grid whose last tiles are partly empty."""
import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["stored in FP32", "preconditioned", "preconditioned in FP32"])
def test_sixteen_rows_as_eight(kind):
    from paper_1311_7477_amd import dg
    print(f"cell waves {kind}", flush=True)
    n, nx, ny = 5, 100, 76
    mode = dg.DG_PREC_MIXED if kind == "stored in FP32" else dg.DG_WS_FD | dg.DG_WS_FD_PRODUCTS
    opts = dg.cg_opts(rtol=1e-11, max_iter=200 if mode == dg.DG_PREC_MIXED else 20,
                      precision=dg.DG_PREC_FP64 if kind == "preconditioned" else dg.DG_PREC_MIXED,
                      precond=dg.DG_PRECOND_NONE if mode == dg.DG_PREC_MIXED else dg.DG_PRECOND_FD)
    w = torch.from_numpy(I.white_noise(n, nx, ny, seed=4)).cuda()
    out = []
    for cw in (8, 16):
        grid = dg.Grid(n, nx, ny, 0.0, 2.0, 0.0, 1.5)
        grid.set_tiles(cw, 8)
        assert grid.tiles() == (cw, 8)
        psi = torch.zeros_like(w)
        res = dg.cg_solve_poisson(grid, w, psi, dg.Workspace(grid, mode), opts)
        out.append((res.iters, psi, dg.laplace_apply(grid, psi)))
    assert out[0][0] == out[1][0] > 0
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])
