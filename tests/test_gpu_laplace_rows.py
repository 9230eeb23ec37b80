"""The Laplacian on both sides of the rules that choose between staged rows of cells
and lanes that read their own, against the oracle: narrow, flat and small grids,
periodic and with walls."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KIND = {0: "periodic", 1: "dirichlet"}


# rounding of one operator row, as in the other element-wise parity tests
@pytest.mark.parametrize("n,nx,ny,walls", [
    (3, 39, 20, (0, 0)), (3, 40, 20, (0, 0)), (4, 39, 9, (0, 0)), (4, 41, 9, (0, 0)),
    (5, 64, 64, (0, 0)), (5, 600, 7, (0, 0)), (5, 600, 8, (0, 0)), (5, 39, 120, (0, 0)),
    (3, 387, 387, (1, 1)), (3, 388, 387, (0, 1)), (4, 180, 166, (1, 1)), (4, 180, 170, (1, 1)),
    (4, 244, 240, (0, 1)), (4, 256, 240, (1, 0)), (5, 64, 64, (1, 1)), (5, 65, 64, (1, 1)),
    (5, 64, 64, (1, 0)), (5, 62, 66, (0, 1)),
])
@pytest.mark.parametrize("square", [True, False])
def test_laplacian(n, nx, ny, walls, square):
    from paper_1311_7477_amd import dg
    print(f"laplacian rows n={n} {nx}x{ny} {walls} square={square}", flush=True)
    box = (0.0, nx / 8.0, 0.0, ny / 8.0) if square else (0.0, 2.0, -1.0, 1.5)
    u = np.random.default_rng(nx + ny).standard_normal((ny, nx, n, n))
    ref = O.laplacian(O.Grid2D(n, nx, ny, *box, *[KIND[w] for w in walls]), u)
    buf = torch.full((u.size + 1,), float("nan"), dtype=torch.float64, device="cuda")
    out = buf[1:].view(u.shape)
    dg.laplace_apply(dg.Grid(n, nx, ny, *box, *walls), torch.from_numpy(u).cuda(), out=out)
    got = out.cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
