"""The bracket and the right-hand side on both sides of the line between the row
kernel and the kernel that walks strips of cells, for the orders and widths where
strips need longer runs, against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# 62 cells a strip; rows of strips over the resident waves (4096, 1024, 1024): five
# at n = 2; from n = 4 on, with the two rows before a run, less than 5/4 (n = 4) or
# 3/2 (n = 5) of what the cells would fill.  The first of each pair takes strips.
SIZES = [(2, 47, 20480), (2, 47, 20479), (2, 1240, 1024), (2, 1240, 1023),
         (4, 62, 8193), (4, 62, 8192), (4, 683, 1157), (4, 683, 1156),
         (5, 62, 4097), (5, 62, 4096), (5, 94, 7470), (5, 94, 7469)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def line(n, nx, ny):
    strips, waves = -(-nx // 62), {2: 4096, 4: 1024, 5: 1024}[n]
    if n == 2:
        return 4 * nx >= 3 * 62 * strips and strips * ny >= 5 * waves
    return 62 * (strips * ny + 2 * waves) < (1.25 if n == 4 else 1.5) * nx * ny


# tolerance: rounding of one operator row, as in the other element-wise tests
@pytest.mark.parametrize("n,nx,ny", SIZES)
def test_bracket(n, nx, ny):
    from paper_1311_7477_amd import dg
    print(f"strip rule bracket n={n} {nx}x{ny}", flush=True)
    assert line(n, nx, ny) == (SIZES.index((n, nx, ny)) % 2 == 0)
    g = O.Grid2D(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    grid = dg.Grid(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    f, w = I.white_noise(n, nx, ny, seed=n), I.white_noise(n, nx, ny, seed=n + 10)
    got = dg.poisson_bracket(grid, dev(f), dev(w)).cpu().numpy()
    ref = O.bracket(g, f, w)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))


# one explicit Euler step with the solution the step itself solved for: the
# right-hand side is dt times its own rounding away, plus that of omega
@pytest.mark.parametrize("n,nx,ny", [(2, 1240, 1024), (4, 683, 1157), (5, 94, 7470)])
def test_right_hand_side(n, nx, ny):
    from paper_1311_7477_amd import dg
    print(f"strip rule rhs n={n} {nx}x{ny}", flush=True)
    g = O.Grid2D(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    grid = dg.Grid(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    w0 = I.white_noise(n, nx, ny, seed=n)
    w, ab, ws = dev(w0), dg.AbState(grid, 1), dg.Workspace(grid, dg.DG_WS_FD)
    D, opts = 0.3, dg.cg_opts(rtol=1e-9, precond=dg.DG_PRECOND_FD)
    dt = 0.01 / np.max(np.abs(O.laplacian(g, w0)))
    assert dg.ab_step(grid, w, ab, ws, dt, D, opts).converged
    rhs = -O.bracket(g, ab.psi().cpu().numpy(), w0) + D * O.laplacian(g, w0)
    got = (w.cpu().numpy() - w0) / dt
    tol = 1e-12 * np.max(np.abs(rhs)) + 2.0 ** -51 * np.max(np.abs(w0)) / dt
    assert np.max(np.abs(got - rhs)) <= tol
