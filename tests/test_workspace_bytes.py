"""Device memory of a workspace: four CG vectors (whose rows are padded to 64 cells)
and two canonical fields, and only a periodic FP64 workspace has a fifth vector in
place of one of the fields.  Host only."""
import pytest

from paper_1311_7477_amd import dg

MIXED, FD = dg.DG_PREC_MIXED, dg.DG_WS_FD


def sizes(n, nx, ny):
    return 8 * n * n * nx * ny, 8 * n * n * 64 * ((nx + 63) // 64) * ny


# everything else: the reductions' partial sums and counters, at most 64 bytes for
# each of the tiles of 4 rows (60 x 2 cells stored in the iteration kernel, two sets)
# and a few tens of KB
def rest(nx, ny):
    return 65536 + 64 * ((nx + 59) // 60 + 1) * (ny + 2)


@pytest.mark.parametrize("n", [1, 2, 3, 5])
@pytest.mark.parametrize("nx,ny", [(1, 5000), (65, 900), (64, 900), (129, 301), (1000, 7)])
def test_vectors_and_fields(n, nx, ny):
    F, L = sizes(n, nx, ny)
    periodic = dg.Grid(n, nx, ny)
    for walls in ((1, 1), (0, 1), (1, 0)):
        b = dg.Grid(n, nx, ny, bc_x=walls[0], bc_y=walls[1]).workspace_bytes()
        assert 4 * L + 2 * F <= b <= 4 * L + 2 * F + rest(nx, ny)
    b = periodic.workspace_bytes()
    assert 5 * L + F <= b <= 5 * L + F + rest(nx, ny)
    b = periodic.workspace_bytes(MIXED)
    assert 5.5 * L + 2 * F <= b <= 5.5 * L + 2 * F + rest(nx, ny)


# what the preconditioner itself takes is the same beside FP64 and FP32 vectors
@pytest.mark.parametrize("n,nx,ny", [(2, 65, 90), (3, 1, 200), (5, 33, 40)])
def test_preconditioned(n, nx, ny):
    F, L = sizes(n, nx, ny)
    grid = dg.Grid(n, nx, ny)
    more = grid.workspace_bytes(MIXED) - grid.workspace_bytes()
    assert abs(more - (0.5 * L + F)) <= 16           # (fields begin on 16 bytes)
    assert grid.workspace_bytes(FD | MIXED) - grid.workspace_bytes(FD) == more
    # z, omega's copy
    planes = grid.workspace_bytes(FD | MIXED) - grid.workspace_bytes(MIXED) - L - F
    walls = dg.Grid(n, nx, ny, bc_x=1)
    assert 0 < planes < 4 * (n * n * 8 * (nx + 2) * (ny + 2)) + 64 * (n * max(nx, ny)) ** 2 + 65536
    assert walls.workspace_bytes(FD) > walls.workspace_bytes() + L + F
