"""The bracket / right-hand-side kernel that walks strips of cells, which the
larger periodic grids take: whole and ragged strips, runs that pass the ends of
the rows, few long and many short rows, each order, on both sides of the sizes
where it takes over, against the oracle."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# strips x rows over the resident waves (6144, 4096, 2048, 1024, 1024): at least
# 4 rows a wave (6 from n = 4 on); 62 cells a strip, three quarters of them used
SIZES = [(1, 62, 24576), (1, 1300, 1171), (2, 1024, 964), (2, 47, 16384), (3, 620, 820),
         (3, 621, 745), (3, 8192, 62), (4, 620, 615), (4, 47, 6144), (4, 621, 559),
         (4, 620, 614), (5, 62, 6145), (5, 683, 513)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# rounding of one operator row, as in the other element-wise parity tests
@pytest.mark.parametrize("n,nx,ny", SIZES)
def test_bracket(n, nx, ny):
    from paper_1311_7477_amd import dg
    print(f"strip bracket n={n} {nx}x{ny}", flush=True)
    g = O.Grid2D(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    grid = dg.Grid(n, nx, ny, 0.0, 2.0, -1.0, 1.5)
    f, w = I.white_noise(n, nx, ny, seed=n), I.white_noise(n, nx, ny, seed=n + 10)
    buf = torch.full((f.size + 1,), float("nan"), dtype=torch.float64, device="cuda")
    got = dg.poisson_bracket(grid, dev(f), dev(w), out=buf[1:].view(f.shape)).cpu().numpy()
    ref = O.bracket(g, f, w)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
    if n == 3:
        for form, name in ((dg.DG_FORM_PP, "pp"), (dg.DG_FORM_PX, "px"), (dg.DG_FORM_XP, "xp")):
            got = dg.bracket_form(grid, dev(f), dev(w), form).cpu().numpy()
            one = O.bracket(g, f, w, form=name)
            assert np.max(np.abs(got - one)) <= 1e-12 * np.max(np.abs(ref))


# one explicit Euler step with the solution the step itself solved for: the
# right-hand side is dt times its own rounding away, plus that of omega
@pytest.mark.parametrize("n,nx,ny", [(2, 1024, 964), (4, 621, 615), (5, 620, 615)])
def test_right_hand_side(n, nx, ny):
    from paper_1311_7477_amd import dg
    print(f"strip rhs n={n} {nx}x{ny}", flush=True)
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


# a whole step (the three stage combinations), both sides with the exact
# preconditioner
def test_rk_step():
    from paper_1311_7477_amd import dg
    n, nx, ny = 3, 621, 820
    print(f"strip rk n={n} {nx}x{ny}", flush=True)
    g, grid = O.Grid2D(n, nx, ny), dg.Grid(n, nx, ny)
    w0 = I.random_modes(n, nx, ny, seed=5) + 1e-2 * I.white_noise(n, nx, ny, seed=6)
    dt, D = 1e-4, 1e-4
    ref = O.rk3_step_pcg(g, w0, 0.0, dt, D, O.PsiHistory(), rtol=1e-12,
                          precond=O.FastDiagonalisation(g).apply)[0]
    w, ws = dev(w0), dg.Workspace(grid, dg.DG_WS_FD)
    opts = dg.cg_opts(rtol=1e-12, precond=dg.DG_PRECOND_FD)
    assert dg.rk_step(grid, w, dg.State(grid), ws, dt, D, opts).converged
    e = w.cpu().numpy() - ref
    assert math.sqrt(O.inner(g, e, e)) <= 1e-12 * math.sqrt(O.inner(g, ref, ref))


# a batch with members on both kernels: bitwise as stepped alone
@pytest.mark.parametrize("graphs", [True, False])
def test_batch_members(graphs):
    from paper_1311_7477_amd import dg
    print(f"strip batch graphs={graphs}", flush=True)
    opts, dt, D = dg.cg_opts(rtol=1e-3), 1e-5, 1e-4
    batch, inst = dg.Batch(3, use_graphs=graphs), []
    for n, nx, ny in ((3, 621, 745), (3, 40, 30), (4, 620, 615)):
        grid = dg.Grid(n, nx, ny)
        w0 = dev(I.random_modes(n, nx, ny, seed=nx))
        w = w0.clone()
        inst.append((batch.attach(grid, w, dt, D), grid, w0, w))
    assert batch.rk_step(opts)[1]
    for slot, grid, w0, w in inst:
        st = dg.State(grid)
        dg.rk_step(grid, w0, st, dg.Workspace(grid), dt, D, opts)
        assert torch.equal(w, w0)
        assert torch.equal(batch.psi(slot), st.psi())
