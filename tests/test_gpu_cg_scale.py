"""Plain solves do not depend on the size of the vorticity: scaled by a power of
two, every iterate is the scaled iterate, up to sizes whose squares (<r, r>, <p, A
p>) are near the largest double; and on domains of any size."""
import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# |omega| < 2^3 and W < 2^3 summed over the domain: <r, r> stays under 2^1024 up to
# scales of 2^507; <A p, A p> itself would pass it from 2^503 (n = 1) and 2^499 on.
@pytest.mark.parametrize("n,N,power", [(1, 40, 504), (3, 24, 502), (4, 24, 502), (3, 24, -300)])
def test_scaled_vorticity(n, N, power):
    from paper_1311_7477_amd import dg
    print(f"cg scale n={n} N={N} 2^{power}", flush=True)
    grid = dg.Grid(n, N, N)
    w = torch.from_numpy(I.white_noise(n, N, N, seed=2)).cuda()
    out = []
    for s in (1.0, 2.0 ** power):
        psi = torch.zeros_like(w)
        res = dg.cg_solve_poisson(grid, w * s, psi, dg.Workspace(grid), dg.cg_opts(rtol=1e-10))
        assert res.converged
        out.append((res.iters, psi / s))
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])
    w1, w2 = w.clone(), w * 2.0 ** power
    batch = dg.Batch(2)
    # (D = 0, dt = 0; the first solve alone: the bracket of the scaled fields overflows)
    a, b = batch.attach(grid, w1, 0.0, 0.0), batch.attach(grid, w2, 0.0, 0.0)
    iters, _ = batch.rk_step(dg.cg_opts(rtol=1e-10, max_iter=2000))
    assert iters[a][0] == iters[b][0] == out[0][0] > 10


@pytest.mark.parametrize("power", [-200, 200])
def test_scaled_domain(power):
    from paper_1311_7477_amd import dg
    print(f"cg domain 2^{power}", flush=True)
    N = 30                # n = 1: no jump penalty, whose size depends on the cell
    w = torch.from_numpy(I.white_noise(1, N, N, seed=3)).cuda()
    out = []
    for s in (1.0, 2.0 ** power):
        grid = dg.Grid(1, N, N, 0.0, s, 0.0, s)
        psi = torch.zeros_like(w)
        res = dg.cg_solve_poisson(grid, w, psi, dg.Workspace(grid), dg.cg_opts(rtol=1e-10))
        assert res.converged
        out.append((res.iters, psi / s ** 2))
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])
