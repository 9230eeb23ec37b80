"""How often a solve is polled, and how many iterations it is allowed, change
neither its result nor its end, up to the largest values of their type."""
import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

INT_MAX = 2 ** 31 - 1


@pytest.mark.parametrize("every", [1, 2, 7, 2000, 2001, INT_MAX - 1, INT_MAX])
def test_check_every(every):
    from paper_1311_7477_amd import dg
    print(f"cg check_every={every}", flush=True)
    grid = dg.Grid(3, 20, 18)
    w = torch.from_numpy(I.white_noise(3, 20, 18, seed=1)).cuda()
    out = []
    for e in (0, every):
        psi = torch.zeros_like(w)
        res = dg.cg_solve_poisson(grid, w, psi, dg.Workspace(grid),
                                  dg.cg_opts(rtol=1e-12, max_iter=2000, check_every=e))
        assert res.converged
        out.append((res.iters, psi))
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("graphs", [True, False])
def test_batch_iterations_allowed(graphs):
    from paper_1311_7477_amd import dg
    print(f"batch max_iter graphs={graphs}", flush=True)
    w0 = torch.from_numpy(I.white_noise(3, 20, 18, seed=1)).cuda()
    out = []
    for most in (100000, INT_MAX):
        batch, w = dg.Batch(1, use_graphs=graphs), w0.clone()
        slot = batch.attach(dg.Grid(3, 20, 18), w, 1e-4, 1e-3)
        iters, ok = batch.rk_step(dg.cg_opts(rtol=1e-12, max_iter=most))
        assert ok
        out.append((iters[slot], w))
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])


# Solves that are over before their first iteration, on a grid of few blocks and on
# one of more than are summed directly: the guess stays, and only its mean goes.
@pytest.mark.parametrize("n,nx,ny", [(3, 20, 18), (1, 610, 196)])
def test_nothing_to_iterate(n, nx, ny):
    from paper_1311_7477_amd import dg
    print(f"cg nothing to do n={n} {nx}x{ny}", flush=True)
    grid = dg.Grid(n, nx, ny)
    ws = dg.Workspace(grid)
    guess = torch.from_numpy(I.white_noise(n, nx, ny, seed=1)).cuda()
    w = -dg.laplace_apply(grid, guess)
    psi = [guess + 2.0, guess + 2.0]
    done = dg.cg_solve_poisson(grid, w, psi[0], ws, dg.cg_opts(rtol=1e-9))
    none = dg.cg_solve_poisson(grid, w, psi[1], ws, dg.cg_opts(rtol=1e-30, max_iter=0))
    assert done.converged and done.iters == 0
    assert not none.converged and none.iters == 0
    assert torch.equal(psi[0], psi[1])
    shift = psi[0] - guess
    assert float((shift - shift.mean()).abs().max()) <= 4 * 2.0 ** -52 * float(guess.abs().max() + 2)
