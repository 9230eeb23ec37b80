"""A batch with more launch groups than streams for their CG chunks (orders 1
to 5, two tile heights), stepped on a stream of the caller's: every member
bitwise as when stepped alone, with and without graphs."""
import numpy as np
import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MEMBERS = [(1, 40, 8), (2, 26, 8), (3, 21, 8), (3, 30, 16), (4, 18, 8), (4, 70, 4), (5, 14, 8)]


@pytest.mark.parametrize("graphs", [True, False])
def test_more_groups_than_lanes(graphs):
    from paper_1311_7477_amd import dg
    print(f"batch lanes graphs={graphs}", flush=True)
    D, opts, dt = 1e-4, dg.cg_opts(rtol=1e-11), 2e-3
    batch, inst = dg.Batch(len(MEMBERS), use_graphs=graphs), []
    stream = torch.cuda.Stream()
    for n, N, cw in MEMBERS:
        grid = dg.Grid(n, N, N)
        grid.set_tiles(cw, 8)
        w0 = torch.from_numpy(I.random_modes(n, N, N, seed=N)).cuda()
        w = w0.clone()
        inst.append((batch.attach(grid, w, dt, D), grid, w0, w))
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(2):
            assert batch.rk_step(opts)[1]
    stream.synchronize()
    for slot, grid, w0, w in inst:
        ws, st = dg.Workspace(grid), dg.State(grid)
        for _ in range(2):
            dg.rk_step(grid, w0, st, ws, dt, D, opts)
        assert np.array_equal(w.cpu().numpy(), w0.cpu().numpy())
        assert np.array_equal(batch.psi(slot).cpu().numpy(), st.psi().cpu().numpy())
