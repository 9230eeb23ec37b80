"""The tile tuner times kernels that differ by the tile it chooses, so that it
chooses the same each time."""
import pytest

from paper_1311_7477_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# at n = 5 and few tiles the two-kernel iteration takes 21 us with cw = 4 and 27 with 8
# (16 runs as 8 there); the one-kernel iteration, whose tiles do not follow cw, 10
def test_cell_tiles():
    from paper_1311_7477_amd import dg
    print("tune cell tiles", flush=True)
    grid = dg.Grid(5, 128, 128)
    w = torch.from_numpy(I.white_noise(5, 128, 128, seed=1)).cuda()
    for _ in range(3):
        (cw, _rw), ms = grid.tune(w, reps=50)
        assert cw == 4
        assert 1.1 * ms[0] < ms[1] == ms[2]


# a grid walked by strips: one kernel whatever rw, which stays 8
def test_strips():
    from paper_1311_7477_amd import dg
    print("tune strips", flush=True)
    grid = dg.Grid(5, 62, 6145)
    grid.set_tiles(8, 16)
    w = torch.from_numpy(I.white_noise(5, 62, 6145, seed=1)).cuda()
    (_cw, rw), ms = grid.tune(w, reps=3)
    assert rw == 8 and ms[3] == ms[4] > 0
