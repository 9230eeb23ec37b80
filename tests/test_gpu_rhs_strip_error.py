"""Rounding of the bracket on smooth fields: the kernel that walks strips of cells
(larger periodic grids) against the row kernel, which a grid of one period of the
same fields takes.  Both are compared with the bracket in extended precision."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LD = np.longdouble


def gauss(n):
    """Gauss-Legendre nodes and weights in extended precision (Newton on P_n)."""
    x = np.polynomial.legendre.leggauss(n)[0].astype(LD)
    for _ in range(4):
        p0, p1 = np.ones_like(x), x.copy()
        for k in range(2, n + 1):
            p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / k
        d = n * (x * p1 - p0) / (x * x - 1)
        x = x - p1 / d
    return x, 2 / ((1 - x * x) * d * d)


def centred(n):
    """Blocks (self, right, left) of the centred derivative on cells of size 1."""
    x, w = gauss(n)
    c = [1 / np.prod([x[i] - x[m] for m in range(n) if m != i]) for i in range(n)]
    at = lambda y: np.array([c[i] * np.prod([y - x[m] for m in range(n) if m != i])
                             for i in range(n)], dtype=LD)
    dl = np.zeros((n, n), dtype=LD)
    for k in range(n):
        for i in range(n):
            if i != k:
                dl[k, i] = c[i] / c[k] / (x[k] - x[i])
        dl[k, k] = -dl[k].sum()
    up, um = at(LD(1)), at(LD(-1))
    iw = (2 / w)[:, None]
    return (-iw * (dl * w[:, None]).T + iw / 2 * (np.outer(up, up) - np.outer(um, um)),
            iw / 2 * np.outer(up, um), -iw / 2 * np.outer(um, up))


def product(M, u, axis):
    """M along a node axis (2: y, 3: x) of a field [cy][cx][j][i]."""
    v = np.moveaxis(u, axis, 0)
    out = np.zeros_like(v)
    for i in range(M.shape[0]):
        for m in range(M.shape[1]):
            out[i] += M[i, m] * v[m]
    return np.moveaxis(out, 0, axis)


def exact_bracket(f, g, h):
    C, R, L = centred(f.shape[3])

    def D(u, cells, nodes):
        return (product(C, u, nodes) + product(R, np.roll(u, -1, cells), nodes)
                + product(L, np.roll(u, 1, cells), nodes)) / h

    dx, dy = (lambda u: D(u, 1, 3)), (lambda u: D(u, 0, 2))
    f, g = f.astype(LD), g.astype(LD)
    fx, fy, gx, gy = dx(f), dy(f), dx(g), dy(g)
    return (fx * gy - fy * gx + dx(f * gy - fy * g) + dy(fx * g - f * gx)) / 3


# T x T cells of period 1, repeated on the large grid (enough rows of strips).
# The errors are averaged over T^2 n^2 >= 16384 nodes of rounding errors that are
# nearly independent, so that their rms is known to a few per cent: 1.05.
@pytest.mark.parametrize("n,T,times", [(2, 64, 18), (3, 64, 12), (4, 64, 13), (5, 64, 10)])
@pytest.mark.parametrize("k", [1, 4])
def test_no_further_from_exact_than_row_kernel(n, T, times, k):
    from paper_1311_7477_amd import dg
    print(f"strip error n={n} T={T} x {times} k={k}", flush=True)
    x = (np.arange(T)[:, None] + 0.5 + 0.5 * np.polynomial.legendre.leggauss(n)[0]) / T
    X = 2 * np.pi * x[None, :, None, :]
    Y = 2 * np.pi * x[:, None, :, None]
    f = np.sin(k * X + 1) * np.cos(Y) + 0.5 * np.cos(X - 2 * k * Y)
    g = np.cos(X + 0.3) * np.sin(k * Y) + 0.7 * np.sin(k * X + Y)
    one = dg.poisson_bracket(dg.Grid(n, T, T, 0.0, 1.0, 0.0, 1.0), torch.from_numpy(f).cuda(),
                             torch.from_numpy(g).cuda()).cpu().numpy()
    big = dg.Grid(n, T * times, T * times, 0.0, float(times), 0.0, float(times))
    tile = lambda u: torch.from_numpy(u).cuda().repeat(times, times, 1, 1)
    many = dg.poisson_bracket(big, tile(f), tile(g))
    ref = exact_bracket(f, g, LD(1) / T)
    rms = lambda u: float(np.sqrt(np.mean((u.astype(LD) - ref) ** 2)))
    errs = [rms(many[a * T:(a + 1) * T, a * T:(a + 1) * T].cpu().numpy())
            for a in range(0, times, 5)]
    print(f"  rms error: rows {rms(one):.3e}, strips {errs}", flush=True)
    assert not np.array_equal(one, many[:T, :T].cpu().numpy())     # two kernels
    assert max(errs) <= 1.05 * rms(one)
