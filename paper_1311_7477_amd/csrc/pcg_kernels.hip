// First iteration and end of a preconditioned solve in one pass over the cells
// (cell per lane; layouts and the operator are in cg_body.h).
//
// The preconditioner is the inverse of -Lap_h, exact up to rounding (FP64) or
// up to the FP32 arithmetic of its transforms, so the first CG step length
// <r,z> / <z, A z> is 1 to that accuracy and the step x1 = x0 + z, r1 = r0 - A z
// needs neither sum.  This kernel takes it: r1 (whose norm, summed from r1
// itself, decides convergence as ever) and psi = x1 minus its mean, which
// stands if the solve has converged, as it nearly always has.  Otherwise CG
// starts afresh from x1 and r1 (the next beta is 0).
// Bound by memory: reads z, r and x, writes r and psi (n = 5, 1024^2: 213 us,
// 4.9 TB/s).  The direction, residual and finish kernels that it replaces here
// read z twice more and r and x as often, and the dot kernel before them had to
// read r for <r,z>: the four together n = 4, 512^2 72 -> 46 us, n = 5, 1024^2 456
// -> 283 us, and two launches fewer.  Tiles as the Laplacian's (laplace_waves):
// its LDS is the same, the face scalars and then the staged rows of psi.
#include "cg_body.h"
#include "dg_launch.h"

namespace dgk {

namespace {

template <int N, int WV, bool DIR, bool ISO>
__global__ __launch_bounds__(64 * WV, (N == 4 && !DIR) ? 4 : 1) void k_pcg_first(
    Geom g, int tilesX, int nblocks, OpConst<double> k, const double* __restrict__ x,
    const double* __restrict__ z, double* __restrict__ r, double* __restrict__ psi, CgScalars* sc,
    unsigned* counter, double* partials) {
    __shared__ LaplaceLds<N, WV> lds;
    // the setup may have ended the solve (r0 within the tolerance, b = 0, no
    // iteration allowed): then psi = x0, or 0
    const bool done = sc->done, zero = sc->zero;
    const double mean = done ? sc->mean_x : sc->mean_x + sc->mean_p;
    const CellCtx c = make_cell_ctx<N, WV>(g, tilesX, nblocks, blockIdx.x);
    double zv[N * N], part[1] = {0.0};
    zero_cell<N>(zv);
    if (!done) {
        SrcL64<N, double> src{z};
        double q[N * N];
        if (c.active) src(c.self, zv);
        lap_cell<N, WV, DIR, ISO>(c, k, src, zv, lds, q);      // q = Lap z = -A z
        if (c.active) {
            double rv[N * N];
            ld_l64<N>(r, c.self, rv);
#pragma unroll
            for (int e = 0; e < N * N; ++e) rv[e] += q[e];
            st_l64<N>(r, c.self, rv);
            part[0] = wdot_cell<N>(k, rv, rv);
        }
        __syncthreads();      // the face scalars are read: the buffers are free
    }
    if (c.active && !zero) {
        double xv[N * N];
        ld_l64<N>(x, c.self, xv);
#pragma unroll
        for (int e = 0; e < N * N; ++e) zv[e] = (xv[e] + zv[e]) - mean;
    } else {
        zero_cell<N>(zv);
    }
    if constexpr (staged_rows(N)) stage_out<N>(psi + c.row0, c.count, lds.row(c.wave), c.lane, zv);
    else if (c.active) st_canon<N>(psi, c.self, zv);
    if (done) return;
    double tot[1];
    if (reduce_last<1, 64 * WV>(part, partials, counter, nblocks, blockIdx.x, tot) &&
        threadIdx.x == 0) {
        const double rrn = tot[0];
        if (!(rrn < __builtin_inf())) {    // non-finite data: x stays x0
            sc->done = 1;
            sc->breakdown = 1;
            return;
        }
        sc->rr = rrn;
        sc->rz = 0.0;
        sc->alpha = 1.0;
        sc->mean_x += sc->mean_p;
        sc->first = 0;
        sc->iter = 1;
        if (rrn <= sc->tol2 * sc->bb) {
            sc->done = 1;
            sc->converged = 1;
            sc->pending = 1;
        } else if (sc->max_iter <= 1) {
            sc->done = 1;
            sc->pending = 1;
        }
    }
}

}  // namespace

hipError_t launch_pcg_first(const Geom& g, const OpConst<double>& k, const double* x,
                            const double* z, double* r, double* psi, const DevScratch& d,
                            hipStream_t s) {
    const CellLaunch L(g, laplace_waves(g.n, g.cw));
#define DG_FIRST(W, DIR, ISO)                                                                     \
    hipLaunchKernelGGL((k_pcg_first<NN, laplace_waves(NN, W), DIR, ISO>), dim3(L.nblocks),        \
                       dim3(64 * laplace_waves(NN, W)), 0, s, g, L.tilesX, L.nblocks, k, x, z, r, \
                       psi, d.sc, d.counters + kCntRes * kCntStride, d.partials)
    if (dirichlet(g)) {
        if (g.cw != kDirichletCellWaves) return hipErrorInvalidValue;
        if (iso_dir(g, k)) {
            DG_DISPATCH_N(g.n, DG_FIRST(kDirichletCellWaves, true, true));
        } else {
            DG_DISPATCH_N(g.n, DG_FIRST(kDirichletCellWaves, true, false));
        }
    } else if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, DG_FIRST(WW, false, true));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, DG_FIRST(WW, false, false));
    }
#undef DG_FIRST
    return hipGetLastError();
}

}  // namespace dgk
