// Single-instance launches of the LDG Laplacian and CG kernels (cell per
// lane; the device code and its layout conventions are in cg_body.h).  One
// block per 64 x WV tile (WV = the grid's cell tile height g.cw, one of 4, 8,
// 16); block b processes tile xcd_tile(b).
#include <type_traits>

#include "cg_body.h"
#include "dg_launch.h"

namespace dgk {

template <int N, int WV, bool DIR, bool ISO, bool STAGED>
__global__ __launch_bounds__(64 * WV) void k_laplace(
    Geom g, int tilesX, int nblocks, OpConst<double> k,
    const double* __restrict__ u, double* __restrict__ out) {
    __shared__ RowsLds<N, WV, STAGED> lds;
    laplace_body<N, WV, DIR, ISO, STAGED>(blockIdx.x, g, tilesX, nblocks, k, u, out, lds);
}

template <int N, int WV, bool DIR, bool ISO, bool PRE>
__global__ __launch_bounds__(64 * WV) void k_cg_init(
    Geom g, int tilesX, int nblocks, OpConst<double> k,
    const double* __restrict__ omega, const double* __restrict__ pa,
    const double* __restrict__ pb, double ca, double cb, double inv_area,
    double* __restrict__ x, double* __restrict__ r, CgScalars* sc,
    unsigned* counter, double* partials, InitImage img) {
    __shared__ PairFaces<N, double, WV> lds;
    cg_init_body<N, WV, DIR, ISO, PRE>(blockIdx.x, g, tilesX, nblocks, k, omega, pa, pb, ca, cb,
                                       inv_area, x, r, sc, counter, partials, lds, img);
}

// At n = 4 the periodic direction and residual kernels are held to 128
// VGPRs (four waves per SIMD): with the paired 16-byte accesses they would
// take 132 / 134 and drop to three, which costs more than the 20 bytes per
// lane the residual kernel then spills.
template <int N, class S, int WV, bool DIR, bool ISO>
__global__ __launch_bounds__(64 * WV, (N == 4 && !DIR) ? 4 : 1) void k_cg_dir(
    Geom g, int tilesX, int nblocks, OpConst<double> k, const S* __restrict__ r,
    S* p0, S* p1, double* __restrict__ x, CgScalars* sc, unsigned* counter,
    double* partials) {
    __shared__ PairFaces<N, double, WV> lds;
    cg_dir_body<N, S, WV, DIR, ISO>(blockIdx.x, g, tilesX, nblocks, k, r, p0, p1, x, sc,
                               counter, partials, lds);
}

template <int N, class S, int WV, bool DIR, bool ISO>
__global__ __launch_bounds__(64 * WV, (N == 4 && !DIR) ? 4 : 1) void k_cg_res(
    Geom g, int tilesX, int nblocks, OpConst<double> k, const S* p0, const S* p1,
    S* __restrict__ r, CgScalars* sc, unsigned* counter, double* partials) {
    __shared__ PairFaces<N, double, WV> lds;
    cg_res_body<N, S, WV, DIR, ISO>(blockIdx.x, g, tilesX, nblocks, k, p0, p1, r, sc, counter,
                               partials, lds);
}

template <int N, int WV, bool ISO>
__global__ __launch_bounds__(64 * WV) void k_mixed_replace(
    Geom g, int tilesX, int nblocks, OpConst<double> k,
    const double* __restrict__ omega, const double* __restrict__ x,
    const float* __restrict__ q0, const float* __restrict__ q1,
    float* __restrict__ r32, CgScalars* sc, unsigned* counter, double* partials) {
    __shared__ PairFaces<N, double, WV> lds;
    mixed_replace_body<N, WV, ISO>(blockIdx.x, g, tilesX, nblocks, k, omega, x, q0, q1, r32,
                          sc, counter, partials, lds);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int cell_blocks(const Geom& g) { return CellLaunch(g).nblocks; }

// A grid with a homogeneous Dirichlet axis runs the DIR variants, built for
// 64 x 8 cell tiles only; square cells with the same boundary kind on both
// axes run the ISO variants (identical x and y blocks).
bool dirichlet(const Geom& g) { return g.bcx || g.bcy; }
bool iso(const Geom& g, const OpConst<double>& k) { return !dirichlet(g) && k.ihx == k.ihy; }
bool iso_dir(const Geom& g, const OpConst<double>& k) {
    return g.bcx && g.bcy && k.ihx == k.ihy;
}

// Whether the Laplacian of a grid stages its rows of cells, against lanes reading
// their own.  Staging moves whole runs of 64 cells, so it loses where a wave's row is
// short, and where the halo rows are most of what a tile reads; with walls it also takes
// the registers of a wave per SIMD.  us, lanes and staged:
// periodic  n = 3, 1 x 40000 29.7 and 36.7; n = 4, 12 x 3333 8.7 and 10.0, 48 x 833
//           equal, 512^2 22.1 and 16.0; n = 5, 32 x 1250 10.5 and 11.7, 16384 x 5 13.5 and
//           15.1, 8 rows equal, 8^2 9.2 and 7.1
// walls     n = 3, 333 x 257 7.2 and 8.3, 16384 x 12 13.3 and 11.0, 512^2 13.4 and 10.3; n
//           = 4, walls all round, 100 x 400 10.4 and 12.2, 180^2 9.8 and 8.4, 1024^2 68.8 and
//           57.2; two periodic sides, 128^2 8.9 and 9.4, 256^2 10.5 and 10.1, 1448^2 138 and
//           145; n = 5, 32 x 1250 14.4 and 18.1, 128^2 18.6 and 12.1, two periodic sides,
//           48^2 11.2 and 12.7, 128^2 12.9 and 12.2
static bool laplace_staged(const Geom& g) {
    if (!staged_rows(g.n)) return false;
    const long cells = (long)g.nx * g.ny, lanes = 64L * ((g.nx + 63) / 64);
    const bool all = g.bcx && g.bcy, mixed = !all && dirichlet(g);
    if (g.n == 5 && !mixed && cells <= 4096) return true;
    if (!dirichlet(g)) return g.nx >= 40 && (g.n < 5 || g.ny >= 8);
    if (g.n == 5) return 4 * g.nx >= 3 * lanes && g.ny >= 8 && (all || cells >= 4096);
    if (8 * g.nx < 7 * lanes) return false;
    if (g.n == 3) return g.ny >= 8 && cells >= 150000;
    if (g.ny < 32) return false;
    return all ? g.nx >= 128 && cells >= 30000 : cells >= 60000 && cells < 1600000;
}

hipError_t launch_laplace(const Geom& g, const OpConst<double>& k,
                          const double* u, double* out, hipStream_t s) {
    const bool staged = laplace_staged(g);
    const CellLaunch L(g, staged ? laplace_waves(g.n, g.cw) : cell_waves(g.n, g.cw));
#define DG_LAP_W(W, DIR, ISO, STAGED)                                                             \
    hipLaunchKernelGGL((k_laplace<NN, W, DIR, ISO, STAGED>), dim3(L.nblocks), dim3(64 * (W)), 0,  \
                       s, g, L.tilesX, L.nblocks, k, u, out)
#define DG_LAP(W, DIR, ISO)                                                     \
    if (staged) DG_LAP_W(laplace_waves(NN, W), DIR, ISO, staged_rows(NN));      \
    else DG_LAP_W(cell_waves(NN, W), DIR, ISO, false)
    if (dirichlet(g)) {
        if (g.cw != kDirichletCellWaves) return hipErrorInvalidValue;
        if (iso_dir(g, k)) {
            DG_DISPATCH_N(g.n, DG_LAP(kDirichletCellWaves, true, true));
        } else {
            DG_DISPATCH_N(g.n, DG_LAP(kDirichletCellWaves, true, false));
        }
    } else if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, DG_LAP(WW, false, true));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, DG_LAP(WW, false, false));
    }
#undef DG_LAP
#undef DG_LAP_W
    return hipGetLastError();
}

hipError_t launch_cg_init(const Geom& g, const OpConst<double>& k,
                          const double* omega, const double* pa,
                          const double* pb, double ca, double cb, double area, double* x,
                          double* r, const DevScratch& d, hipStream_t s, const InitImage& img) {
    CellLaunch L(g);
    const double inv_area = dirichlet(g) ? 0.0 : 1.0 / area;
#define DG_INIT(W, DIR, ISO, PRE)                                                                \
    hipLaunchKernelGGL((k_cg_init<NN, W, DIR, ISO, PRE>), dim3(L.nblocks), dim3(64 * (W)), 0, s, \
                       g, L.tilesX, L.nblocks, k, omega, pa, pb, ca, cb, inv_area, x, r, d.sc,   \
                       d.counters + kCntInit * kCntStride, d.partials, img)
#define DG_INIT_PRE(W, DIR, ISO)             \
    if (img.on) DG_INIT(W, DIR, ISO, true);  \
    else DG_INIT(W, DIR, ISO, false)
    if (dirichlet(g)) {
        if (g.cw != kDirichletCellWaves) return hipErrorInvalidValue;
        if (iso_dir(g, k)) {
            DG_DISPATCH_N(g.n, DG_INIT_PRE(kDirichletCellWaves, true, true));
        } else {
            DG_DISPATCH_N(g.n, DG_INIT_PRE(kDirichletCellWaves, true, false));
        }
    } else if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, DG_INIT_PRE(cell_waves(NN, WW), false, true));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, DG_INIT_PRE(cell_waves(NN, WW), false, false));
    }
#undef DG_INIT_PRE
#undef DG_INIT
    return hipGetLastError();
}

template <class S>
hipError_t launch_cg_dir(const Geom& g, const OpConst<double>& k, double* x, S* r, S* p0,
                         S* p1, CgScalars* sc, const DevScratch& d, hipStream_t s) {
    CellLaunch L(g);
    if (dirichlet(g)) {
        if constexpr (std::is_same<S, double>::value) {
            if (g.cw != kDirichletCellWaves) return hipErrorInvalidValue;
            if (iso_dir(g, k)) {
                DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_cg_dir<NN, S, kDirichletCellWaves, true, true>),
                                                      dim3(L.nblocks),
                                                      dim3(64 * kDirichletCellWaves), 0, s, g,
                                                      L.tilesX, L.nblocks, k, r, p0, p1, x, sc,
                                                      d.counters + kCntDir * kCntStride, d.partials));
            } else {
                DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_cg_dir<NN, S, kDirichletCellWaves, true, false>),
                                                      dim3(L.nblocks),
                                                      dim3(64 * kDirichletCellWaves), 0, s, g,
                                                      L.tilesX, L.nblocks, k, r, p0, p1, x, sc,
                                                      d.counters + kCntDir * kCntStride, d.partials));
            }
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_cg_dir<NN, S, cell_waves(NN, WW), false, true>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, r, p0, p1, x, sc,
                                              d.counters + kCntDir * kCntStride, d.partials));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_cg_dir<NN, S, cell_waves(NN, WW), false, false>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, r, p0, p1, x, sc,
                                              d.counters + kCntDir * kCntStride, d.partials));
    }
    return hipGetLastError();
}

template <class S>
hipError_t launch_cg_res(const Geom& g, const OpConst<double>& k, S* r, S* p0, S* p1,
                         CgScalars* sc, const DevScratch& d, hipStream_t s) {
    CellLaunch L(g);
    if (dirichlet(g)) {
        if constexpr (std::is_same<S, double>::value) {
            if (g.cw != kDirichletCellWaves) return hipErrorInvalidValue;
            if (iso_dir(g, k)) {
                DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_cg_res<NN, S, kDirichletCellWaves, true, true>),
                                                      dim3(L.nblocks),
                                                      dim3(64 * kDirichletCellWaves), 0, s, g,
                                                      L.tilesX, L.nblocks, k, p0, p1, r, sc,
                                                      d.counters + kCntRes * kCntStride, d.partials));
            } else {
                DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_cg_res<NN, S, kDirichletCellWaves, true, false>),
                                                      dim3(L.nblocks),
                                                      dim3(64 * kDirichletCellWaves), 0, s, g,
                                                      L.tilesX, L.nblocks, k, p0, p1, r, sc,
                                                      d.counters + kCntRes * kCntStride, d.partials));
            }
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_cg_res<NN, S, cell_waves(NN, WW), false, true>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, p0, p1, r, sc,
                                              d.counters + kCntRes * kCntStride, d.partials));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_cg_res<NN, S, cell_waves(NN, WW), false, false>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, p0, p1, r, sc,
                                              d.counters + kCntRes * kCntStride, d.partials));
    }
    return hipGetLastError();
}

template <class S>
hipError_t launch_cg_iter(const Geom& g, const OpConst<double>& k, double* x, S* r,
                          S* p0, S* p1, CgScalars* sc, const DevScratch& d,
                          hipStream_t s) {
    hipError_t e = launch_cg_dir<S>(g, k, x, r, p0, p1, sc, d, s);
    if (e != hipSuccess) return e;
    return launch_cg_res<S>(g, k, r, p0, p1, sc, d, s);
}

#define DG_INST(S)                                                             \
    template hipError_t launch_cg_dir<S>(const Geom&, const OpConst<double>&,   \
                                         double*, S*, S*, S*, CgScalars*,       \
                                         const DevScratch&, hipStream_t);       \
    template hipError_t launch_cg_res<S>(const Geom&, const OpConst<double>&, S*, \
                                         S*, S*, CgScalars*, const DevScratch&, \
                                         hipStream_t);                          \
    template hipError_t launch_cg_iter<S>(const Geom&, const OpConst<double>&,  \
                                          double*, S*, S*, S*, CgScalars*,      \
                                          const DevScratch&, hipStream_t);
DG_INST(double)
DG_INST(float)
#undef DG_INST

hipError_t launch_mixed_replace(const Geom& g, const OpConst<double>& k,
                                const double* omega, const double* x, const float* q0,
                                const float* q1, float* r32, const DevScratch& d,
                                hipStream_t s) {
    CellLaunch L(g);
    if (dirichlet(g)) return hipErrorInvalidValue;
    if (iso(g, k)) {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_mixed_replace<NN, cell_waves(NN, WW), true>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, omega, x, q0, q1, r32,
                                              d.sc, d.counters + kCntDot * kCntStride, d.partials));
    } else {
        DG_DISPATCH_NW(g.n, g.cw, hipLaunchKernelGGL((k_mixed_replace<NN, cell_waves(NN, WW), false>),
                                                     dim3(L.nblocks),
                                              dim3(64 * cell_waves(NN, WW)), 0, s, g, L.tilesX,
                                              L.nblocks, k, omega, x, q0, q1, r32,
                                              d.sc, d.counters + kCntDot * kCntStride, d.partials));
    }
    return hipGetLastError();
}

}  // namespace dgk
