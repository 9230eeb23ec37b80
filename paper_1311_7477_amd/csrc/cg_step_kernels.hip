// Single-instance launches of the one-kernel CG iteration (device code in
// cg_step_body.h): block b processes tile xcd_tile(b).
#include <hip/hip_ext.h>

#include "cg_step_body.h"
#include "dg_launch.h"

namespace dgk {

template <int N, int WV, bool ISO, bool WRAP>
__global__ __launch_bounds__(64 * WV, N == 4 ? 4 : 1) void k_cg_step(
    Geom g, int tilesX, int nblocks, OpConst<double> k, LapScale sl, int par, const double* __restrict__ rin,
    double* __restrict__ rout, const double* __restrict__ pin, double* __restrict__ pout,
    double* __restrict__ x, const CgScalars* __restrict__ sc_in, CgScalars* __restrict__ sc_out,
    const double* __restrict__ part_in, double* part_out, unsigned* counter) {
    __shared__ StepLds<N, WV> lds;
    cg_step_body<N, WV, ISO, WRAP>(blockIdx.x, g, tilesX, nblocks, k, sl, par, rin, rout, pin, pout, x,
                             sc_in, sc_out, part_in, part_out, counter, lds);
}

// Waves per tile, by the grid alone (the cell tile height is that of the other
// kernels): 8, but 4
// - where tiles of 4 are one per CU at most, two at n = 5, whose tiles of 8 fit one at a
//   time (more of the chip at work; us per iteration with tiles of 4 and 8: n = 3,
//   128^2 6.6 and 7.5, n = 5 10.4 and 13.7, 120 x 512 20.4 and 22.6, 20000 x 1 15.4 and
//   30.4; at 400 tiles of 4 n = 4, 200^2 12.2 and 11.1, n = 5 16.4 and 15.9);
// - for n >= 4 where tiles of 8 would be 2 to 3.5 a CU, of which two fit at once, and a
//   row of tiles is short enough for the L2 to hold the next one's halo (n = 4, 450^2
//   29.7 and 31.4, 512^2 37.8 and 38.3, n = 5, 512^2 65.3 and 70.8; but n = 5, 600^2,
//   3.9 a CU, 102 and 94, and n = 4, 4096 x 64, 69 tiles a row, 47.8 and 41.4);
// - at n = 5 on rows of up to 4 tiles, whose next row the L2 always holds (128 x 512
//   26.5 and 36.7, 180 x 4096 209 and 247, 128 x 4096 180 and 192; 5 tiles: 256^2 23.7
//   and 18.9, 256 x 4096 314 and 335).
// Elsewhere the larger share of recomputed cells costs more or as much (n = 4, 256^2
// 15.2 and 13.1; n = 5, 800^2 182 and 177).
int step_waves(const Geom& g) {
    constexpr int kCu = 256;
    const StepLaunch s8(g, 8);
    const bool few = StepLaunch(g, 4).nblocks <= (g.n == 5 ? 2 : 1) * kCu;
    const bool rounds = s8.nblocks > 2 * kCu && 2 * s8.nblocks < 7 * kCu && s8.tilesX <= 32;
    return few || (g.n >= 4 && rounds) || (g.n == 5 && s8.tilesX <= 4) ? 4 : 8;
}

int step_max_blocks(const Geom& g) { return StepLaunch(g, 4).nblocks; }

size_t step_part_bytes(const Geom& g) {
    return 2 * step_part_stride(step_max_blocks(g)) * sizeof(double);
}

hipError_t launch_cg_step(const Geom& g, const OpConst<double>& k, int par, const StepBuffers& v,
                          unsigned* counters, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    if (g.bcx || g.bcy) return hipErrorInvalidValue;
    const StepLaunch L(g, step_waves(g));
    const size_t stride = step_part_stride(v.max_blocks);
    const double* rin = par ? v.r1 : v.r0;
    double* rout = par ? v.r0 : v.r1;
    const double* pin = par ? v.p1 : v.p0;
    double* pout = par ? v.p0 : v.p1;
    const double* part_in = v.part + (par ? stride : 0);
    double* part_out = v.part + (par ? 0 : stride);
    unsigned* counter = counters + kCntDir * kCntStride;
#define DG_STEP(ISO, WRAP)                                                                           \
    DG_DISPATCH_NS(g.n, L.wv,                                                                  \
                   hipExtLaunchKernelGGL((k_cg_step<NN, WW, ISO, WRAP>), dim3(L.nblocks),            \
                                         dim3(64 * WW), 0, s, start, stop, 0, g, L.tilesX,     \
                                         L.nblocks, k, v.scale, par, rin, rout, pin, pout, v.x,      \
                                         (const CgScalars*)v.sc[par], v.sc[1 - par], part_in,  \
                                         part_out, counter))
    const bool wrap = step_wraps(g);
    if (k.ihx == k.ihy) {
        if (wrap) {
            DG_STEP(true, true);
        } else {
            DG_STEP(true, false);
        }
    } else if (wrap) {
        DG_STEP(false, true);
    } else {
        DG_STEP(false, false);
    }
#undef DG_STEP
    return hipGetLastError();
}

}  // namespace dgk
