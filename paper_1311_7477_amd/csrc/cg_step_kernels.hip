// Single-instance launches of the one-kernel CG iteration (device code in
// cg_step_body.h): block b processes tile xcd_tile(b).
#include <hip/hip_ext.h>

#include "cg_step_body.h"
#include "dg_launch.h"

namespace dgk {

template <int N, int WV, bool ISO>
__global__ __launch_bounds__(64 * WV, N == 4 ? 4 : 1) void k_cg_step(
    Geom g, int tilesX, int nblocks, OpConst<double> k, LapScale sl, int par, const double* __restrict__ rin,
    double* __restrict__ rout, const double* __restrict__ pin, double* __restrict__ pout,
    double* __restrict__ x, const CgScalars* __restrict__ sc_in, CgScalars* __restrict__ sc_out,
    const double* __restrict__ part_in, double* part_out, unsigned* counter) {
    __shared__ StepLds<N, WV> lds;
    cg_step_body<N, WV, ISO>(blockIdx.x, g, tilesX, nblocks, k, sl, par, rin, rout, pin, pout, x,
                             sc_in, sc_out, part_in, part_out, counter, lds);
}

// Waves per tile: the grid's cell tile height, except that its default of 8
// gives way to 4 where tiles of 4 are one per CU at most (more of the chip at
// work: 6.6 against 7.5 us per iteration at n = 3, 128^2, 10.5 against 14.0 at
// n = 5) and, for n >= 4, where tiles of 8 are between one and two rounds (two
// fit a CU at once: 39.0 against 41.3 us at n = 4, 512^2, 67 against 73 at n =
// 5).  Elsewhere their larger share of recomputed cells costs more (n = 4,
// 256^2: 15.2 against 13.6 us; n = 5, 1024^2: 301 against 288).
int step_waves(const Geom& g) {
    constexpr int kCu = 256;
    if (g.cw != 8) return g.cw;
    const int b8 = StepLaunch(g, 8).nblocks;
    const bool few = StepLaunch(g, 4).nblocks <= kCu;
    return few || (g.n >= 4 && b8 > 2 * kCu && b8 < 4 * kCu) ? 4 : 8;
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
#define DG_STEP(ISO)                                                                           \
    DG_DISPATCH_NW(g.n, L.wv,                                                                  \
                   hipExtLaunchKernelGGL((k_cg_step<NN, WW, ISO>), dim3(L.nblocks),            \
                                         dim3(64 * WW), 0, s, start, stop, 0, g, L.tilesX,     \
                                         L.nblocks, k, v.scale, par, rin, rout, pin, pout, v.x,      \
                                         (const CgScalars*)v.sc[par], v.sc[1 - par], part_in,  \
                                         part_out, counter))
    if (k.ihx == k.ihy) {
        DG_STEP(true);
    } else {
        DG_STEP(false);
    }
#undef DG_STEP
    return hipGetLastError();
}

}  // namespace dgk
