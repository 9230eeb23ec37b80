// One iteration of the plain FP64 conjugate-gradient solve in one kernel
// (periodic grids, cell per lane, L64 vectors).
//
// Textbook CG needs two grid-wide sums per iteration, <p, A p> before r is
// updated and <r, r> before p is, hence two launches.  With
//     <r_{k+1}, r_{k+1}> = <r_k, r_k> - 2 alpha_k <r_k, q_k> + alpha_k^2 <q_k, q_k>,
// q_k = A p_k, both alpha_k and beta_{k+1} follow from the sums of one pass
// over p_k (the identity holds whatever the directions are, so only its
// rounding matters); <r_k, r_k> itself is summed from the updated residual, so
// alpha and the convergence test never see the recurrence.  The launch of
// iteration k forms
//     r_k = r_{k-1} - alpha_{k-1} A p_{k-1},   p_k = r_k + beta_k p_{k-1},
// and sums <p_k, A p_k>, <A p_k, A p_k>, <r_k, A p_k>, <r_k, r_k>, from which
// the next launch takes its scalars.  A p_{k-1} is formed again here instead
// of being stored: reading and writing it would be two more fields.
// A is formed in units of its size (LapScale, a power of two: every rounding as
// without it), so that <q, q> overflows no earlier than <r, r> and <p, A p>.
// Per launch: read r, p; write r, p (4 fields); every other one also p_{k-2}
// and x (7 fields) -- 5.5 on average against 7.5 of the two-launch form.
// Microseconds per iteration, two launches -> this kernel: n = 3, 128^2
// 16.5 -> 6.6; n = 4, 512^2 49.5 -> 38.1 (4.8 TB/s of the 5.5 fields; counted,
// 6.1 are moved: 4.1 without x, 8.0 with it, most likely as the halo rows of r and p
// then no longer stay in the L2); n = 5, 1024^2 355 -> 288.  Small grids are bound by the chain of one launch (asking
// for the cells and the previous sums at once, one barrier per operator, no
// ticket), large ones by memory; in between a wave's loads, two operators and
// stores follow one another with too few waves to overlap them wholly.
//
// r_k and p_k are needed one cell beyond the cells whose A p_k is summed, so a
// tile is 64 x WV cells of which the inner 60 x (WV - 2) are summed and
// stored (all 64 lanes on rows of 61 to 64 cells, step_rim); the rest is formed
// again by the neighbouring tiles (the two outer lanes on each side have no valid
// neighbour and only feed the next ones; the face scalars beyond the first and last
// cell row are taken from a row loaded for them).  r and p are double-buffered.  Leaving face scalars for the
// neighbouring tiles in memory instead, so that no cell is formed twice, was
// measured: what a rim wave has to read and do made every wave of its tile wait
// (58 against 43 us per iteration at n = 4, 512^2; 9.9 against 7.0 us at n = 3,
// 128^2).
#pragma once

#include "cg_body.h"

namespace dgk {

// Up to kStepDirect blocks each launch sums the previous one's block sums
// itself (every wave, in the same order), so that no block waits for another;
// beyond, the last block of each of the kTicketGroups ticket groups sums its
// group first.
constexpr int kStepDirect = 256;
constexpr int kStepSums = 4;

// Doubles of the block sums of one launch parity.
__host__ __device__ constexpr size_t step_part_stride(int nblocks) {
    return (size_t)kStepSums * (nblocks + kTicketGroups);
}

// Tiles of one launch: 64 x wv cells, of which (64 - 2 rim) x (wv - 2) are stored.
struct StepLaunch {
    int wv, tilesX, tilesY, nblocks;
    __host__ __device__ StepLaunch(const Geom& g, int waves) : wv(waves) {
        const int w = 64 - 2 * step_rim(g);
        tilesX = (g.nx + w - 1) / w;
        tilesY = (g.ny + wv - 3) / (wv - 2);
        nblocks = tilesX * tilesY;
    }
};

template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
    return v + __hiloint2double(hi, lo);
}

__device__ __forceinline__ double read_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// v[lane & 3] summed over the wave's rows of 16 lanes (a fixed order by DPP
// moves: pairs, quads, halves), in every lane of the row.
__device__ __forceinline__ double row_sums4(const double (&v)[4], int lane) {
    double a[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        a[m] = add_dpp<0xb1>(v[m]);      // lane ^ 1
        a[m] = add_dpp<0x4e>(a[m]);      // lane ^ 2
        a[m] = add_dpp<0x141>(a[m]);     // 7 - lane within 8: the other quad
        a[m] = add_dpp<0x140>(a[m]);     // 15 - lane within 16: the other half
    }
    const double lo = lane & 1 ? a[1] : a[0], hi = lane & 1 ? a[3] : a[2];
    return lane & 2 ? hi : lo;
}

// The four sums over the wave, each in every lane.
__device__ __forceinline__ void wave_sums4(double (&v)[4], int lane) {
    double m = row_sums4(v, lane);
    m += __shfl_xor(m, 16);
    m += __shfl_xor(m, 32);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = read_lane(m, i);
}

template <int N, int WV>
struct StepLds {
    // y face scalars [row 0 .. WV + 1][lR, lL][i][lane]: row w + 1 is wave w's,
    // the outer ones those of the rows beyond the tile
    double face[(WV + 2) * 2 * N * 64];
    double red[WV * 4 * kStepSums];
};

// Lap_h u (times sl.unit) at node (j, i) from the cell's values and its face scalars.
template <int N, bool ISO>
__device__ __forceinline__ double lap_node(const OpConst<double>& k, const LapScale& sl,
                                           const double (&u)[N * N], int j, int i, double fR,
                                           double fL, double fU, double fD) {
    const double* L0y = ISO ? k.L0x : k.L0y;
    const double* eRy = ISO ? k.eRx : k.eRy;
    double lx = fmx(k.eRx[i], fR, k.eL[i] * fL);
    double ly = fmx(eRy[j], fU, k.eL[j] * fD);
#pragma unroll
    for (int m = 0; m < N; ++m) {
        lx = fmx(k.L0x[i * N + m], u[j * N + m], lx);
        ly = fmx(L0y[j * N + m], u[m * N + i], ly);
    }
    return fmx(lx, sl.x, ly * sl.y);
}

// x += ap pp + a p on one cell (n >= 4: in parts of at most eight nodes, so
// that what is in flight fits beside p_k).
template <int N>
__device__ __forceinline__ void add_to_x(double* __restrict__ x, const double* pp, const double* p,
                                         const CellRef& c, double a, double ap) {
    constexpr int P = (N * N) & ~1, M = N >= 4 ? 4 : P / 2 + (P == 0);
#pragma unroll
    for (int e0 = 0; e0 < P; e0 += 2 * M) {
        double2 xv[M], v[M], w[M];
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (e0 + 2 * m < P) {
                const long o = l64_at<N>(c.l64, e0 + 2 * m);
                xv[m] = *reinterpret_cast<const double2*>(x + o);
                v[m] = *reinterpret_cast<const double2*>(pp + o);
                w[m] = *reinterpret_cast<const double2*>(p + o);
            }
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (e0 + 2 * m < P) {
                xv[m].x = fmx(a, w[m].x, fmx(ap, v[m].x, xv[m].x));
                xv[m].y = fmx(a, w[m].y, fmx(ap, v[m].y, xv[m].y));
                *reinterpret_cast<double2*>(x + l64_at<N>(c.l64, e0 + 2 * m)) = xv[m];
            }
        if (N >= 4) __builtin_amdgcn_sched_barrier(0);
    }
    if (P < N * N) {
        const long o = l64_at<N>(c.l64, N * N - 1);
        x[o] = fmx(a, p[o], fmx(ap, pp[o], x[o]));
    }
}

// kWrap: there may be rows of 61 to 63 cells, which end within the wave (a template
// parameter: compiled in, other rows take 8 to 30% longer at n = 5).
// par: the launch's parity, that of the iteration while the solve runs.  The
// scalars and block sums written by the launch before are read from sc_in and
// part_in, this launch's go to sc_out and part_out.
template <int N, int WV, bool ISO, bool kWrap>
__device__ __forceinline__ void cg_step_body(
    int b, Geom g, int tilesX, int nblocks, const OpConst<double>& k, const LapScale& sl, int par,
    const double* __restrict__ rin, double* __restrict__ rout, const double* __restrict__ pin,
    double* __restrict__ pout, double* __restrict__ x, const CgScalars* __restrict__ sc_in,
    CgScalars* __restrict__ sc_out, const double* __restrict__ part_in, double* part_out,
    unsigned* counter, StepLds<N, WV>& lds) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = xcd_tile(b, nblocks);
    const int ty = t / tilesX, tx = t - ty * tilesX;
    const int rim = step_rim(g);
    const int cx = tx * (64 - 2 * rim) + lane - rim, cy = ty * (WV - 2) + wave - 1;
    const bool inner = wave > 0 && wave < WV - 1 && cy < g.ny;        // wave-uniform
    const bool store = inner && lane >= rim && lane < 64 - rim && cx < g.nx;
    // past the rims the outermost cell again, which its neighbours have read
    const int cxr = cx < g.nx + 1 ? cx : g.nx + 1, cyr = cy < g.ny + 1 ? cy : g.ny + 1;
    int gx = cxr < 0 ? cxr + 2 * g.nx : cxr;                          // cx >= -2, nx >= 1
    if (gx >= g.nx) gx %= g.nx;
    const int gy = (cyr + g.ny) % g.ny;
    const int G = (g.nx + 63) / 64;
    const CellRef self = cell_ref<N>(g, G, gx, gy);

    // A launch queued after the solve has stopped has nothing to do.  More blocks
    // than are summed directly find that out first; else they would read all of r
    // and p before (n = 4, 1448^2: 100 us for each of up to 64 such launches)
    if (nblocks > kStepDirect && sc_in->done) {
        if (b == 0 && threadIdx.x == 0) *sc_out = *sc_in;
        return;
    }
    // the previous launch's block sums and the cells' values, asked for before
    // anything is known of the solve's state (at the first iteration p, h and
    // the sums are not used)
    const int slots = nblocks <= kStepDirect ? nblocks : kTicketGroups;
    const double* src = nblocks <= kStepDirect ? part_in : part_in + (size_t)kStepSums * nblocks;
    double sum[kStepSums] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < kStepDirect / 64; ++u)
        if (lane + 64 * u < slots) {
            const double2* v = reinterpret_cast<const double2*>(src + kStepSums * (lane + 64 * u));
            const double2 v0 = v[0], v1 = v[1];
            sum[0] += v0.x;
            sum[1] += v0.y;
            sum[2] += v1.x;
            sum[3] += v1.y;
        }
    double p[N * N], r[N * N];
    ld_l64<N>(pin, self, p);
    ld_l64<N>(rin, self, r);
    const double* lLy = ISO ? k.lLx : k.lLy;
    constexpr int FR = 2 * N * 64;                          // one row of the face array
    double* face = lds.face + (wave + 1) * FR + lane;       // lR . u at i * 64, lL . u at (N + i) * 64
    if (wave == 0 || wave == WV - 1) {
        const int hrow = wave == 0 ? (gy > 0 ? gy - 1 : g.ny - 1) : (gy + 1 < g.ny ? gy + 1 : 0);
        double h[N * N];
        ld_l64<N>(pin, cell_ref<N>(g, G, gx, hrow), h);
        if (wave == 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) face[-FR + (N + i) * 64] = ydot<N>(h, i, lLy);
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) face[FR + i * 64] = ydot<N>(h, i, k.lR);
        }
    }

    // the scalars of this iteration
    CgScalars s = *sc_in;
    const bool first = s.first == 1;
    double alpha = 0.0, beta = 0.0;
    if (!s.done && !first) {
        wave_sums4(sum, lane);
        const double pq = sum[0], qq = sum[1], rq = sum[2], rr = sum[3];
        // rr = <r, r> of iteration s.iter
        s.rr = rr;
        s.pq = pq;
        // x lacks the last alpha p after an odd number of directions (the
        // launch of an even iteration applies both updates before it)
        if (rr <= s.tol2 * s.bb) {
            s.done = 1;
            s.converged = 1;
            s.pending = s.iter & 1;
        } else if (!(rr == rr)) {
            s.done = 1;
            s.breakdown = 1;
            s.pending = s.iter & 1;
        } else if (s.iter >= s.max_iter) {
            s.done = 1;
            s.pending = s.iter & 1;
        } else if (!(pq > 0.0)) {   // breakdown (or non-finite data)
            s.done = 1;
            s.breakdown = 1;
            s.pending = s.iter & 1;
        } else {
            alpha = rr / pq;
            const double next = fmx(alpha, fmx(alpha, qq, -2.0 * rq), rr);
            beta = next > 0.0 ? next / rr : 0.0;
            s.alpha_prev = s.alpha;
            s.alpha = alpha * sl.unit;
            s.beta = beta;
            s.iter += 1;
        }
    }
    s.first = 0;
    if (b == 0 && threadIdx.x == 0) *sc_out = s;
    if (s.done) return;
    // (the same in every lane: held once)
    alpha = read_lane(alpha, 0);
    beta = read_lane(beta, 0);
    const double ax = read_lane(s.alpha, 0), ax_prev = read_lane(s.alpha_prev, 0);

    const int end = step_wraps(g) ? g.nx - 1 : 64, start = step_wraps(g) ? 0 : 64;
    double fR[N], fL[N];
    // this cell's face scalars to the neighbouring waves and lanes
    auto publish = [&](const double (&u)[N * N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            face[i * 64] = ydot<N>(u, i, k.lR);
            face[(N + i) * 64] = ydot<N>(u, i, lLy);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const double toL = xdot<N>(u, j, k.lR), toR = xdot<N>(u, j, k.lLx);
            fR[j] = lane_next(toL);
            fL[j] = lane_prev(toR);
            if (kWrap) {
                const double first = read_lane(toL, 0), last = read_lane(toR, end & 63);
                if (lane == end) fR[j] = first;
                if (lane == start) fL[j] = last;
            }
        }
    };

    if (first) {
#pragma unroll
        for (int e = 0; e < N * N; ++e) p[e] = r[e];
    } else {
        publish(p);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double fU = face[FR + i * 64], fD = face[-FR + (N + i) * 64];
#pragma unroll
            for (int j = 0; j < N; ++j)
                r[j * N + i] = fmx(alpha, lap_node<N, ISO>(k, sl, p, j, i, fR[j], fL[j], fU, fD),
                                   r[j * N + i]);
        }
#pragma unroll
        for (int e = 0; e < N * N; ++e) p[e] = fmx(beta, p[e], r[e]);
        __syncthreads();
    }
    publish(p);
    if (store) st_l64<N>(rout, self, r);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kStepSums; ++v) sum[v] = 0.0;
    if (inner) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double fU = face[FR + i * 64], fD = face[-FR + (N + i) * 64];
            double a[kStepSums] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const double q = lap_node<N, ISO>(k, sl, p, j, i, fR[j], fL[j], fU, fD);
                const double wq = k.w[j] * q;
                a[0] = fmx(-wq, p[j * N + i], a[0]);
                a[1] = fmx(wq, q, a[1]);
                a[2] = fmx(-wq, r[j * N + i], a[2]);
                a[3] = fmx(k.w[j], r[j * N + i] * r[j * N + i], a[3]);
            }
#pragma unroll
            for (int v = 0; v < kStepSums; ++v) sum[v] = fmx(k.w[i], a[v], sum[v]);
        }
    }
    // x takes the two updates before this iteration at every even one, last,
    // when r is no longer held: p_{k-1} is read again, and p_{k-2} where p_k is
    // stored
    if (store) {
        if (par == 0 && !first) add_to_x<N>(x, pout, pin, self, ax, ax_prev);
        st_l64<N>(pout, self, p);
    }
#pragma unroll
    for (int v = 0; v < kStepSums; ++v) sum[v] = store ? sum[v] * k.wq : 0.0;
    const double mine = row_sums4(sum, lane);
    if ((lane & 15) < kStepSums) lds.red[(wave * 4 + (lane >> 4)) * kStepSums + (lane & 3)] = mine;
    __syncthreads();
    if (wave != 0) return;
    // entries e = lane / 4, + 16, ... of sum lane & 3, then over the lanes
    double tot = 0.0;
#pragma unroll
    for (int u = 0; u < WV * 4; u += 16) tot += lds.red[u * kStepSums + lane];
    tot = add_dpp<0x124>(tot);     // 4 lanes on within 16
    tot = add_dpp<0x128>(tot);     // 8 lanes on
    tot += __shfl_xor(tot, 16);
    tot += __shfl_xor(tot, 32);
    if (nblocks <= kStepDirect) {
        if (lane < kStepSums) part_out[(size_t)kStepSums * b + lane] = tot;
        return;
    }
    // ticket groups (the guarantee relied on is reduce_last's)
    if (lane < kStepSums)
        __hip_atomic_store(&part_out[(size_t)kStepSums * b + lane], tot, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    const int gi = b % kTicketGroups;
    const int gsize = (nblocks - gi + kTicketGroups - 1) / kTicketGroups;
    unsigned* gc = counter + kCntLine * (1 + gi);
    unsigned tk = 0;
    if (lane == 0)
        tk = __hip_atomic_fetch_add(gc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tk = __builtin_amdgcn_readfirstlane(tk);
    if (tk != (unsigned)(gsize - 1)) return;
    double a[kStepSums] = {0.0, 0.0, 0.0, 0.0};
    for (int q = lane; q < gsize; q += 64) {
        const double* v = part_out + (size_t)kStepSums * (gi + (size_t)q * kTicketGroups);
#pragma unroll
        for (int m = 0; m < kStepSums; ++m)
            a[m] += __hip_atomic_load(&v[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    wave_sums4(a, lane);
    if (lane == 0) {
        double* o = part_out + (size_t)kStepSums * nblocks + (size_t)kStepSums * gi;
#pragma unroll
        for (int m = 0; m < kStepSums; ++m) o[m] = a[m];
        __hip_atomic_store(gc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace dgk
