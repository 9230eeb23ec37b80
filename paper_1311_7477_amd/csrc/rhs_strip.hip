// Fused bracket / right-hand-side kernel of the larger periodic grids: a wave owns
// a strip of up to 62 cells along x (a cell per lane, one halo lane either side)
// and walks up a run of cell rows.  A row's fields come through LDS in order,
// loaded a row ahead into registers; everything else stays in the lanes: x
// neighbours exchange traces by wave rotations, and of the rows above and below a
// cell needs only traces of f, g and b = c2 Dx f g - c1 f Dx g (and of the viscous
// term), which one pass over the next row and the row just left behind provide.
// No barrier, no other wave.
//
// Against the row-per-lane kernel (rhs_body.h), which is bound by LDS (rows
// staged and read back by columns for every y derivative) and computes 1.5 times
// the cells in its halos: bracket n = 5, 2048^2 806 -> 647 us (3.9 TB/s), n = 4,
// 2048^2 456 -> 387, 1024^2 110 -> 101, n = 3, 2048^2 262 -> 195, n = 2, 2048^2 122
// -> 88, n = 1, 2048^2 27 -> 19; with the viscous term and the stage combination
// n = 5, 1024^2 317 -> 253.  What bounds it from n = 4 on is the chain of its vector
// instructions (2550 a row of 62 cells at n = 5, 2400 of them FP64; 1400 at n = 4)
// on one wave per SIMD: a cell's two fields, its sums, the traces and the row ahead
// take 300 - 500 registers.  Counted at n = 5, 2048^2: one is issued in 54% of a
// wave's cycles, most of the rest is the latency between those that need each
// other's results; 2.63 GB moved, 1.05 times the three fields.  A second wave hides
// little more: n = 4 without the row ahead fits two, 2048^2 387 -> 369 us, and then
// spills with the viscous term.
#include "dg_launch.h"
#include "dg_stage.h"

namespace dgk {

namespace {

// The centred derivative is odd under reflection (C0[i][m] = -C0[n-1-i][n-1-m],
// cL[i] = -cR[n-1-i], sL[i] = sR[n-1-i]) and annihilates constants (the sR sum to
// one).  On the sums e_p = u[p] - 2 u[h] + u[n-1-p] and differences o_p = u[p] -
// u[n-1-p] of mirrored values it takes half the products, its traces and face
// terms likewise: with p, i < h = n / 2,
//   res[i], res[n-1-i] = y_i +- x_i,  res[h] = mid . o + cc (fR - fL) for odd n
//   x_i = sum_p xe[i][p] e_p + t[i] (fR - 2 u[h] + fL)
//   y_i = sum_p yo[i][p] o_p + d[i] (fR - fL)
//   sR . u, sL . u = (u[h] + se . e) +- so . o
// Sums of the mirrored values themselves would be rounded at twice the size of a
// field that the derivative then cancels: the bracket of smooth fields was 1.2 (n =
// 2) to 1.5 times (n = 5) as far from the exact one as with plain products.  The
// sums less 2 u[h] are small and rounded at the field's size once, before the last
// addition: 0.85 to 0.95 times as far.
template <int N>
struct Mirror {
    static constexpr int H = N / 2, M = H > 0 ? H : 1;
    double xe[M][M], t[M], yo[M][M], d[M], mid[M], cc, se[M], so[M];
    explicit Mirror(const OpConst<double>& k) {
        for (int i = 0; i < H; ++i) {
            const int r = N - 1 - i;
            for (int p = 0; p < H; ++p) {
                xe[i][p] = 0.5 * (k.C0[i * N + p] + k.C0[i * N + N - 1 - p]);
                yo[i][p] = 0.5 * (k.C0[i * N + p] - k.C0[i * N + N - 1 - p]);
            }
            t[i] = 0.5 * (k.cR[i] - k.cR[r]);
            d[i] = 0.5 * (k.cR[i] + k.cR[r]);
            mid[i] = N % 2 ? k.C0[H * N + i] : 0.0;
            se[i] = 0.5 * (k.sR[i] + k.sR[r]);
            so[i] = 0.5 * (k.sR[i] - k.sR[r]);
        }
        cc = N % 2 ? k.cR[H] : 0.0;
    }
};

template <int N>
__device__ __forceinline__ double c0_times(const OpConst<double>& k, int i, int m, double u,
                                           double a) {
    const int e = i * N + m, r = N * N - 1 - e;
    if (e == r) return a;
    return e < r ? fmx(k.C0[e], u, a) : fmx(-k.C0[r], u, a);
}

template <int N>
__device__ __forceinline__ double c0_faces(const OpConst<double>& k, int i, double hi, double lo) {
    return fmx(k.cR[i], hi, -k.cR[N - 1 - i] * lo);
}

// The centred derivative along x of a node row (times hx)
template <int N>
__device__ __forceinline__ void row_deriv(const Mirror<N>& q, const double (&u)[N],
                                          double (&res)[N]) {
    constexpr int H = N / 2;
    const double c = u[H];
    double e[H + 1], o[H + 1], P = c, Q = 0;
#pragma unroll
    for (int p = 0; p < H; ++p) {
        o[p] = u[p] - u[N - 1 - p];
        e[p] = 2 * p + 2 == N ? o[p] : fmx(-2.0, c, u[p]) + u[N - 1 - p];
    }
#pragma unroll
    for (int p = 0; p < H; ++p) {
        P = fmx(q.se[p], e[p], P);
        Q = p == 0 ? q.so[p] * o[p] : fmx(q.so[p], o[p], Q);
    }
    const double fR = lane_next(P + Q), fL = lane_prev(P - Q);
    const double T = fmx(-2.0, c, fR) + fL, D = fR - fL;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        double x = q.t[i] * T, y = q.d[i] * D;
#pragma unroll
        for (int p = 0; p < H; ++p) {
            x = fmx(q.xe[i][p], e[p], x);
            y = fmx(q.yo[i][p], o[p], y);
        }
        res[i] = y + x;
        res[N - 1 - i] = y - x;
    }
    if (N % 2) {
        double y = q.cc * D;
#pragma unroll
        for (int p = 0; p < H; ++p) y = fmx(q.mid[p], o[p], y);
        res[H] = y;
    }
}

// The second derivative's row (times hx^2)
template <int N>
__device__ __forceinline__ void row_second(const OpConst<double>& k, const double (&u)[N],
                                           double (&res)[N]) {
    double dR = 0, dL = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        dR = fmx(k.lR[m], u[m], dR);
        dL = fmx(k.lLx[m], u[m], dL);
    }
    const double fR = lane_next(dR), fL = lane_prev(dL);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double a = fmx(k.eRx[i], fR, k.eL[i] * fL);
#pragma unroll
        for (int m = 0; m < N; ++m) a = fmx(k.L0x[i * N + m], u[m], a);
        res[i] = a;
    }
}

// Values that have to be there at this point: node rows follow one another
// instead of being interleaved by the compiler, whose temporaries would not fit
// the registers.
template <int M>
__device__ __forceinline__ void pin(double (&u)[M]) {
#pragma unroll
    for (int i = 0; i < M; ++i) asm volatile("" : "+v"(u[i]));
}

// What the cells above and below need of a row of cells
template <int N, bool VISC>
struct Traces {
    double f[N], g[N], b[N], v[VISC ? N : 1];
    __device__ void clear() {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            f[i] = g[i] = b[i] = 0;
            if (VISC) v[i] = 0;
        }
    }
    __device__ void pin() {
        ::dgk::pin(f);
        ::dgk::pin(g);
        ::dgk::pin(b);
        if (VISC) ::dgk::pin(v);
    }
    // node row j's part, weights t (f, g, b) and tv (the viscous term)
    __device__ void add(double t, double tv, const double (&F)[N], const double (&G)[N],
                        const double (&B)[N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            f[i] = fmx(t, F[i], f[i]);
            g[i] = fmx(t, G[i], g[i]);
            b[i] = fmx(t, B[i], b[i]);
            if (VISC) v[i] = fmx(tv, G[i], v[i]);
        }
    }
};

template <int N>
__device__ __forceinline__ void lds_row(const double* cell, int j, double (&u)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = cell[j * N + i];
}

// A row's 64 cells from column x0 - 1 on (periodic), element by element in order
// through the wave's buffers, cells at the stride CS there.
template <int N>
struct Strip {
    int first;      // offset of the first cell from the start of its row
    int total;      // doubles in a row
    bool wraps;     // the run passes an end of the row
};

template <int N>
__device__ __forceinline__ void strip_load(const double* __restrict__ f,
                                           const double* __restrict__ g, const Strip<N>& st,
                                           int lane, double (&vf)[N * N], double (&vg)[N * N]) {
    if (!st.wraps) {
        f += st.first;
        g += st.first;
#pragma unroll
        for (int it = 0; it < N * N; ++it) {
            vf[it] = (f + it * 64)[(unsigned)lane];
            vg[it] = (g + it * 64)[(unsigned)lane];
        }
    } else {
        int first = st.first + lane;
        asm volatile("" : "+v"(first));       // (not kept from row to row)
#pragma unroll
        for (int it = 0; it < N * N; ++it) {
            int o = first + it * 64;
            o = o < 0 ? o + st.total : (o >= st.total ? o - st.total : o);
            const unsigned b = 8u * (unsigned)(o < st.total ? o : st.total - 1);
            vf[it] = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(f) + b);
            vg[it] = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(g) + b);
        }
        asm volatile("");       // (the two ways stay two: the other needs no addresses)
    }
}

template <int N>
__device__ __forceinline__ int strip_at(int it, int lane) {
    constexpr int NN = N * N, CS = Stage<N>::CS;
    return CS == NN ? it * 64 + lane : lane + (CS - NN) * (lane / NN) + it * (64 / NN * CS);
}

template <int N>
__device__ __forceinline__ void strip_put(const double (&v)[N * N], double* buf, int lane) {
#pragma unroll
    for (int it = 0; it < N * N; ++it) buf[strip_at<N>(it, lane)] = v[it];
}

template <int N, bool VISC>
__global__ __launch_bounds__(64, N >= 4 ? 1 : 2) void k_rhs_strip(
    int nx, int ny, int strips, int nblocks, const OpConst<double> k0,
    const Mirror<N> q0,
    const double* __restrict__ f, const double* __restrict__ gg, const double* __restrict__ wn,
    double* __restrict__ out, RhsArgs ra) {
    using S = Stage<N>;
    constexpr int NN = N * N;
    __shared__ double lds[2 * S::SIZE];
    double* const lF = lds;
    double* const lG = lds + S::SIZE;
    const int lane = threadIdx.x;
    const int t = xcd_tile(blockIdx.x, nblocks);
    const int ty = t / strips, tx = t - ty * strips;
    // strips of equal width, rows of equal number
    const int segs = nblocks / strips;
    const auto part = [](int n, int i, int of) {
        return __builtin_amdgcn_readfirstlane((int)((long)n * i / of));
    };
    const int x0 = part(nx, tx, strips), x1 = part(nx, tx + 1, strips);
    const int y0 = part(ny, ty, segs), y1 = part(ny, ty + 1, segs);
    const int w = x1 - x0;
    Strip<N> st;
    st.first = (x0 - 1) * NN;
    st.total = nx * NN;
    st.wraps = x0 == 0 || x0 + 63 > nx;
    const long rowlen = st.total;
    auto row_of = [&](int y) { return (long)(y < 0 ? y + ny : (y >= ny ? y - ny : y)) * rowlen; };

    const double* mF = lF + lane * S::CS;
    const double* mG = lG + lane * S::CS;
    int zero = 0;
    auto fresh = [&](const auto& table) -> const auto& {
        asm volatile("" : "+s"(zero));
        return (&table)[zero];
    };
    const double sb = (VISC ? -ra.scale : ra.scale) * k0.ihy * k0.ihx;      // of the bracket's terms, formed unscaled
    const double dx = VISC ? ra.D * k0.ihx2 : 0.0, dv = VISC ? ra.D * k0.ihy2 : 0.0;

    // the traces of the row of cells in LDS
    auto trace_pass = [&](bool above, Traces<N, VISC>& T) {
        const OpConst<double>& k = fresh(k0);
        const Mirror<N>& q = fresh(q0);
        const double* tv = above ? k.lR : k.lLy;
        T.clear();
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double Fj[N], Gj[N], DxF[N], DxG[N], B[N];
            lds_row<N>(mF, j, Fj);
            lds_row<N>(mG, j, Gj);
            row_deriv<N>(q, Fj, DxF);
            row_deriv<N>(q, Gj, DxG);
#pragma unroll
            for (int i = 0; i < N; ++i) B[i] = fmx(ra.c2 * Gj[i], DxF[i], -(ra.c1 * Fj[i] * DxG[i]));
            T.add(above ? k.sR[j] : k.sR[N - 1 - j], VISC ? tv[j] : 0.0, Fj, Gj, B);
            T.pin();
        }
    };

    double vF[NN], vG[NN];
    double F[NN], G[NN];
    Traces<N, VISC> dn, up;
    strip_load<N>(f + row_of(y0 - 1), gg + row_of(y0 - 1), st, lane, vF, vG);
    wave_lds_fence();
    strip_put<N>(vF, lF, lane);
    strip_put<N>(vG, lG, lane);
    strip_load<N>(f + row_of(y0), gg + row_of(y0), st, lane, vF, vG);
    wave_lds_fence();
    trace_pass(false, dn);
    wave_lds_fence();
    strip_put<N>(vF, lF, lane);
    strip_put<N>(vG, lG, lane);
    strip_load<N>(f + row_of(y0 + 1), gg + row_of(y0 + 1), st, lane, vF, vG);
    wave_lds_fence();
    auto take = [&]() {
        // (the empty asm: read again, not held from the trace pass on)
        int mine = lane * S::CS;
        asm volatile("" : "+v"(mine));
#pragma unroll
        for (int e = 0; e < NN; ++e) {
            F[e] = lF[mine + e];
            G[e] = lG[mine + e];
        }
    };
    take();
    for (int y = y0; y < y1; ++y) {
        wave_lds_fence();
        strip_put<N>(vF, lF, lane);
        strip_put<N>(vG, lG, lane);
        if (y + 1 < y1) {
            strip_load<N>(f + row_of(y + 2), gg + row_of(y + 2), st, lane, vF, vG);
        }
        wave_lds_fence();
        trace_pass(true, up);

        // the row between: acc = the terms of the y derivatives of b (and of the
        // viscous term) from above and below, then node row by node row
        const OpConst<double>& k = fresh(k0);
        const Mirror<N>& q = fresh(q0);
        double acc[NN];
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int i = 0; i < N; ++i) acc[m * N + i] = c0_faces<N>(k, m, up.b[i], dn.b[i]);
        Traces<N, VISC> next;
        next.clear();
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double Fj[N], Gj[N], cF[N], cG[N], DxF[N], DxG[N], B[N], A[N], DxA[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                Fj[i] = F[j * N + i];
                Gj[i] = G[j * N + i];
                cF[i] = ra.c1 * Fj[i];
                cG[i] = ra.c2 * Gj[i];
            }
            row_deriv<N>(q, Fj, DxF);
            row_deriv<N>(q, Gj, DxG);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                B[i] = fmx(cG[i], DxF[i], -(cF[i] * DxG[i]));
                double a = c0_faces<N>(k, j, up.f[i], dn.f[i]);
                double c = c0_faces<N>(k, j, up.g[i], dn.g[i]);
#pragma unroll
                for (int m = 0; m < N; ++m) {
                    a = c0_times<N>(k, j, m, F[m * N + i], a);
                    c = c0_times<N>(k, j, m, G[m * N + i], c);
                }
                A[i] = fmx(cF[i], c, -(a * cG[i]));
                acc[j * N + i] = fmx(ra.c0, fmx(DxF[i], c, -(a * DxG[i])), acc[j * N + i]);
            }
            next.add(k.sR[N - 1 - j], VISC ? k.lLy[j] : 0.0, Fj, Gj, B);
#pragma unroll
            for (int m = 0; m < N; ++m)
#pragma unroll
                for (int i = 0; i < N; ++i)
                    acc[m * N + i] = c0_times<N>(k, m, j, B[i], acc[m * N + i]);
            row_deriv<N>(q, A, DxA);
#pragma unroll
            for (int i = 0; i < N; ++i) acc[j * N + i] += DxA[i];
            next.pin();
            pin(acc);
        }
        if (VISC) {
            // the viscous term, node row by node row
#pragma unroll
            for (int j = 0; j < N; ++j) {
                double Gj[N], Lx[N];
#pragma unroll
                for (int i = 0; i < N; ++i) Gj[i] = G[j * N + i];
                row_second<N>(k, Gj, Lx);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    double a = fmx(k.eRy[j], up.v[i], k.eL[j] * dn.v[i]);
#pragma unroll
                    for (int m = 0; m < N; ++m) a = fmx(k.L0y[j * N + m], G[m * N + i], a);
                    acc[j * N + i] = fmx(dx, Lx[i], fmx(dv, a, sb * acc[j * N + i]));
                }
                pin(acc);
            }
        } else {
#pragma unroll
            for (int e = 0; e < NN; ++e) acc[e] *= sb;
        }
        dn = next;
        if (VISC && !ra.only_r) {
#pragma unroll
            for (int e = 0; e < NN; ++e) acc[e] = ra.b * (G[e] + ra.dt * acc[e]);
        }
        take();                    // row y + 1: the buffers are free
        wave_lds_fence();
        // rows of the strip's own cells, lanes 1 .. w, in order
        double* dst = out + row_of(y) + (long)x0 * NN;
        const double* add = (VISC && !ra.only_r && ra.a != 0.0)
                                ? wn + row_of(y) + (long)x0 * NN
                                : nullptr;
        if (lane >= 1) {
            double* o = lF + (lane - 1) * S::CS;
#pragma unroll
            for (int e = 0; e < NN; ++e) o[e] = acc[e];
        }
        wave_lds_fence();
        const int own = w * NN;
        if (VISC && add) {
#pragma unroll
            for (int it = 0; it < NN; ++it) {
                const int e = it * 64 + lane;
                acc[it] = add[(unsigned)(e < own ? e : own - 1)];
            }
        }
#pragma unroll
        for (int it = 0; it < NN; ++it) {
            if (it * 64 + lane < own) {
                double r = lF[strip_at<N>(it, lane)];
                if (VISC && add) r = fmx(ra.a, acc[it], r);
                (dst + it * 64)[(unsigned)lane] = r;
            }
        }
        wave_lds_fence();
    }
}

}  // namespace

// Waves resident at a time, by order (registers); all strips run in one go.
constexpr int kStripWaves[kMaxN + 1] = {0, 6144, 4096, 2048, 1024, 1024};

int strip_count(const Geom& g) { return (g.nx + 61) / 62; }

// Grids that take strips.  A run begins with two rows that only give traces, so
// short runs lose, and so do strips with idle lanes.  Bracket, rows per lane ->
// strips, us (rows of cells per wave, part of the lanes used):
//   n = 1: 1000^2 (2.8) 9.0 -> 9.3; 1200^2 (3.9) 11.2 -> 9.2; 94 x 18000 (5.9,
//     0.76) 15.1 -> 11.3
//   n = 2: 1024^2 (4.3) 22.4 -> 25.1; 1100^2 (4.8) 27.2 -> 25.9; 1300^2 (6.7) 38.1
//     -> 34.1; 94 x 12492 (6.1, 0.76) 33.8 -> 28.8; 140 x 8328 (6.1, 0.75) 27.7 -> 29.1
//   n = 3: 512^2 (2.3) 18.2 -> 18.6; 700^2 (4.1) 28.6 -> 26.6; 94 x 6246 (6.1, 0.76)
//     39.4 -> 35.9
//   n = 4: 512^2 (4.5) 27.9 -> 32.7; 700^2 (8.2) 47.2 -> 51.3; 800^2 (10.2) 67.3 ->
//     64.6; 1024^2 (17) 110 -> 101; 140 x 3000 (8.8, 0.75) 41.0 -> 49.7; 94 x 20480
//     (40, 0.76) 204 -> 214; 118 x 10240 (20, 0.95) 134 -> 122
//   n = 5: 512^2 (4.5) 52.4 -> 53.4; 600^2 (5.9) 68.0 -> 63.2; 1024^2 (17) 206 ->
//     183; 94 x 5120 (10, 0.76) 101 -> 103; 94 x 10240 (20, 0.76) 195 -> 185
// From n = 4 on, where both kernels are bound by arithmetic, the line is one of
// cost: a wave's rows and the two before them against 5/4 (n = 4) or 3/2 (n = 5)
// of the rows that its cells would fill.
bool rhs_strips(const Geom& g) {
    if (g.bcx || g.bcy || (long)g.nx * g.n * g.n >= 1L << 28) return false;
    const long strips = strip_count(g), waves = kStripWaves[g.n];
    const long rows = strips * g.ny;
    if (strips > waves) return false;
    if (g.n >= 4) {
        const long cost = 62 * (rows + 2 * waves), cells = (long)g.nx * g.ny;
        return g.n == 4 ? 4 * cost < 5 * cells : 2 * cost < 3 * cells;
    }
    return 4L * g.nx >= 3 * 62 * strips && rows >= (g.n == 2 ? 5 : 4) * waves;
}

hipError_t launch_rhs_strip(const Geom& g, const OpConst<double>& k, const double* f,
                            const double* gg, const double* wn, double* out, const RhsArgs& ra,
                            bool visc, hipStream_t s) {
    const int strips = strip_count(g);
    const int nblocks = strips * (kStripWaves[g.n] / strips);
    if (visc) {
        DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_rhs_strip<NN, true>), dim3(nblocks), dim3(64), 0,
                                              s, g.nx, g.ny, strips, nblocks, k, Mirror<NN>(k), f, gg, wn, out,
                                              ra));
    } else {
        DG_DISPATCH_N(g.n, hipLaunchKernelGGL((k_rhs_strip<NN, false>), dim3(nblocks), dim3(64), 0,
                                              s, g.nx, g.ny, strips, nblocks, k, Mirror<NN>(k), f, gg, wn, out,
                                              ra));
    }
    return hipGetLastError();
}

}  // namespace dgk
