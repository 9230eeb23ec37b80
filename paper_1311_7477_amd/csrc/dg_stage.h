// Canonical fields through LDS: a wave's 64 consecutive cells are one
// contiguous run of 64 n^2 doubles, which the wave moves 16 bytes a lane in
// order and hands to its lanes, one cell each, through a buffer of its own
// (no barrier).  Each lane reading its own cell instead makes every load
// instruction touch 64 lines of 128 bytes for 8 or 16 bytes each.
#pragma once

#include "dg_device.h"

namespace dgk {

// Two doubles at any address a double may have (the public fields are only
// 8-byte aligned; a 16-byte access needs no more than 4 on this target).
struct Double2u {
    double x, y;
};

// LDS layout: a cell's n^2 values at a stride that spreads the lanes' 16-byte
// (even n: n^2 + 2 doubles) or 8-byte (odd n: n^2) accesses over all banks.
template <int N>
struct Stage {
    static constexpr int NN = N * N;
    static constexpr bool kPairs = NN % 2 == 0;
    static constexpr int CS = kPairs ? NN + 2 : NN;
    static constexpr int SIZE = 64 * CS;            // doubles per wave (even)
    static constexpr int ITER = (64 * NN / 2 + 63) / 64;
    // LDS place of pair q of the run
    __device__ static constexpr int at(int q) {
        return kPairs ? q / (NN / 2) * CS + 2 * (q % (NN / 2)) : 2 * q;
    }
};

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The run of `count` cells at src as it lies, `it` after `it`; every lane of
// the wave takes part.
template <int N>
__device__ __forceinline__ void stage_load(const double* __restrict__ src, int count, int lane,
                                           Double2u (&v)[Stage<N>::ITER]) {
    using S = Stage<N>;
    const int total = count * S::NN;
    if (count == 64) {
#pragma unroll
        for (int it = 0; it < S::ITER; ++it) {
            const int q = it * 64 + lane;
            v[it].x = v[it].y = 0.0;
            if (2 * 64 * (it + 1) <= 64 * S::NN || 2 * q < 64 * S::NN)
                v[it] = *reinterpret_cast<const Double2u*>(src + 2 * q);
        }
        return;
    }
#pragma unroll
    for (int it = 0; it < S::ITER; ++it) {
        const int q = it * 64 + lane;
        v[it].x = v[it].y = 0.0;
        if (2 * q + 1 < total) v[it] = *reinterpret_cast<const Double2u*>(src + 2 * q);
        else if (2 * q < total) v[it].x = src[2 * q];
    }
}

// The run to the lanes: u = the values of cell `lane` (zeros past the run).
template <int N>
__device__ __forceinline__ void stage_spread(const Double2u (&v)[Stage<N>::ITER], double* buf,
                                             int lane, double (&u)[N * N]) {
    using S = Stage<N>;
    wave_lds_fence();      // earlier reads of the buffer
#pragma unroll
    for (int it = 0; it < S::ITER; ++it) {
        const int q = it * 64 + lane;
        if (2 * 64 * (it + 1) <= 64 * S::NN || 2 * q < 64 * S::NN)
            *reinterpret_cast<double2*>(buf + S::at(q)) = make_double2(v[it].x, v[it].y);
    }
    wave_lds_fence();
    const double* mine = buf + lane * S::CS;
    if constexpr (S::kPairs) {
#pragma unroll
        for (int e = 0; e < S::NN; e += 2) {
            const double2 w = *reinterpret_cast<const double2*>(mine + e);
            u[e] = w.x;
            u[e + 1] = w.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < S::NN; ++e) u[e] = mine[e];
    }
}

template <int N>
__device__ __forceinline__ void stage_in(const double* __restrict__ src, int count, double* buf,
                                         int lane, double (&u)[N * N]) {
    Double2u v[Stage<N>::ITER];
    stage_load<N>(src, count, lane, v);
    stage_spread<N>(v, buf, lane, u);
}

// The reverse: the cells of lanes 0 .. count - 1 to the contiguous run at dst.
template <int N>
__device__ __forceinline__ void stage_out(double* __restrict__ dst, int count, double* buf, int lane,
                                          const double (&u)[N * N]) {
    using S = Stage<N>;
    wave_lds_fence();
    double* mine = buf + lane * S::CS;
    if constexpr (S::kPairs) {
#pragma unroll
        for (int e = 0; e < S::NN; e += 2)
            *reinterpret_cast<double2*>(mine + e) = make_double2(u[e], u[e + 1]);
    } else {
#pragma unroll
        for (int e = 0; e < S::NN; ++e) mine[e] = u[e];
    }
    wave_lds_fence();
    const int total = count * S::NN;
#pragma unroll
    for (int it = 0; it < S::ITER; ++it) {
        const int q = it * 64 + lane;
        if (2 * q >= total) continue;
        const double2 w = *reinterpret_cast<const double2*>(buf + S::at(q));
        if (2 * q + 1 < total) {
            Double2u o;
            o.x = w.x;
            o.y = w.y;
            *reinterpret_cast<Double2u*>(dst + 2 * q) = o;
        } else {
            dst[2 * q] = w.x;
        }
    }
}

}  // namespace dgk
