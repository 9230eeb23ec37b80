// Matrix products of the fast-diagonalisation transforms on the matrix cores
// (v_mfma_*_16x16x4): the small and middle sizes, where the library's tiles
// leave most of the chip idle and its launches of both folded halves follow one
// another.  One launch does the products of both halves of a transform (and all
// their batches); a block of four waves computes a tile of 32 x 32, each wave
// 16 x 16, from LDS chunks of 64 of the summed index (registers hold the next
// chunk while this one is multiplied).  What bounds these sizes is the chain of
// chunks -- load, store to LDS, fragments, products -- and how many CUs share
// it, hence the small tiles and the long chunks: the whole inverse of n = 4,
// 255 x 187 cells took 104 us with the library's products and takes 78, n = 3,
// 127 x 127 64 and 36; with walls, n = 3, 128 x 128, 73 and 58.  Chunks of 32 in
// two buffers measured the same, tiles of 64 x 32 were no faster at any size
// that comes here, fragments read a group ahead were slower (86 us).
#include <hip/hip_runtime.h>

#include "dg_launch.h"

namespace dgk {

namespace {

template <class T> struct Frag;
template <> struct Frag<double> {
    using V = double __attribute__((ext_vector_type(4)));
    static __device__ V mma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // row of accumulator r of lane group q = lane / 16
    static __device__ constexpr int row(int r, int q) { return 4 * r + q; }
};
template <> struct Frag<float> {
    using V = float __attribute__((ext_vector_type(4)));
    static __device__ V mma(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ constexpr int row(int r, int q) { return 4 * q + r; }
};

constexpr int kTile = 32, kChunk = 64;
// Every fourth step of the sum has an accumulator of its own: short sums keep the
// rounding below that of one long chain.
constexpr int kSums = 4;

// One operand's chunk, kTile rows by kChunk summed indices.  KF: the operand is
// contiguous along the summed index and kept [row][k]; otherwise contiguous
// along its rows and kept [k][row].  The strides spread a fragment read (16 rows
// x 4 summed indices over the wave) over all banks and keep the stores, which
// follow the contiguous index, in order.
template <class T, bool KF>
struct Operand {
    static constexpr int STRIDE = KF ? kChunk + (sizeof(T) == 8 ? 2 : 4) : kTile + 16;
    static constexpr int SIZE = KF ? kTile * STRIDE : kChunk * STRIDE;
    static constexpr int EACH = kTile * kChunk / 256;   // per thread
    static __device__ int k_of(int e) { return KF ? e % kChunk : e / kTile; }
    static __device__ int row_of(int e) { return KF ? e / kChunk : e % kTile; }
    static __device__ int at(int row, int k) { return KF ? row * STRIDE + k : k * STRIDE + row; }
    // Past the ends the last row and index are read again: a row too many only
    // fills accumulators that are not stored, a summed index too many is set to
    // zero when the chunk is stored to LDS (where the empty asm keeps the
    // compiler from turning the select into a branch with the load in it).
    static __device__ void load(const T* __restrict__ X, long ld, int row0, int rows, int k0, int ks,
                                T (&v)[EACH]) {
#pragma unroll
        for (int u = 0; u < EACH; ++u) {
            const int e = threadIdx.x + 256 * u, k = k0 + k_of(e), r = row0 + row_of(e);
            const int kc = k < ks ? k : ks - 1, rc = r < rows ? r : rows - 1;
            v[u] = X[KF ? kc + rc * ld : rc + kc * ld];
        }
    }
    static __device__ void store(T* lds, int k0, int ks, T (&v)[EACH]) {
#pragma unroll
        for (int u = 0; u < EACH; ++u) {
            const int e = threadIdx.x + 256 * u;
            asm volatile("" : "+v"(v[u]));
            lds[at(row_of(e), k_of(e))] = k0 + k_of(e) < ks ? v[u] : T(0);
        }
    }
};

template <class T, bool AK, bool BK>
__global__ __launch_bounds__(256) void k_gemm_pair(GemmPair<T> g, int batch) {
    using OA = Operand<T, AK>;
    using OB = Operand<T, BK>;
    using V = typename Frag<T>::V;
    __shared__ T la[OA::SIZE], lb[OB::SIZE];
    // tile -> (batch, half, tile of the half), the tiles that share the fields'
    // operand (A when it is transposed, else B) next to each other
    int t = blockIdx.x;
    const int per = gridDim.x / batch;
    const int z = t / per;
    t -= z * per;
    const int tm0 = (g.half[0].m + kTile - 1) / kTile;
    const int tn0 = (g.half[0].n + kTile - 1) / kTile;
    const int hi = t >= tm0 * tn0 ? 1 : 0;
    if (hi) t -= tm0 * tn0;
    const GemmHalf<T>& h = g.half[hi];
    const int tm = (h.m + kTile - 1) / kTile, tn = (h.n + kTile - 1) / kTile;
    const int it = AK ? t / tn : t % tm, jt = AK ? t % tn : t / tm;
    const int m0 = it * kTile, n0 = jt * kTile;
    const T* A = h.A + z * g.sa;
    const T* B = h.B + z * g.sb;
    T* C = h.C + z * g.sc;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l = lane & 15, q = lane >> 4;
    const int wm = (wave & 1) * 16, wn = (wave >> 1) * 16;
    V acc[kSums];
#pragma unroll
    for (int p = 0; p < kSums; ++p) acc[p] = V{0, 0, 0, 0};
    T va[OA::EACH], vb[OB::EACH];
    OA::load(A, g.lda, m0, h.m, 0, h.k, va);
    OB::load(B, g.ldb, n0, h.n, 0, h.k, vb);
    const int chunks = (h.k + kChunk - 1) / kChunk;
    for (int c = 0; c < chunks; ++c) {
        OA::store(la, c * kChunk, h.k, va);
        OB::store(lb, c * kChunk, h.k, vb);
        __syncthreads();
        if (c + 1 < chunks) {
            OA::load(A, g.lda, m0, h.m, (c + 1) * kChunk, h.k, va);
            OB::load(B, g.ldb, n0, h.n, (c + 1) * kChunk, h.k, vb);
        }
#pragma unroll
        for (int k = 0; k < kChunk; k += 4) {
            V& a = acc[k / 4 % kSums];
            a = Frag<T>::mma(lb[OB::at(wn + l, k + q)], la[OA::at(wm + l, k + q)], a);
        }
        __syncthreads();
    }
    // accumulator rows are columns of C, its lanes 16 consecutive rows
    const int m = m0 + wm + l;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = n0 + wn + Frag<T>::row(r, q);
        if (m < h.m && n < h.n)
            C[m + n * g.ldc] = (acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r]);
    }
}

}  // namespace

template <class T>
hipError_t launch_gemm_pair(bool a_trans, bool b_trans, const GemmPair<T>& g, int halves, int batch,
                            hipStream_t s) {
    int tiles = 0;      // an empty half (one cell) has none
    for (int i = 0; i < halves; ++i)
        tiles += ((g.half[i].m + kTile - 1) / kTile) * ((g.half[i].n + kTile - 1) / kTile);
    const dim3 grid((unsigned)(tiles * batch));
#define DG_GEMM(AK, BK) \
    hipLaunchKernelGGL((k_gemm_pair<T, AK, BK>), grid, dim3(256), 0, s, g, batch)
    // op(A) = A^T is contiguous along the summed index, op(B) = B too
    if (a_trans && !b_trans) DG_GEMM(true, true);
    else if (!a_trans && b_trans) DG_GEMM(false, false);
    else if (!a_trans) DG_GEMM(false, true);
    else return hipErrorInvalidValue;
#undef DG_GEMM
    return hipGetLastError();
}

template hipError_t launch_gemm_pair<double>(bool, bool, const GemmPair<double>&, int, int,
                                             hipStream_t);
template hipError_t launch_gemm_pair<float>(bool, bool, const GemmPair<float>&, int, int,
                                            hipStream_t);

}  // namespace dgk
