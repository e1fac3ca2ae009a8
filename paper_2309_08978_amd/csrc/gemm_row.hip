// Products of single rows: C[z][i][n] = sum_k A[z][i][k] B[z][k][n], one
// workgroup per row i, column segment, K split and batch slice.  A BatchMatMul
// with M = 1 is what attention does in a decode step (one query per head
// against its cache); a matrix-core tile would spend 31 of its 32 rows on
// padding and leave the chip with one workgroup per 32 columns.
//
// Bandwidth-bound like the GEMV: L lanes span a segment of L * V consecutive
// columns (V = 16 bytes of elements), the workgroup's other lanes are row
// slots of B, and each lane keeps U 128-bit loads in flight.  The loads are
// taken from any element address (gfx950 allows it), so operands of any
// alignment run the same code; a lane whose V columns would pass column N is
// moved back to the last V and stores only the columns that are its own.
//
// Reduction over k in a fixed order: row slots of a wave (butterfly), waves
// (through LDS, in order), splits (a second kernel, as for the GEMM tiles).
#include "kcommon.h"

namespace nnjit {

template <typename T> struct RowT;
template <> struct RowT<float> {
    static constexpr int V = 4;
    struct raw { f32x4u v; };
    __device__ static __forceinline__ raw load(const float *p) { return raw{*(const f32x4u *)p}; }
    __device__ static __forceinline__ float get(const raw &r, int e) { return r.v[e]; }
    __device__ static __forceinline__ void set(raw &r, int e, float x) { r.v[e] = x; }
};
template <> struct RowT<_Float16> {
    typedef _Float16 f16x8u __attribute__((ext_vector_type(8), aligned(2)));
    static constexpr int V = 8;
    struct raw { f16x8u v; };
    __device__ static __forceinline__ raw load(const _Float16 *p) { return raw{*(const f16x8u *)p}; }
    __device__ static __forceinline__ float get(const raw &r, int e) { return (float)r.v[e]; }
    __device__ static __forceinline__ void set(raw &r, int e, _Float16 x) { r.v[e] = x; }
};

template <typename T, int L, int NTHR, int U>
__global__ void __launch_bounds__(NTHR)
gemm_row_kernel(GemmParams p)
{
    typedef RowT<T> O;
    constexpr int V = O::V;
    constexpr int CW = L * V;         // columns per workgroup
    constexpr int R = NTHR / L;       // row slots per workgroup
    constexpr int NW = NTHR / 64;
    static_assert(NTHR % 64 == 0 && 64 % L == 0, "layout");

    const int tid = threadIdx.x;
    const int c = tid % L, rs = tid / L;
    const int tiles = p.tiles_m * p.tiles_n;
    const int gx = gridDim.x;
    const int logical = xcd_remap(blockIdx.x + gx * blockIdx.z, gx * gridDim.z);
    const int z = logical / gx;
    const int rest = logical - z * gx;
    const int s = rest / tiles;
    const int tile = rest - s * tiles;
    int tm, tn;
    tile_of(tile, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const int N = p.N;
    const int kbeg = s * p.kchunk;
    const int kend = min(p.K, kbeg + p.kchunk);
    const int n = tn * CW + c * V;               // first column of this lane
    const bool live = n < N;
    const int nl = max(0, min(n, N - V));         // where its loads begin

    const T *x = (const T *)p.A + (long long)z * p.sA + (long long)tm * p.lda;
    const T *B = (const T *)p.B + (long long)z * p.sB + nl;
    auto bload = [&](int k) {
        const T *src = B + (long long)k * p.ldb;
        if (N >= V) return O::load(src);
        typename O::raw r;                        // fewer columns than one load
#pragma unroll
        for (int e = 0; e < V; ++e) O::set(r, e, src[min(e, N - 1)]);
        return r;
    };

    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (live) {
        int k = kbeg + rs;
        for (; k + (U - 1) * R < kend; k += U * R) {
            typename O::raw w[U];
            T xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = bload(k + u * R);
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = x[k + u * R];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] = __builtin_fmaf((float)xv[u], O::get(w[u], e), acc[e]);
        }
        if (k < kend) {
            // the last rows: rows past the end are read again from the last
            // one, all loads in flight together, and left out of the sum
            typename O::raw w[U];
            T xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = bload(min(k + u * R, kend - 1));
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = x[min(k + u * R, kend - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u * R < kend)
#pragma unroll
                    for (int e = 0; e < V; ++e) acc[e] = __builtin_fmaf((float)xv[u], O::get(w[u], e), acc[e]);
        }
    }

#pragma unroll
    for (int off = L; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
    if constexpr (NW > 1) {
        __shared__ float red[NW][L][V];
        const int wave = tid >> 6, lane = tid & 63;
        if (lane < L)
#pragma unroll
            for (int e = 0; e < V; ++e) red[wave][lane][e] = acc[e];
        __syncthreads();
        if (tid < L) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                float v = red[0][tid][e];
#pragma unroll
                for (int w = 1; w < NW; ++w) v += red[w][tid][e];
                acc[e] = v;
            }
        }
    }
    if (tid >= L || !live) return;
    float *out = p.S > 1 ? p.ws + (((long long)s * p.batch + z) * p.M + tm) * (long long)N
                         : p.C + (long long)z * p.sC + (long long)tm * p.ldc;
#pragma unroll
    for (int e = 0; e < V; ++e)
        if (nl + e >= n && nl + e < N) out[nl + e] = acc[e];
}

template <typename T, int L, int NTHR, int U>
static hipError_t launch_gemm_row(const void *params, dim3 grid, hipStream_t stream)
{
    hipLaunchKernelGGL((gemm_row_kernel<T, L, NTHR, U>), grid, dim3(NTHR), 0, stream, *(const GemmParams *)params);
    return hipGetLastError();
}

constexpr int est_regs_row(int v, int u) { return v + 5 * u + 28; }
#define NNJIT_ROW_VARIANT(T, FAM, TAG, V, L, NTHR, U)                                                     \
    {"gemm_" TAG "r_L" #L "_t" #NTHR "_u" #U, FAM, 0, 0, 1, L * V, NTHR / L, 1, NTHR / 64, 1, 1, 1,       \
     (int)sizeof(T), L, U, NTHR, (NTHR / 64) * L * V * 4, est_regs_row(V, U),                             \
     (const void *)&gemm_row_kernel<T, L, NTHR, U>, &launch_gemm_row<T, L, NTHR, U>, 0, LAYOUT_PLAIN, 0}

#define NNJIT_F32R_LIST(X) \
    X(8, 256, 8) \
    X(16, 256, 8) \
    X(32, 256, 8) \
    X(64, 256, 8) \
    X(8, 1024, 8) \
    X(16, 1024, 8)
#define NNJIT_F16R_LIST(X) \
    X(4, 256, 8) \
    X(8, 256, 8) \
    X(16, 256, 8) \
    X(32, 256, 8) \
    X(4, 1024, 8) \
    X(8, 1024, 8)

#define NNJIT_F32R_INST(L, NTHR, U) template __global__ void gemm_row_kernel<float, L, NTHR, U>(GemmParams);
#define NNJIT_F16R_INST(L, NTHR, U) template __global__ void gemm_row_kernel<_Float16, L, NTHR, U>(GemmParams);
NNJIT_F32R_LIST(NNJIT_F32R_INST)
NNJIT_F16R_LIST(NNJIT_F16R_INST)

#if !defined(__HIP_DEVICE_COMPILE__)
#define NNJIT_F32R_ENTRY(L, NTHR, U) NNJIT_ROW_VARIANT(float, FAM_GEMM_F32, "f32", 4, L, NTHR, U),
#define NNJIT_F16R_ENTRY(L, NTHR, U) NNJIT_ROW_VARIANT(_Float16, FAM_GEMM_F16, "f16", 8, L, NTHR, U),
const Variant kGemmF32rVariants[] = {NNJIT_F32R_LIST(NNJIT_F32R_ENTRY)};
const int kNumGemmF32rVariants = sizeof(kGemmF32rVariants) / sizeof(kGemmF32rVariants[0]);
const Variant kGemmF16rVariants[] = {NNJIT_F16R_LIST(NNJIT_F16R_ENTRY)};
const int kNumGemmF16rVariants = sizeof(kGemmF16rVariants) / sizeof(kGemmF16rVariants[0]);
#endif

}  // namespace nnjit
