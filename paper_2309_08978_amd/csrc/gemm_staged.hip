// fp32 MatMul / BatchMatMul on the bf16 matrix cores ("gemm_f32s"), the
// operands split in three bf16 parts (see split8 in kcommon.h).
//
// Why: the fp32 matrix-core instructions run at 157 TFLOP/s dense and the
// fp32 kernels were at 82-90% of that; six bf16 products per fp32 product run
// at up to 2517 / 6 = 419 TFLOP/s.  The sums are no less accurate: against
// fp64 the relative error (2-norm) of 512 x 32000 x 4096 is 1.0e-6 where the
// fp32 instructions give 1.1e-6, of 1024 x 4096 x 1024 4.9e-7 against 5.7e-7,
// of 256 x 256 x 64 1.1e-7 against 1.4e-7 (16 terms are summed per rounding
// instead of two).
//
// One workgroup computes an Mt x Nt tile for one split of K and one batch
// slice.  Each operand element is loaded into registers once per workgroup,
// split there and stored to LDS as three bf16 planes, so the split costs
// (Mt + Nt) / (Mt Nt) of what splitting each wave's fragments would (that
// form, with fp32 slabs copied straight to LDS, measured the same on 512 x
// 32000 x 4096 but 2-4% slower from 1024 x 4096 x 1024 down).  Three LDS
// stages: slab k is multiplied, k + 1 is visible, k + 2 is being stored, and
// PF more slabs are on their way in registers; one barrier per slab.
//   A plane [Mt rows][Kt halves], 16-byte chunk c of row r at c ^ ((r >> 3) & 1)
//     (Kt = 16) or c ^ ((r >> 2) & 3) (Kt = 32): 16 rows read at one chunk
//     cover the 64 banks once;
//   B plane [Kt k rows][Nt halves] read through ds_read_b64_tr_b16, as in
//     gemm_f16t: the 32-byte unit u of row k at u ^ b_swz(k).
// SQ_LDS_BANK_CONFLICT is 0.
//
// Measured (random operands, one MI355X): 512 x 32000 x 4096, 256 x 256 tiles:
// 947 -> 590-640 us (142 -> 210-228 TFLOP/s, 1.26-1.37 PFLOP/s of bf16 products);
// 1024 x 4096 x 1024, 128 x 128 tiles: 67 -> 49-53 us; 512 x 4096 x 11008:
// 335 -> 218 us.  The large tiles run at the power limit: on zero operands the
// first took 509 us (and now pays the second pass, 665).  Eight waves beat four (one per SIMD) except where LDS
// holds several workgroups.
//
// VEC false: operands of any alignment.  gfx950 loads 16 bytes at any element
// address, so the same 128-bit loads serve; only a slab that reaches past the
// K range or behind the last rows of B takes element loads.
#include "kcommon.h"

namespace nnjit {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

// Operand types of the staged kernel: how eight elements are loaded, and the
// planes of eight halves they become.
template <typename T> struct Staged;
template <> struct Staged<float> {
    static constexpr int PL = 3;            // bf16 planes
    struct raw { f32x4 v[2]; };
    template <bool VEC> __device__ static __forceinline__ raw load(const float *src)
    {
        if constexpr (VEC) return raw{{*(const f32x4 *)src, *(const f32x4 *)(src + 4)}};
        else return raw{{*(const f32x4u *)src, *(const f32x4u *)(src + 4)}};
    }
    // the first `have` elements, the others zero (`zero`: 16 zero bytes; only
    // units that are partly in range load element by element)
    template <bool VEC> __device__ static __forceinline__ raw load_part(const float *src, int have, const float *zero)
    {
        if constexpr (VEC) return raw{{*(const f32x4 *)(have > 0 ? src : zero), *(const f32x4 *)(have > 4 ? src + 4 : zero)}};
        raw r = raw{{*(const f32x4u *)(have >= 8 ? src : zero), *(const f32x4u *)(have >= 8 ? src + 4 : zero)}};
        if (have > 0 && have < 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) r.v[e / 4][e % 4] = *(e < have ? src + e : zero);
        }
        return r;
    }
    __device__ static __forceinline__ void planes(const raw &r, u32x4 (&out)[3], float &top)
    {
        const Split8 v = split8(__builtin_shufflevector(r.v[0], r.v[1], 0, 1, 2, 3, 4, 5, 6, 7), top);
        out[0] = __builtin_bit_cast(u32x4, v.h);
        out[1] = __builtin_bit_cast(u32x4, v.m);
        out[2] = __builtin_bit_cast(u32x4, v.l);
    }
    __device__ static __forceinline__ unsigned least(unsigned least, const raw &r)
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) least = least_of(least, r.v[e / 4][e % 4]);
        return least;
    }
    __device__ static __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
    {
        return mma_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
    }
};
template <> struct Staged<unsigned short> {   // fp16 bits
    static constexpr int PL = 1;
    struct raw { u32x4 v; };
    template <bool VEC> __device__ static __forceinline__ raw load(const unsigned short *src)
    {
        if constexpr (VEC) return raw{*(const u32x4 *)src};
        else return raw{load8_any(src)};
    }
    template <bool VEC>
    __device__ static __forceinline__ raw load_part(const unsigned short *src, int have, const unsigned short *zero)
    {
        if constexpr (VEC) return raw{*(const u32x4 *)(have > 0 ? src : zero)};
        raw r = raw{load8_any(have >= 8 ? src : zero)};
        if (have > 0 && have < 8) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned lo = *(2 * w < have ? src + 2 * w : zero), hi = *(2 * w + 1 < have ? src + 2 * w + 1 : zero);
                r.v[w] = lo | (hi << 16);
            }
        }
        return r;
    }
    __device__ static __forceinline__ void planes(const raw &r, u32x4 (&out)[1], float &) { out[0] = r.v; }
    __device__ static __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

template <typename T, int MT, int NT, int KT, int WM, int WN, int PF, bool VEC>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_staged_kernel(GemmParams p)
{
    typedef Staged<T> O;
    constexpr int PL = O::PL;
    typedef f32x16 acc_t;
    constexpr int ST = 3;
    constexpr int NTHR = WM * WN * 64;
    constexpr int WTM = MT / WM, WTN = NT / WN;
    constexpr int FM = WTM / 32, FN = WTN / 32;
    constexpr int ACH = KT / 8;                      // 8-element units per A row of a slab
    constexpr int AU = MT * ACH, BU = KT * NT / 8;   // units of one slab
    constexpr int NU = AU + BU;
    constexpr int LU = (NU + NTHR - 1) / NTHR;       // units per thread
    constexpr int APL = AU * 16, BPL = BU * 16;      // bytes of one plane
    constexpr int STAGE = PL * (APL + BPL);
    constexpr int NSTEP = KT / 16;                   // matrix-core K steps per slab
    // Split products: where a slab's conversions stand.  Behind its products, the
    // slabs kept apart in the schedule, against before them: 512 x 4096 x 4096 on
    // 128 x 128 tiles 144 and 157 us, on 256 x 128 251 and 268; not on the largest
    // wave tile (512 x 11008 x 4096: 492 and 444), nor on 64 x 64 tiles of any
    // alignment (333 x 1000 x 777: 20.0 and 19.5).
    constexpr bool LATE = PL == 3 && FM * FN < 8 && (VEC || FM * FN > 1);
    static_assert(KT == 16 || KT == 32 || KT == 64, "K slab");
    static_assert(AU % 64 == 0 && BU % 64 == 0, "a wave's units are of one operand");
    static_assert(NT >= 64 && (NT & (NT - 1)) == 0, "B rows of a power of two >= 64");
    static_assert(PF == 1 || PF == ST, "staging sets");
    static_assert(FM >= 1 && FN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile");

    __shared__ __attribute__((aligned(1024))) char smem[ST * STAGE];
    typedef __attribute__((address_space(3))) char lds_char;

    const int tiles = p.tiles_m * p.tiles_n;
    const int gx = gridDim.x;
    const int logical = xcd_remap(blockIdx.x + gx * blockIdx.z, gx * gridDim.z);
    const int M = p.M, N = p.N;
    const long long lda = p.lda, ldb = p.ldb;
    const T *zero = (const T *)p.zero;

    auto a_swz = [](int row) { return KT == 16 ? ((row >> 3) & 1) : KT == 32 ? ((row >> 2) & 3) : ((row >> 1) & 7); };
    auto b_swz = [](int k) { return NT >= 128 ? (((k & 3) << 1) | ((k >> 3) & 1)) : (((k >> 1) & 1) << 1); };

    const int z = logical / gx;
    const int rest = logical - z * gx;
    const int s = rest / tiles;
    const int tile = rest - s * tiles;
    const int kbeg = s * p.kchunk;
    const int kend = min(p.K, kbeg + p.kchunk);
    int tm, tn;
    tile_of(tile, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const int m0 = tm * MT, n0 = tn * NT;
    const int nk = kend > kbeg ? (kend - kbeg + KT - 1) / KT : 0;
    const T *A = (const T *)p.A + (long long)z * p.sA;
    const T *B = (const T *)p.B + (long long)z * p.sB;
    float *C = p.C + (long long)z * p.sC;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int li = lane & 31, lg = lane >> 5;
    // unit u of this wave: of A, of B, or none (the last round may be short)
    auto unit_of_a = [&](int u) { return wave_u * 64 + u * NTHR < AU; };
    auto unit_live = [&](int u) { return NU % NTHR == 0 || u + 1 < LU || wave_u * 64 + u * NTHR < NU; };

    // This thread's units: 8 consecutive k of an A row, or 8 consecutive
    // columns of a B row (which of the two is the same for a whole wave).
    // Rows past M and units past N point at row / column 0: what they bring
    // reaches only outputs that are never stored.
    const T *u_src[LU];
    int u_dst[LU];
#pragma unroll
    for (int u = 0; u < LU; ++u) {
        const int f = tid + u * NTHR;
        if (unit_of_a(u)) {
            const int row = f / ACH, c = f % ACH;
            u_src[u] = A + (long long)(m0 + row < M ? m0 + row : 0) * lda + kbeg + 8 * c;
            u_dst[u] = row * (KT * 2) + 16 * (c ^ a_swz(row));
        } else {
            const int g = f - AU;
            const int k = g / (NT / 8), c = g % (NT / 8);
            u_src[u] = B + (long long)(kbeg + k) * ldb + (n0 + 8 * c < N ? n0 + 8 * c : 0);
            u_dst[u] = PL * APL + k * (NT * 2) + 32 * ((c >> 1) ^ b_swz(k)) + 16 * (c & 1);
        }
    }
    // whole slabs whose units can be read without checks
    const int safe_k = unaligned_safe_k(p, kend);
    const int nfull = safe_k > kbeg ? (safe_k - kbeg) / KT : 0;

    // The 128-row wave tile has no register to spare for the addresses of each
    // stage: its stage offset goes through an opaque scalar, so that they are
    // formed where they are used.
    auto stage_base = [&](int stage) -> lds_char * {
        unsigned off = stage * STAGE;
        if constexpr (FM >= 4 && PL == 3) asm volatile("" : "+s"(off));
        return (lds_char *)smem + off;
    };

    typename O::raw st[PF][LU];
    float top = 0.f;   // the largest operand this thread split
    auto load_full = [&](typename O::raw (&dst)[LU], int kk) {
#pragma unroll
        for (int u = 0; u < LU; ++u) {
            if (!unit_live(u)) continue;
            const bool is_a = unit_of_a(u);
            const T *src = u_src[u] + (is_a ? (long long)(kk * KT) : (long long)(kk * KT) * ldb);
            dst[u] = O::template load<VEC>(src);
        }
    };
    // a slab that reaches past the K range or the last column: elements out
    // of range are read from the zero buffer (only the address is selected)
    auto load_checked = [&](typename O::raw (&dst)[LU], int kk) {
        // indices taken afresh from an opaque copy of the thread id, so that
        // they are not held in registers across the loop over the slabs
        int t = tid;
        asm volatile("v_mov_b32 %0, %0" : "+v"(t));
#pragma unroll
        for (int u = 0; u < LU; ++u) {
            if (!unit_live(u)) continue;
            const int f = t + u * NTHR;
            const bool is_a = unit_of_a(u);
            const T *src = u_src[u] + (is_a ? (long long)(kk * KT) : (long long)(kk * KT) * ldb);
            int have;   // elements of the unit in range
            if (is_a) {
                have = kend - (kbeg + kk * KT + 8 * (f % ACH));
            } else {
                const int g = f - AU;
                const int n = n0 + 8 * (g % (NT / 8));
                have = kbeg + kk * KT + g / (NT / 8) < kend ? (n < N ? N - n : 8) : 0;
                if (n >= N && N < 8) have = min(have, N);
            }
            dst[u] = O::template load_part<VEC>(src, have, zero);
        }
    };
    auto load_units = [&](typename O::raw (&dst)[LU], int kk) {
        if (kk < nfull) load_full(dst, kk);
        else if (kk < nk) load_checked(dst, kk);
    };
    auto load_slab = [&](int set, int kk) { load_units(st[set], kk); };
    auto store_slab = [&](int set, int stage) {
        lds_char *base = stage_base(stage);
#pragma unroll
        for (int u = 0; u < LU; ++u) {
            if (!unit_live(u)) continue;
            const int pl = unit_of_a(u) ? APL : BPL;
            u32x4 v[PL];
            O::planes(st[set][u], v, top);
#pragma unroll
            for (int q = 0; q < PL; ++q) *(lds_u32x4 *)(base + u_dst[u] + q * pl) = v[q];
        }
    };

    acc_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int grp = lane >> 4, tr_r = (lane >> 2) & 3, tr_q = lane & 3;
    const int tr_n = 16 * (grp & 1) + 4 * tr_q;
    struct AFrag { u32x4 p[PL]; };
    auto read_a = [&](int stage, int step, int i) -> AFrag {
        const int row = wm * WTM + 32 * i + li;
        lds_char *a = stage_base(stage) + row * (KT * 2) + 16 * ((2 * step + lg) ^ a_swz(row));
        AFrag f;
#pragma unroll
        for (int q = 0; q < PL; ++q) f.p[q] = *(lds_u32x4 *)(a + q * APL);
        return f;
    };
    auto read_b = [&](int stage, int step, int j, int pl) -> u32x4 {
        const int n = wn * WTN + 32 * j + tr_n;
        s16x4 h[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int k = 16 * step + 8 * (grp >> 1) + 4 * hh + tr_r;
            lds_char *b = stage_base(stage) + PL * APL + pl * BPL + k * (NT * 2) +
                          32 * ((n >> 4) ^ b_swz(k)) + 2 * (n & 15);
            h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)b);
        }
        return __builtin_bit_cast(u32x4, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // fragments of B of one K step (three planes: h, m, l)
    u32x4 b[PL][FN];
    auto mma_part = [&](int i, const u32x4 &x, int part) {
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = O::mma(x, b[part][j], acc[i][j]);
    };

    if (nk > 0) {
        // slabs 0 and 1 into LDS, slabs 2 .. PF + 1 on their way (a set that
        // was not loaded is not split: `top` sees operands only)
        if constexpr (PF == 1) {
            load_slab(0, 0);
            store_slab(0, 0);
            load_slab(0, 1);
            if (nk > 1) store_slab(0, 1);
            load_slab(0, 2);
        } else {
            load_slab(0, 0);
            load_slab(1, 1);
            load_slab(2, 2);
            store_slab(0, 0);
            load_slab(0, 3);
            if (nk > 1) store_slab(1, 1);
            load_slab(1, 4);
        }
        lds_barrier();
        AFrag a = read_a(0, 0, 0);
        auto read_b_part = [&](int stage, int step, int part) {
#pragma unroll
            for (int j = 0; j < FN; ++j) b[part][j] = read_b(stage, step, j, part);
        };
        for (int part = PL - 1; part >= 0; --part) read_b_part(0, 0, part);
        // the products of the slab in stage u.  The next row's A fragments are
        // read while this row's products run; the last row reads the next
        // step's (or the next slab's) first ones, and each part of B again as
        // soon as its last product is issued (so B needs one register set).
        auto compute = [&](int u) {
#pragma unroll
            for (int q = 0; q < NSTEP; ++q)
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    const bool last_row = i + 1 == FM, last = last_row && q + 1 == NSTEP;
                    const int stage = last ? (u + 1) % ST : u, step = last_row ? (q + 1) % NSTEP : q;
                    const AFrag an = read_a(stage, step, last_row ? 0 : i + 1);
                    if constexpr (PL == 3) {
                        mma_part(i, a.p[0], 2);
                        if (last_row) read_b_part(stage, step, 2);
                        mma_part(i, a.p[0], 1);
                        mma_part(i, a.p[1], 1);
                        if (last_row) read_b_part(stage, step, 1);
                        mma_part(i, a.p[2], 0);
                        mma_part(i, a.p[1], 0);
                        mma_part(i, a.p[0], 0);
                        if (last_row) read_b_part(stage, step, 0);
                    } else {
                        u32x4 bn[FN];
                        if (last_row)
#pragma unroll
                            for (int j = 0; j < FN; ++j) bn[j] = read_b(stage, step, j, 0);
                        mma_part(i, a.p[0], 0);
                        if (last_row)
#pragma unroll
                            for (int j = 0; j < FN; ++j) b[0][j] = bn[j];
                    }
                    a = an;
                    // keep the 128-row wave tile within its registers: no
                    // fragment read is moved up past a row of products
                    if constexpr (FM >= 4 && PL == 3) __builtin_amdgcn_sched_barrier(0);
                }
        };
        int it0 = 0;
        // while every slab loaded is whole: one branch-free block per slab
        for (; it0 + ST + 2 + PF <= nfull; it0 += ST) {
#pragma unroll
            for (int u = 0; u < ST; ++u) {
                const int set = PF == 1 ? 0 : (u + 2) % ST;
                if constexpr (LATE) {
                    __builtin_amdgcn_sched_barrier(0);
                    compute(u);
                }
                store_slab(set, (u + 2) % ST);
                load_full(st[set], it0 + u + 2 + PF);
                if constexpr (!LATE) compute(u);
                lds_barrier();
            }
        }
        for (; it0 < nk; it0 += ST) {
#pragma unroll
            for (int u = 0; u < ST; ++u) {
                const int set = PF == 1 ? 0 : (u + 2) % ST;
                if (it0 + u + 2 < nk) store_slab(set, (u + 2) % ST);
                load_slab(set, it0 + u + 2 + PF);
                if (it0 + u < nk) compute(u);
                lds_barrier();
            }
        }
    }

    const int rwave = wm * WTM, cwave = wn * WTN + li;
    auto row_of = [&](int r) { return 8 * (r >> 2) + 4 * lg + (r & 3); };

    float *out = C + (long long)m0 * p.ldc + n0;
    long long ldo = p.ldc;
    const int rows = M - m0, cols = N - n0;
    if (p.S > 1) {
        out = p.ws + (((long long)s * p.batch + z) * (long long)M + m0) * N + n0;
        ldo = N;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = rwave + 32 * i + row_of(r), col = cwave + 32 * j;
                if (row < rows && col < cols) out[(long long)row * ldo + col] = acc[i][j][r];
            }

    if constexpr (PL == 3) {
        // sums that the split does not serve are taken anew in fp32 (kcommon.h)
        // and stored over the others; only those, so that a sum's bits follow from
        // its own row and column.  1024 x 4096 x 1024 (128 x 128 tiles), 512 x 32000 x
        // 4096 (256 x 256): 53 and 625 us; with a row of zeros in every fragment,
        // which costs the second pass, 80 and 835; with a row of infinities in
        // every fragment 315 and 3300.
        float probe = 0.f;
        bool low = false;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            float least = kTinySum;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    probe = __builtin_fmaf(acc[i][j][r], 0.f, probe);
                    least = fminf(least, fabsf(acc[i][j][r]));
                }
            low = low || (least < kTinySum && cwave + 32 * j < cols);
        }
        // (opaque copies: else the conditions of the stores above are kept in
        // scalar registers, more than there are)
        int mrows = rows, mcols = cols;
        asm volatile("" : "+s"(mrows), "+s"(mcols));
        if (mrows < MT && __any(low)) {   // rows past M do not count
            low = false;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                float least = kTinySum;
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        least = fminf(least, rwave + 32 * i + row_of(r) < mrows ? fabsf(acc[i][j][r]) : kTinySum);
                low = low || (least < kTinySum && cwave + 32 * j < mcols);
            }
        }
        const bool open = __syncthreads_or(low || top > kTinyMeets);
        if (open || __any(!(probe == 0.f))) {
            // in LDS: rows of A, groups of 8 columns of B that have a tiny operand;
            // is there a large one
            typedef __attribute__((address_space(3))) int lds_int;
            lds_int *tiny_row = (lds_int *)smem, *tiny_grp = tiny_row + MT, *large = tiny_grp + NT / 8;
            if (open) {
                for (int t = tid; t < MT + NT / 8 + 1; t += NTHR) tiny_row[t] = 0;
                __syncthreads();
                if (top > kTinyMeets) *large = 1;
                // the second pass: the units of SC slabs at a time
                unsigned least[LU];
#pragma unroll
                for (int u = 0; u < LU; ++u) least[u] = kTinyStart;
                constexpr int SC = FM >= 4 ? 2 : 1;   // (as many as leave the main loop its registers)
                for (int kk = 0; kk < nk; kk += SC) {
                    typename O::raw x[SC][LU];
#pragma unroll
                    for (int q = 0; q < SC; ++q) load_units(x[q], min(kk + q, nk - 1));
#pragma unroll
                    for (int q = 0; q < SC; ++q)
#pragma unroll
                        for (int u = 0; u < LU; ++u)
                            if (unit_live(u)) least[u] = O::least(least[u], x[q][u]);
                }
#pragma unroll
                for (int u = 0; u < LU; ++u) {
                    const int f = tid + u * NTHR;
                    if (least[u] >= kTinyLimit) continue;
                    if (unit_of_a(u)) tiny_row[f / ACH] = 1;
                    else tiny_grp[(f - AU) % (NT / 8)] = 1;
                }
                __syncthreads();
            }
            unsigned need[FM][FN], some = 0;   // bit r: sum r is taken anew
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const int col = cwave + 32 * j;
                    const bool tg = open && tiny_grp[col >> 3], meets = open && *large;
                    need[i][j] = 0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = rwave + 32 * i + row_of(r);
                        const float v = fabsf(acc[i][j][r]);
                        const bool tiny = tg || (open && tiny_row[row]);
                        if (!(v < __builtin_inff()) || (tiny && (meets || v < kTinySum)))
                            if (row < mrows && col < mcols) need[i][j] |= 1u << r;
                    }
                    some |= need[i][j];
                }
            if (__any(some != 0)) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
                for (int k = kbeg; k < kend; k += 2) {
                    const int gk = k + lg;
                    float a[FM], b[FN];
#pragma unroll
                    for (int i = 0; i < FM; ++i) {
                        const int gm = m0 + rwave + 32 * i + li;
                        a[i] = *((gm < M && gk < kend) ? A + (long long)gm * lda + gk : zero);
                    }
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        const int gn = n0 + cwave + 32 * j;
                        b[j] = *((gn < N && gk < kend) ? B + (long long)gk * ldb + gn : zero);
                    }
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if ((need[i][j] >> r) & 1)
                                out[(long long)(rwave + 32 * i + row_of(r)) * ldo + cwave + 32 * j] = acc[i][j][r];
            }
        }
    }
}

template <typename T, int MT, int NT, int KT, int WM, int WN, int PF, bool VEC>
static hipError_t launch_gemm_staged(const void *params, dim3 grid, hipStream_t stream)
{
    hipLaunchKernelGGL((gemm_staged_kernel<T, MT, NT, KT, WM, WN, PF, VEC>), grid, dim3(WM * WN * 64), 0, stream,
                       *(const GemmParams *)params);
    return hipGetLastError();
}

// accumulators, two A and one or two sets of B fragments (4 registers per
// plane each), the staging registers and a fixed overhead
constexpr int est_regs_staged(int pl, int mt, int nt, int kt, int wm, int wn, int pf) {
    return (mt / wm) * (nt / wn) / 64 + 4 * pl * (2 + 2 * (nt / wn) / 32) +
           (pf + 1) * (mt + nt) * kt * (pl == 3 ? 2 : 1) / 2 / (wm * wn * 64) + 32;
}
// three stages of the planes; with three planes also the flag of the
// workgroup-wide test
constexpr int lds_staged(int pl, int mt, int nt, int kt) { return 6 * pl * kt * (mt + nt) + (pl == 3 ? 256 : 0); }
#define NNJIT_F32S_VARIANT(MT, NT, KT, WM, WN, PF, VEC)                                                       \
    {"gemm_f32s_" #MT "x" #NT "x" #KT "_w" #WM "x" #WN "_p" #PF "_v" #VEC, FAM_GEMM_F32, 32, 16, MT, NT, KT, WM, WN, 3, PF, \
     1, (VEC ? 16 : 4), 0, 0, WM * WN * 64, lds_staged(3, MT, NT, KT), est_regs_staged(3, MT, NT, KT, WM, WN, PF), \
     (const void *)&gemm_staged_kernel<float, MT, NT, KT, WM, WN, PF, VEC>,                                   \
     &launch_gemm_staged<float, MT, NT, KT, WM, WN, PF, VEC>, 2, LAYOUT_SWIZZLE, 0}
#define NNJIT_F16S_VARIANT(MT, NT, KT, WM, WN, PF, VEC)                                                       \
    {"gemm_f16s_" #MT "x" #NT "x" #KT "_w" #WM "x" #WN "_p" #PF "_v" #VEC, FAM_GEMM_F16, 32, 16, MT, NT, KT, WM, WN, 3, PF, \
     1, (VEC ? 16 : 2), 0, 0, WM * WN * 64, lds_staged(1, MT, NT, KT), est_regs_staged(1, MT, NT, KT, WM, WN, PF), \
     (const void *)&gemm_staged_kernel<unsigned short, MT, NT, KT, WM, WN, PF, VEC>,                          \
     &launch_gemm_staged<unsigned short, MT, NT, KT, WM, WN, PF, VEC>, 2, LAYOUT_SWIZZLE, 0}

#define NNJIT_F32S_LIST(X) \
    X(256, 256, 16, 2, 4, 1, true) \
    X(256, 128, 16, 4, 2, 3, true) \
    X(128, 256, 16, 2, 4, 3, true) \
    X(128, 128, 16, 2, 4, 3, true) \
    X(64, 64, 16, 2, 2, 3, true) \
    X(128, 128, 16, 2, 4, 3, false) \
    X(64, 64, 16, 2, 2, 3, false)

// fp16: what the tuner registers it for are small products (64 slices
// of 43 x 80 x 64 3.9 us, direct-copy tiles 4.2; of 128 x 128 x 64 4.3 and 4.6;
// with a split 128 x 768 x 3072), three sets in flight for some of them.  Larger
// aligned tiles are gemm_f16t's (512 x 4096 x 4096: 26, the same tile staged
// here 35; over 60 shapes no 128 x 128 or larger one was registered).
#define NNJIT_F16S_LIST(X) \
    X(64, 64, 64, 2, 2, 1, true) \
    X(64, 64, 64, 2, 2, 3, true) \
    X(128, 128, 32, 2, 4, 1, false) \
    X(64, 64, 32, 2, 2, 3, false)

#define NNJIT_F32S_INST(...) template __global__ void gemm_staged_kernel<float, __VA_ARGS__>(GemmParams);
#define NNJIT_F16S_INST(...) template __global__ void gemm_staged_kernel<unsigned short, __VA_ARGS__>(GemmParams);
NNJIT_F32S_LIST(NNJIT_F32S_INST)
NNJIT_F16S_LIST(NNJIT_F16S_INST)

#if !defined(__HIP_DEVICE_COMPILE__)
#define NNJIT_F32S_ENTRY(...) NNJIT_F32S_VARIANT(__VA_ARGS__),
const Variant kGemmF32sVariants[] = {NNJIT_F32S_LIST(NNJIT_F32S_ENTRY)};
const int kNumGemmF32sVariants = sizeof(kGemmF32sVariants) / sizeof(kGemmF32sVariants[0]);
#define NNJIT_F16S_ENTRY(...) NNJIT_F16S_VARIANT(__VA_ARGS__),
const Variant kGemmF16sVariants[] = {NNJIT_F16S_LIST(NNJIT_F16S_ENTRY)};
const int kNumGemmF16sVariants = sizeof(kGemmF16sVariants) / sizeof(kGemmF16sVariants[0]);
#endif

}  // namespace nnjit
