// Device-side helpers shared by the GEMM and GEMV kernel templates.
#pragma once

#include <hip/hip_runtime.h>
#include "internal.h"

namespace nnjit {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Workgroups of one dispatch are handed to the 8 XCDs of the chip in turn
// (flat id 0 -> XCD 0, 1 -> XCD 1, ...), and each XCD has its own L2.  This
// renumbering makes ids that are consecutive in the new numbering run on the
// same XCD, so tiles that share operand rows or columns share an L2.  It is a
// bijection of [0, G) for any G.
__device__ __forceinline__ int xcd_remap(int flat, int G) {
    const int q = G >> 3, r = G & 7;
    const int xcd = flat & 7, local = flat >> 3;
    return (xcd < r) ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
}

// Tile of a GEMM launch from its index in the (XCD-renumbered) order: tiles
// run in groups of G tile rows, each group column by column (G rows of one
// tile column, then the next column), so that the run of consecutive tiles an
// XCD holds at once covers about G rows and (run / G) columns of tiles -- A
// rows and B columns that the XCD's L2 shares -- instead of one whole column
// of tiles, which makes every XCD read all of A.  G = tiles_m is the plain
// column-major order.  A bijection of [0, tiles_m * tiles_n).
__device__ __forceinline__ void tile_of(int tile, int tiles_m, int tiles_n, int G, int &tm, int &tn)
{
    const int span = G * tiles_n;
    const int g = tile / span, local = tile - g * span;
    const int rows = min(G, tiles_m - g * G);
    tm = g * G + local % rows;
    tn = local / rows;
}

// 16 bytes from an address aligned to an element only (gfx950 takes 128-bit
// global loads at any address).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned short u16x8u __attribute__((ext_vector_type(8), aligned(2)));
__device__ __forceinline__ u32x4 load8_any(const unsigned short *src)
{
    return __builtin_bit_cast(u32x4, *(const u16x8u *)src);
}

// Rows of B from which a chunk of up to 8 elements that begins before column N
// can be read whole: it may run on into the next row (which no stored output
// uses), but behind the last rows it would leave the operand.  The bound of a
// K range [.., kend) below which every chunk of A and B can be read unchecked.
__device__ __forceinline__ int unaligned_safe_k(const GemmParams &p, int kend)
{
    if ((p.N & 7) == 0) return kend;
    return min(kend, p.K - (p.ldb >= 7 ? 1 : 7));
}

// Wait until at most N vector memory operations of this wave are pending.
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N <= 63, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// 16 bytes per lane from global memory to LDS: lane l's bytes land at LDS
// address lds + 16 l (lds must be wave-uniform).  Issued as inline assembly
// so that the compiler does not treat the copy as an LDS store of unknown
// target and wait for every copy in flight before each LDS read; the kernel
// orders the copies against the reads itself (counted vmcnt waits plus a
// barrier).  Vector memory loads complete in issue order, so the compiler's
// own vmcnt waits stay correct with these extra loads in the queue.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is written on purpose
__device__ __forceinline__ void copy16_to_lds(const void *src, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop

// Workgroup barrier for the copy pipeline: this wave's LDS reads are complete
// and every wave has arrived.  Global memory ordering is not needed here (the
// copies are waited for by count), so unlike __syncthreads() it does not
// wait for all outstanding vector memory operations.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

struct Split8 {
    bf16x8 h, m, l;
};

// An fp32 product on the bf16 matrix cores: each operand is split, exactly,
// into three bf16 parts x = h + m + l (8 + 8 + 8 significand bits, each
// rounded to nearest even), and the product is taken as the six part products
//     hl + lh + mm + hm + mh + hh,
// summed in fp32 (v_mfma_f32_32x32x16_bf16).  |m| is at most 2^-8 and |l| at
// most 2^-17 of the operand's power of two, so the three dropped products are
// together at most 2^-24 of |a b| (nearly reached by a = b = 1.0038986): half an
// ulp, one fp32 rounding of the product, of the same sign for equal operands.
// Random operands: see the errors against fp64 in gemm_staged.hip.
//
// Two kinds of operands do not survive the split, and the kernels take the sums
// they reach anew on the fp32 matrix cores, straight from memory:
//   - one that is not finite or rounds to a bf16 infinity (its parts do not add
//     up to it), or a sum that overflows: the sum is then left not finite for
//     good, so it is enough to test the sums once, at the end;
//   - one below 2^-110 but not zero (tiny): its last bits are below the
//     smallest bf16 subnormal, 2^-133 (conversion and matrix cores keep
//     subnormals), and what they lose, up to 2^-134, counts times the other
//     operand.  If no operand is above 2^32, K products lose at most K 2^-101,
//     half of what the K roundings of an fp32 sum of at least 2^-76 may take;
//     so tiny operands are looked for, with a second pass over the operands,
//     only where a sum is below 2^-76 or an operand above 2^32.  A sum of a row
//     of A or column of B that has a tiny one is then taken anew if it is below
//     2^-76 or the tile has an operand above 2^32.  Sums of a peaked softmax's
//     weights times ordinary values thus cost nothing, and zero sums of zero
//     rows or columns the second pass.
//
// The second pass takes the smallest magnitude in as (bits << 1) - 1: zeros wrap
// to the largest.  (The bits are taken of a scalar: of an element of a vector,
// __builtin_bit_cast takes those of the first one.)
constexpr unsigned kTinyStart = 0xffffffffu;
constexpr unsigned kTinyLimit = (17u << 24) - 1u;   // 2^-110
constexpr float kTinySum = 0x1p-76f;
constexpr float kTinyMeets = 0x1p32f;
__device__ __forceinline__ unsigned least_of(unsigned least, float x)
{
    return min(least, (__builtin_bit_cast(unsigned, x) << 1) - 1u);
}

// Eight fp32 values as three bf16 parts each (exact: x = h + m + l while h is
// finite and x zero or at least 2^-110); `top` takes their largest magnitude
// in.  12 instructions per pair: three v_cvt_pk_bf16_f32, per remainder two
// unpacks and two subtractions, and a v_max3_f32.
__device__ __forceinline__ Split8 split8(f32x8 x, float &top)
{
    u32x4 h, m, l;
    auto parts = [](float a, float b, float &ra, float &rb) -> unsigned {
        const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
        ra = a - __builtin_bit_cast(float, u << 16);
        rb = b - __builtin_bit_cast(float, u & 0xffff0000u);
        return u;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float r0, r1, s0, s1, z0, z1;
        h[q] = parts(x[2 * q], x[2 * q + 1], r0, r1);
        m[q] = parts(r0, r1, s0, s1);
        l[q] = parts(s0, s1, z0, z1);
        top = fmaxf(fmaxf(fabsf(x[2 * q]), fabsf(x[2 * q + 1])), top);
    }
    return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

__device__ __forceinline__ f32x16 mma_bf16(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

}  // namespace nnjit
