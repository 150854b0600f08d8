// Matrix-core step and index arithmetic shared by the any-shape kernels (mask_generic_impl.h, attn_generic_impl.h).
#pragma once
#include "common.h"

namespace hipattn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 gen_bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float gen_f32x4;

// acc += A B for one 16-byte chunk per lane: 16 fp32 or 32 bf16 channels of 16 rows each
template <typename T> __device__ __forceinline__ gen_f32x4 mfma_chunk(const uint4 &a, const uint4 &b, gen_f32x4 acc);
template <> __device__ __forceinline__ gen_f32x4 mfma_chunk<float>(const uint4 &a, const uint4 &b, gen_f32x4 acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ gen_f32x4 mfma_chunk<bf16_t>(const uint4 &a, const uint4 &b, gen_f32x4 acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(gen_bf16x8, a), __builtin_bit_cast(gen_bf16x8, b), acc, 0, 0, 0);
}

// fp32 operands as three bf16 planes (high, middle, low: 8 significand bits each, every remainder rounded to nearest), so
// that a product runs at the bf16 rate, 16 times the fp32 one.  x = h + m + l exactly down to 2^-110; below, bits under 2^-133 are
// lost: the kernels do in fp32 what comes out small enough for that to show, and query rows that reach further (QueryReach).  Six of the nine products are formed; the ones
// left out (m l, l m, l l) are below 2^-25 of the product, half an ulp of fp32 being 2^-24.  A part of an infinite value, or
// of one that rounds up to infinity, is NaN: so is what it is multiplied into, and the kernels do that again too.
// Error of 128-channel products against 64 bits, over the sum of the products' magnitudes, rms / largest: fp32 instruction 2.8e-8 /
// 2.7e-7, planes 0.9e-8 / 1.0e-7 (normal operands); 8.2e-8 / 6.0e-7 and 6.1e-8 / 4.6e-7 (magnitudes over 2^-20 to 2^20).
struct Planes { uint32_t h, m, l; };  // of two values
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 pair_t;
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f2_t;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2_t{a, b}), pair_t));
}
__device__ __forceinline__ Planes split_planes(float a, float b)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 pair_t;
    // (the remainder as one dot product with (-1, 0) or (0, -1): exact, and nothing to unpack.  The two constants are kept in
    // registers: as a literal, 0xbf800000 is encoded as the inline constant -1.0, which this instruction does not read as a pair.)
    uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
    asm("" : "+s"(c0));
    asm("" : "+s"(c1));
    const pair_t m0 = __builtin_bit_cast(pair_t, c0), m1 = __builtin_bit_cast(pair_t, c1);
    const auto rest = [&](uint32_t plane) __attribute__((always_inline)) {
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(pair_t, plane), m0, a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(pair_t, plane), m1, b, false);
    };
    Planes p;
    p.h = pack_bf16(a, b);
    rest(p.h);
    p.m = pack_bf16(a, b);
    rest(p.m);
    p.l = pack_bf16(a, b);
    return p;
}
// the planes of eight channels of a lane: operands of one 16x16x32 step
struct Planes8 { uint4 h, m, l; };
__device__ __forceinline__ Planes8 split_planes8(const uint4 &a, const uint4 &b)
{
    const Planes x = split_planes(__uint_as_float(a.x), __uint_as_float(a.y)), y = split_planes(__uint_as_float(a.z), __uint_as_float(a.w));
    const Planes z = split_planes(__uint_as_float(b.x), __uint_as_float(b.y)), w = split_planes(__uint_as_float(b.z), __uint_as_float(b.w));
    return Planes8{make_uint4(x.h, y.h, z.h, w.h), make_uint4(x.m, y.m, z.m, w.m), make_uint4(x.l, y.l, z.l, w.l)};
}
// How far the values of a query row reach: their largest magnitude, and whether one that is not 0 has lost bits to the planes' range
// (what such a value is multiplied with may be large enough for that to show, whatever the product's size).
struct QueryReach {
    uint32_t largest = 0u, smallest = ~0u;  // bits of the magnitude; twice those less one, which takes 0 out
    __device__ __forceinline__ void add(const uint4 &x)
    {
        largest = max(max(largest, max(x.x & 0x7fffffffu, x.y & 0x7fffffffu)), max(x.z & 0x7fffffffu, x.w & 0x7fffffffu));
        smallest = min(min(smallest, min((x.x << 1) - 1u, (x.y << 1) - 1u)), min((x.z << 1) - 1u, (x.w << 1) - 1u));
    }
    __device__ __forceinline__ bool loses_bits() const { return smallest < ((127u - 110u) << 24) - 1u; }
};
// hi += the products of the high planes, lo += the five smaller ones: kept apart, so that adding a small one does not round
// the large sum.  One operand against N, so that 2 N sums take turns on the matrix pipe; ONE_IS_A: it is the rows of the result.
template <bool ONE_IS_A, int N>
__device__ __forceinline__ void mfma_planes(const Planes8 &one, const Planes8 (&many)[N], gen_f32x4 (&hi)[N], gen_f32x4 (&lo)[N])
{
    const auto add = [](const uint4 &x, const uint4 &y, gen_f32x4 &to) __attribute__((always_inline)) {
        to = ONE_IS_A ? mfma_chunk<bf16_t>(x, y, to) : mfma_chunk<bf16_t>(y, x, to);
    };
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.h, many[i].l, lo[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.h, many[i].h, hi[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.h, many[i].m, lo[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.m, many[i].m, lo[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.m, many[i].h, lo[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) add(one.l, many[i].h, lo[i]);
}
// (by bits that the compiler knows nothing of: it may assume that no float is a NaN)
__device__ __forceinline__ bool not_finite(float x)
{
    uint32_t u = __float_as_uint(x);
    asm volatile("" : "+v"(u));
    return (u & 0x7f800000u) == 0x7f800000u;
}

// n / d for 0 <= n < 2^16, 1 <= d <= 16, with m = div_magic(d)
inline uint32_t div_magic(int d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / (uint32_t)d + 1); }
__device__ __forceinline__ int div_small(int n, uint32_t m) { return (int)__umulhi((uint32_t)n, m) + (n & (m ? 0 : -1)); }

}  // namespace hipattn
