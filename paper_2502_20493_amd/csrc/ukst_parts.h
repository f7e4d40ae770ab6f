// fp32 operands on the bf16 matrix pipe: an fp32 value is the exact sum of three bf16 parts
// (24 significant bits = 3 x 8; each part is the remainder rounded to nearest even), so
//     x*w = x0*w0 + (x0*w1 + x1*w0) + (x1*w1 + x0*w2 + x2*w0) + [x1*w2 + x2*w1 + x2*w2]
// and the six products outside the bracket, each exact in fp32 and summed in fp32 by the MFMA, leave
// out less than 2^-25 of a product.  v_mfma_f32_32x32x16_bf16 multiplies 16 times as fast as
// v_mfma_f32_32x32x2_f32, so six of them per 16 channels take 6/16 of the time of the fp32 pipe, and
// the sum is rounded 6 times per 16 channels instead of 8.  Measured against 64-bit sums the error is
// below that of the fp32 pipe (128 channels x 25 taps: see the kernels that use this).
//
// The parts hold what the value holds only while no part under- or overflows: operands that are
// infinite, NaN, at least 2^62 or below 2^-100 (but not 0) are noticed while they are staged, and the
// block that met one computes its tile again with fp32 multiply-adds.
// (128 -> 128 channels, 64 x 64, n = 5: 574 us; 530 with the minimum of the leading parts, which counts
// values below 2^-134 as 0 and is not used for that; 580 with a class test per value.)
#pragma once
#include "ukst_internal.h"

namespace ukst {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u4v_t __attribute__((ext_vector_type(4)));
typedef unsigned u2v_t __attribute__((ext_vector_type(2)));
typedef unsigned short us2_t __attribute__((ext_vector_type(2)));

constexpr int kRawBuffer = 0x00020000;        // raw 32-bit buffer, gfx9 family
constexpr unsigned kNoByte = 0xFFFFFF00u;     // byte offset that is out of range for any buffer

// What a thread has staged: the largest leading part (two lanes of 16 bits) and the smallest fp32 magnitude but 0 (its
// bits without the sign, less 1, so that zeros wrap around to the top).  The smallest is taken from the values and
// not from the leading parts: a value below 2^-134 has leading part 0 and would be lost among the zeros.
struct PartRange {
    us2_t hi = {0, 0};
    unsigned lo = 0xFFFFFFFFu;
    __device__ __forceinline__ void see_parts(unsigned p0)
    {
        hi = __builtin_elementwise_max(hi, __builtin_bit_cast(us2_t, p0 & 0x7FFF7FFFu));
    }
    __device__ __forceinline__ void see_values(float a, float b)
    {
        const unsigned ua = (__float_as_uint(a) << 1) - 1u, ub = (__float_as_uint(b) << 1) - 1u;
        const unsigned m = ua < ub ? ua : ub;
        lo = lo < m ? lo : m;
    }
    __device__ __forceinline__ bool bad() const
    {
        constexpr unsigned short top = (127 + 62) << 7;
        constexpr unsigned bottom = ((unsigned)(127 - 100) << 24) - 1u;
        return hi.x >= top || hi.y >= top || lo < bottom;
    }
    // an infinity or NaN alone (operands that are bf16 already)
    __device__ __forceinline__ bool not_finite() const { return hi.x >= 0x7F80 || hi.y >= 0x7F80; }
};

__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    const bf16x2_t p = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned, p);
}

// three bf16 parts of a pair of values, packed (a in the low half)
__device__ __forceinline__ void split_pair(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2,
                                           PartRange& seen)
{
    seen.see_values(a, b);
    p0 = pack_bf16(a, b);
    seen.see_parts(p0);
    a -= __uint_as_float(p0 << 16);
    b -= __uint_as_float(p0 & 0xFFFF0000u);
    p1 = pack_bf16(a, b);
    a -= __uint_as_float(p1 << 16);
    b -= __uint_as_float(p1 & 0xFFFF0000u);
    p2 = pack_bf16(a, b);
}

// 8 consecutive K values (raw dwords as loaded; bf16 operands: one value per dword) -> PARTS vectors
// of 8 bf16, the layout of one MFMA operand lane
template <int PARTS>
__device__ __forceinline__ void to_parts(const unsigned (&v)[8], u4v_t (&out)[PARTS], PartRange& seen)
{
    if constexpr (PARTS == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[0][i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], 0x05040100u);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned p0, p1, p2;
            split_pair(__uint_as_float(v[2 * i]), __uint_as_float(v[2 * i + 1]), p0, p1, p2, seen);
            out[0][i] = p0;
            out[1][i] = p1;
            out[2][i] = p2;
        }
    }
}

// the products of two operands' parts that are multiplied, smallest first
template <int PARTS>
struct PartProducts;
template <>
struct PartProducts<1> {
    static constexpr int count = 1;
    static constexpr int a[1] = {0}, b[1] = {0};
};
template <>
struct PartProducts<3> {
    static constexpr int count = 6;
    static constexpr int a[6] = {2, 0, 1, 1, 0, 0}, b[6] = {0, 2, 1, 0, 1, 0};
};

template <typename T>
__device__ __forceinline__ unsigned load_element(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff)
{
    if constexpr (sizeof(T) == 2)
        return (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rs, voff, soff, 0);
    else
        return __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0);
}
__device__ __forceinline__ float element_f32(float v) { return v; }
__device__ __forceinline__ float element_f32(uint16_t v) { return __uint_as_float((unsigned)v << 16); }

}  // namespace ukst
