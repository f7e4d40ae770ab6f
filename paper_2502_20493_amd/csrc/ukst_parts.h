// fp32 operands on the bf16 matrix pipe: an fp32 value is the exact sum of three bf16 parts
// (24 significant bits = 3 x 8; each part is the remainder rounded to nearest even), so
//     x*w = x0*w0 + (x0*w1 + x1*w0) + (x1*w1 + x0*w2 + x2*w0) + [x1*w2 + x2*w1 + x2*w2]
// and the six products outside the bracket, each exact in fp32 and summed in fp32 by the MFMA, leave
// out at most about 2^-24 of a product, half a unit in its last place (|x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|:
// x = w = 1 + 2^-8 - 2^-17 comes to 1.98 * 2^-25).  v_mfma_f32_32x32x16_bf16 multiplies 16 times as fast as
// v_mfma_f32_32x32x2_f32, so six of them per 16 channels take 6/16 of the time of the fp32 pipe, and
// the sum is rounded 6 times per 16 channels instead of 8.  Measured against 64-bit sums the error is
// below that of the fp32 pipe (128 channels x 25 taps: see the kernels that use this).
//
// The parts hold what the value holds only while none of them under- or overflows.  Values are multiplied by
// 2^24 before they are split, which makes the last bit of the smallest denormal, 2^-149, a normal bf16 value:
// nothing underflows, and the sums, 2^48 times too large, are scaled back (and rounded to a denormal, if it is
// one) at the store.  Operands from 2^104 and sums from 2^80 on overflow and leave an infinity or NaN in every
// sum they belong to.  A block that finds one takes the 32 x 32 tiles of sums that hold one again, from memory
// on the fp32 pipe.  Sums that are not finite then either and whose window reaches into the halo, whose zeros have no
// part in the sum but make NaN of an infinite operand, are listed and taken with fp32 multiply-adds, four per thread.
// (32 x 128 -> 128 channels, 64 x 64, n = 5: 531 us with one multiplication per value; 585 with a test of every value's
// range, which took whole blocks again, 14.6 ms, for one weight of 1e-35 in 64 channels.  Every tile again, operands of
// 1e15: 2.0 ms, fp32 pipe 0.89.)
#pragma once
#include "ukst_internal.h"

namespace ukst {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u4v_t __attribute__((ext_vector_type(4)));
typedef unsigned u2v_t __attribute__((ext_vector_type(2)));

constexpr int kRawBuffer = 0x00020000;        // raw 32-bit buffer, gfx9 family
constexpr unsigned kNoByte = 0xFFFFFF00u;     // byte offset that is out of range for any buffer

constexpr float kPartsUp = 0x1p24f, kPartsDown = 0x1p-48f;  // of an operand, of a sum of products

__device__ __forceinline__ bool group_bad(const f32x16_t& v, int g)  // of registers 4*g .. 4*g + 3
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(v[4 * g + i], 0.f, s);
    return s != s;
}
// largest magnitude of m and v, NaN if there is one (one v_maximum3_f32 per pair)
__device__ __forceinline__ float peak(const f32x16_t& v, float m)
{
#pragma unroll
    for (int i = 0; i < 16; i += 2)
        m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(v[i])), fabsf(v[i + 1]));
    return m;
}
__device__ __forceinline__ bool wave_finite(const f32x16_t& v)  // uniform
{
    return __builtin_amdgcn_ballot_w64(!(peak(v, 0.f) < __builtin_inff())) == 0;
}
__device__ __forceinline__ bool all_nan(const float (&s)[4])
{
    return s[0] != s[0] && s[1] != s[1] && s[2] != s[2] && s[3] != s[3];
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    const bf16x2_t p = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned, p);
}

// three bf16 parts of a pair of values (times 2^24), packed (a in the low half)
__device__ __forceinline__ void split_pair(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2)
{
    a *= kPartsUp;
    b *= kPartsUp;
    p0 = pack_bf16(a, b);
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
__device__ __forceinline__ void to_parts(const unsigned (&v)[8], u4v_t (&out)[PARTS])
{
    if constexpr (PARTS == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[0][i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], 0x05040100u);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned p0, p1, p2;
            split_pair(__uint_as_float(v[2 * i]), __uint_as_float(v[2 * i + 1]), p0, p1, p2);
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
template <typename T>
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff)
{
    return __uint_as_float(load_element<T>(rs, voff, soff) << (sizeof(T) == 2 ? 16 : 0));
}
__device__ __forceinline__ bool wave_nan(const f32x16_t& v)  // every sum (uniform): nothing is left to add then
{
    bool nan = true;
#pragma unroll
    for (int i = 0; i < 16; ++i) nan = nan && v[i] != v[i];
    return __builtin_amdgcn_ballot_w64(!nan) == 0;
}
// acc[k] += the products of NB 32 x 32 tiles that share their rows, over c = c0 .. c1 - 1, on the fp32 pipe.  Byte
// offsets of the lane's row (a) and columns (b) for c = 0, kNoByte where there is none; astep and bstep from one c to
// the next
template <typename T, int NB>
__device__ __forceinline__ void sum_tiles(f32x16_t (&acc)[NB], __amdgpu_buffer_rsrc_t rs_a, unsigned ao, unsigned astep,
                                          __amdgpu_buffer_rsrc_t rs_b, const unsigned (&bo)[NB], unsigned bstep, int c0,
                                          int c1)
{
    const int gk = (threadIdx.x & 63) >> 5;
    for (int cb = c0; cb < c1; cb += 16) {
        bool nan = true;
#pragma unroll
        for (int k = 0; k < NB; ++k) nan = nan && wave_nan(acc[k]);
        if (nan) return;
        float a[8], b[NB][8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = cb + 2 * i;
            const bool in = c + gk < c1;
            a[i] = load_f32<T>(rs_a, in ? ao + gk * astep : kNoByte, c * astep);
#pragma unroll
            for (int k = 0; k < NB; ++k)
                b[k][i] = load_f32<T>(rs_b, in && bo[k] != kNoByte ? bo[k] + gk * bstep : kNoByte, c * bstep);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < NB; ++k) acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[k][i], acc[k], 0, 0, 0);
    }
}
// put(register, value) for all sixteen; list: group(g), of registers 4*g .. 4*g + 3, is listed in LDS if one of them is
// not finite: a count, then 16-bit group numbers in no particular order, redo_bytes of at most `groups` of them
constexpr size_t redo_bytes(int groups) { return 16 + 2 * (size_t)groups; }
template <typename Put, typename Group>
__device__ __forceinline__ void put_tile(unsigned char* lds, const f32x16_t& v, bool list, Put put, Group group)
{
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int i = 4 * g; i < 4 * g + 4; ++i) put(i, v[i]);
        if (list && group_bad(v, g))
            reinterpret_cast<unsigned short*>(lds + 16)[atomicAdd(reinterpret_cast<unsigned*>(lds), 1u)] =
                (unsigned short)group(g);
    }
}
// sum[k] += p[c] * q[k][c] over c = c0 .. c1 - 1, byte offsets po and qo[k], pstep and qstep apart (NaN stays NaN:
// nothing is left to add then)
template <typename T>
__device__ __forceinline__ void sum_products(float (&sum)[4], __amdgpu_buffer_rsrc_t rs_p, unsigned po, unsigned pstep,
                                             __amdgpu_buffer_rsrc_t rs_q, const unsigned (&qo)[4], unsigned qstep,
                                             int c0, int c1)
{
    for (int cb = c0; cb < c1 && !all_nan(sum); cb += 8) {
        const int ce = cb + 8 < c1 ? cb + 8 : c1;
#pragma unroll 4
        for (int c = cb; c < ce; ++c) {
            const float v = load_f32<T>(rs_p, po, c * pstep);
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[k] = fmaf(v, load_f32<T>(rs_q, qo[k], c * qstep), sum[k]);
        }
    }
}

}  // namespace ukst
