// Matrix products of float32 operands on the bf16 matrix cores.
//
// A float is the exact sum of three bfloat16 numbers (8 significant bits
// each, rounded to nearest, so the parts' signs differ and cover all 24
// bits): x = h + m + l.  Of the nine products of two such sums the six of
// relative size 2^-18 and above are formed,
//   a b = ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + O(2^-26 |a b|),
// each an exact product accumulated in fp32 by v_mfma_f32_16x16x32_bf16.
// Six of those take 6/16 of the time of the fp32 matrix instructions for the
// same product (2.5 PFLOP/s against 157 TFLOP/s).  The error against 64 bits
// is a third to a half of the fp32 instructions' (256 -> 256 3x3 at 14x14: 2.6e-7
// against 5.9e-7), since the small products are summed apart (mfma_split).
// Where a sum of parts is not the sum of the operands it is formed again in
// plain fp32 by the kernels' epilogues (`again`):
//  - it is not finite: the split of an infinity, a NaN or a float that rounds
//    to infinity in bfloat16 holds a NaN, and a product of two parts rounded up
//    can pass the largest float where the operands' product does not;
//  - it is below 2^-100: an operand's third part is exact down to bfloat16's
//    smallest number, 2^-133, so of operands below 2^-110 low bits are lost, by
//    at most 2^-134 each.  A sum of at least 2^-100 does not see that, and one
//    of a training step never gets there.
//
// bf16 mode is the same with the first part only: operands rounded to
// nearest even, one product.  The kernels pad a block's products with zeros
// on one side only, and a zero times an infinity or NaN that the padding met
// makes a sum NaN that has no such operand: formed again in the same way.
#pragma once
#include <hip/hip_runtime.h>

namespace psw {

typedef float sp_v4f __attribute__((ext_vector_type(4)));
typedef __bf16 sp_v8b __attribute__((ext_vector_type(8)));

// two floats to bfloat16 (nearest even), the first in the low half
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, b2));
}

// an operand as the products of NS parts take it
template <int NS>
__device__ __forceinline__ float operand(float v)
{
    return NS == 1 ? (float)(__bf16)v : v;
}

// The sums to form again: for single ones, and whether there are any.
template <int NS>
__device__ __forceinline__ bool again(float v)
{
    if constexpr (NS == 1) return v != v;
    // the bits without the sign, from infinity's up and round to zero's and on to 2^-100's
    const uint32_t u = (__float_as_uint(v) << 1) - 0xff000000u;
    return u < 0x01000000u + (27u << 24) && u != 0x01000000u;
}
struct Again {
    float t = 0.f;              // NaN once a sum was not finite
    uint32_t least = ~0u;       // the smallest sum that is not zero: twice its bits, less one
    template <int NS>
    __device__ __forceinline__ void add(const sp_v4f& v)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            t = fmaf(v[i], 0.f, t);
            if (NS == 3) least = min(least, (__float_as_uint(v[i]) << 1) - 1u);
        }
    }
    __device__ __forceinline__ bool any() const { return t != t || least < (27u << 24) - 1u; }
};

// parts[0] = h, parts[1] = m, parts[2] = l of eight floats (NS = 1: h alone)
template <int NS>
__device__ __forceinline__ void split8(const float (&v)[8], sp_v8b (&parts)[NS])
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    u4 p[NS];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = v[2 * i], b = v[2 * i + 1];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint32_t u = bf16_pair(a, b);
            p[s][i] = u;
            if (s + 1 < NS) {
                a -= __uint_as_float(u << 16);
                b -= __uint_as_float(u & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) parts[s] = __builtin_bit_cast(sp_v8b, p[s]);
}

// Loads of a tensor through a buffer descriptor: a lane offset (bytes) of
// kOutside, or any at or past `bytes`, reads zero, so what lies outside a
// tensor needs neither a branch nor a select; the second offset is uniform,
// at most `bytes`, and costs no vector register per load.
constexpr int kOutside = (int)0x80000000;
using Buffer = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Buffer make_buffer(const float* p, int64_t bytes)
{
    const int n = bytes > 0x7fffffff ? 0x7fffffff : (int)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, n, 0x00020000);
}
__device__ __forceinline__ float buffer_load(Buffer b, int lane_bytes, int uniform_bytes)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, lane_bytes, uniform_bytes, 0));
}

// acc += A B for one 16x16x32 block.  A matrix instruction rounds its result
// at the running sum's size, so six of them into one sum err 1.1 to 1.9 times
// as far as the fp32 instructions (and FC's depth of 4096 2.4 times).  The
// five small products are therefore summed apart, smallest first: OWN in `lo`,
// which the kernel adds at its end and keeps in registers, and otherwise from
// zero for each block (4 additions of the vector units a block, no register
// that lives on).
template <int NS, bool OWN>
__device__ __forceinline__ void mfma_split(const sp_v8b (&a)[NS], const sp_v8b (&b)[NS], sp_v4f& acc, sp_v4f& lo)
{
    if constexpr (NS == 3) {
        sp_v4f t = OWN ? lo : sp_v4f{0.f, 0.f, 0.f, 0.f};
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], t, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc, 0, 0, 0);
        if constexpr (OWN)
            lo = t;
        else
            acc += t;
    } else {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc, 0, 0, 0);
    }
}

}  // namespace psw
