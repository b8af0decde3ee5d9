// Device helpers shared by the kernels that keep one vocabulary row of 16-bit values packed in
// registers (1024 threads x 16 bytes per step): the acceptance kernel and the draft-sampling kernel.
#pragma once
#include "device_utils.h"

namespace adaspec {

template <class T> struct Pair16;
template <> struct Pair16<BF16> {
    static constexpr uint32_t kNegInf2 = 0xFF80FF80u;
    static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
    static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
};
template <> struct Pair16<F16> {
    static constexpr uint32_t kNegInf2 = 0xFC00FC00u;
    static __device__ __forceinline__ float lo(uint32_t w) { return f16_bits_to_float((uint16_t)(w & 0xffffu)); }
    static __device__ __forceinline__ float hi(uint32_t w) { return f16_bits_to_float((uint16_t)(w >> 16)); }
};

// Opaque to the optimiser: forces later code to unpack the 16-bit pairs again instead of
// keeping 128 unpacked floats alive across the phases (the row must stay packed to fit).
__device__ __forceinline__ void keep_packed(uint4 &v)
{
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

typedef short short2v __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// sum over the 16 lanes of a DPP row (every lane of the row ends up with the row's total)
__device__ __forceinline__ float row16_sum(float v)
{
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x124, 0xF, 0xF, true));  // row_ror 4
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, true));  // row_ror 8
    return v;
}

// Weights of 16-bit logits are 2^fma(l, c, -r), relative to r and not to the maximum m.  r is a whole number near m c: what
// moves a sum from one reference to another (the maxima seen so far, those of threads and parts) is then an exact power of
// two.  With r = m c rounded and factors of 2^((a - b) c) the roundings of the products stayed in the sum, 1e-6 to 1e-5 of it
// where m c is 20 to 100, and nothing took them out of p = weight / sum.
__device__ __forceinline__ float scaled_ref(float m, float c) { return ceilf(m * c); }

// Maxima at or below this count as -inf: their product with c, from 2^31 on, is so coarse (or not finite at all) that weights relative
// to it overflow, and what moves such a sum elsewhere is 0.  They are those of threads, wavefronts and parts of which a mask has
// left nothing, where it wrote the type's lowest number in place of -inf.
// (With the largest scale, a power of two, products are exact as long as they are finite.)
constexpr float kLargestScale = 4194304.f;
template <class LT>
__device__ __forceinline__ float lowest_ref(float c)
{
    return sizeof(typename LT::storage) == 2 ? (c == kLargestScale ? -3.0e38f : -1.9e9f) * __builtin_amdgcn_rcpf(c) : -INFINITY;
}

// log2(e) / T.  For 16-bit rows no more than 2^22: a reference (or a product m c) from 2^31 on is so coarse that what it
// leaves of the largest logit's exponent overflows.  Below T = 3.4e-7, where that sets in, 16-bit logits that differ at all
// differ by a weight of 0, unless all of them are below 1e-2.
template <class LT>
__device__ __forceinline__ float exponent_scale(float T)
{
    const float c = 1.4426950408889634f / T;
    return sizeof(typename LT::storage) == 2 ? fminf(c, kLargestScale) : c;
}

}  // namespace adaspec
