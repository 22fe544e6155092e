// fp32 values as three bf16 parts, for the kernels that form fp32 products on
// the bf16 matrix cores (internal header). Each part is the bf16 rounding of what
// the parts before it leave, which has at most 16, then 8 significant bits.
//  * x = h + m + l exactly for 2^-110 <= |x| < 2^128 - 2^119. Below, the last bits
//    lie under bf16's least subnormal, 2^-133: the parts are then x to the nearest
//    multiple of that (an error of up to 2^-134: 2^-24 of x at 2^-110, 5e-5 of
//    1e-36). From 2^128 - 2^119 on, and for infinities and NaN, h is not finite
//    and neither is any sum x enters.
//  * A product of two such values takes the six part products of weight 2^-16 or
//    more (hh, hm, mh, mm, hl, lh); the three dropped are at most 2^-24 of it
//    together (2^-26 on average). With the rounding of the sum a single product
//    is within 2^-23 of exact (9.1e-8 the largest seen; one fp32 fma: 2^-24, 6.0e-8);
//    sums of more are closer than fp32 chains, since the hh products, exact in
//    fp32, round into the main sum once per matrix instruction.
//  * h can round up past x, so that hh overflows where x * y does not.
// The kernels therefore take sums that are not finite again in fp32.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// bf16 parts of eight floats, two to a register.
struct Parts {
    u32x4_t h, m, l;
};

// Parts of floats 2*i and 2*i + 1; with r what the parts before leave.
__device__ __forceinline__ void split2(Parts &p, int i, float x, float y) {
    const f32x2_t v = {x, y};
    const uint32_t hb = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
    const f32x2_t r1 = {x - __uint_as_float(hb << 16), y - __uint_as_float(hb & 0xffff0000u)};
    const uint32_t mb = __builtin_bit_cast(uint32_t, __builtin_convertvector(r1, bf16x2_t));
    const f32x2_t r2 = {r1.x - __uint_as_float(mb << 16), r1.y - __uint_as_float(mb & 0xffff0000u)};
    p.h[i] = hb;
    p.m[i] = mb;
    p.l[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r2, bf16x2_t));
}

// Buffer descriptor of a wave-uniform range. Parts of its address come from
// divisions and 64-bit products, which run on the vector unit: without the way
// back to scalars every load through it becomes a loop over the lanes'
// descriptors.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const float *p, uint32_t bytes) {
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

}  // namespace
