// fp32 values as three bf16 parts, for the kernels that form fp32 products on
// the bf16 matrix cores (internal header). x = h + m + l exactly: each part is
// the bf16 rounding of what the parts before it leave, which has at most 16,
// then 8 significant bits. A product of two such values takes the six part
// products of weight 2^-16 or more (hh, hm, mh, mm, hl, lh); what is dropped
// is at most 2^-23 of it and 2^-26 on average. Infinities (and values that round to one in bf16) have
// no finite parts: every sum they enter is NaN.
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
