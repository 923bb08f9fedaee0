// Device helpers shared by the fragment-weight kernels (conv_slices.hip,
// upsample.hip): one MFMA over a 64-byte K step, bf16 packing, LDS staging.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rtcc {
namespace kern {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

// c += a . b over one K step of 64 bytes per row (32 bf16, 16 float32):
// lane (fr = lane % 16, fk = lane / 16) holds 16 bytes of row fr of both
// operands; it ends with rows 4 fk .. 4 fk + 3 of column fr.
template <typename T>
struct Step;
template <>
struct Step<uint16_t> {
    static constexpr int EPV = 8;  // elements per 16-byte vector
    __device__ static inline f32x4_t mma(uint4 a, uint4 b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                       __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <>
struct Step<float> {
    static constexpr int EPV = 4;
    __device__ static inline f32x4_t mma(uint4 a, uint4 b, f32x4_t c) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    }
};

// two floats to bf16, round to nearest even
__device__ inline uint32_t pack_bf16(float a, float b) {
    uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    ua += 0x7fffu + ((ua >> 16) & 1u);
    ub += 0x7fffu + ((ub >> 16) & 1u);
    return (ua >> 16) | (ub & 0xffff0000u);
}

// 16 bytes per lane from global memory into LDS at lds_addr + 16 * lane
// (lds_addr wave-uniform).  The caller waits with s_waitcnt vmcnt.
__device__ inline void load_lds16(const void *g, uint32_t lds_addr) {
    const uint32_t a = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(a) : "memory", "m0");
}

__device__ inline uint32_t lds_address(const void *p) {
    return __builtin_amdgcn_readfirstlane(uint32_t(reinterpret_cast<uintptr_t>((lds_void *)p)));
}

}  // namespace
}  // namespace kern
}  // namespace rtcc
