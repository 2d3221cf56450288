// What several kernels use: vector types, 16-byte loads, moves between lanes, digits of an index.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace fea {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// (ONCE: bytes that nobody else reads and that need not stay in the caches)
template <bool ONCE = false> __device__ __forceinline__ u32x4 ld16(const void* p) {
    return ONCE ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)) : *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ uint32_t bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// x from another lane of its row of 16, as the DPP control says, without a detour through LDS.
template <int CTRL> __device__ __forceinline__ float lanes_moved(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// x mod d, and x becomes x / d (x >= 0); the divisors are mostly powers of two (1 among them), and a true division is 40 dependent
// instructions, one of 64 bits a hundred.
template <typename Int> __device__ __forceinline__ int take_digit(Int& x, int d) {
    const Int v = x;
    if ((d & (d - 1)) == 0) { x = v >> (31 - __clz(d)); return (int)(v & (d - 1)); }
    x = v / d;
    return (int)(v - x * d);
}

}  // namespace fea
