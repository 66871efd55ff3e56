// tbn_codes8.h -- the 8-bit-activation matrix instructions and the decode of their two-bit filter
// operands, shared by the int8 and fp8 forward kernels.
#pragma once

#include "tbn_device.h"

namespace tbn {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ i32x16 mfma_i8(i32x4 a, i32x4 b, i32x16 c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// The 16 codes of one packed word as int8, element e in byte e % 4 of dword e / 4.
__device__ __forceinline__ i32x4 decode_i8(uint32_t w) {
    // bytes (magnitude even, magnitude odd, magnitude even, magnitude odd) and the same
    // for the sign planes; both sources are w, so the byte order of the pair is immaterial
    const uint32_t pm = __builtin_amdgcn_perm(w, w, 0x02000200u);
    const uint32_t ps = __builtin_amdgcn_perm(w, w, 0x03010301u);
    // element 4d + b: its magnitude to bit 2d of byte b, its sign to bit 2d + 1
    const uint32_t m = (pm & 0x0000FFFFu) | ((pm >> 1) & 0xFFFF0000u);
    const uint32_t s = ((ps << 1) & 0x0000FFFFu) | (ps & 0xFFFF0000u);
    const uint32_t z = (m & 0x55555555u) | (s & 0xAAAAAAAAu);
    constexpr uint32_t LUT = 0xFEFF0201u;  // index magnitude + 2 sign -> 1, 2, -1, -2
    i32x4 r;
    r.x = (int)__builtin_amdgcn_perm(LUT, LUT, z & 0x03030303u);
    r.y = (int)__builtin_amdgcn_perm(LUT, LUT, (z >> 2) & 0x03030303u);
    r.z = (int)__builtin_amdgcn_perm(LUT, LUT, (z >> 4) & 0x03030303u);
    r.w = (int)__builtin_amdgcn_perm(LUT, LUT, (z >> 6) & 0x03030303u);
    return r;
}

typedef int i32x8 __attribute__((ext_vector_type(8)));

// D += A B with A the E2M1 filter operand (format 4) and B the E4M3 activation operand
// (format 0), both scales 2^0 (E8M0 code 127)
__device__ __forceinline__ f32x16 mfma_f4f8(i32x8 fil, i32x8 act, f32x16 c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fil, act, c, 4, 0, 0, 127, 0, 127);
}

// (t << 1) + c in one v_lshl_add_u32 (c in a scalar register: the three-operand form takes
// no literal)
__device__ __forceinline__ uint32_t shl1_add(uint32_t t, uint32_t c) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(r) : "v"(t), "s"(c));
    return r;
}

// The 32 E2M1 values of words w0 (elements 0..15) and w1 (16..31) of the repacked layout;
// two22 = 0x22222222 (the 2 of every nibble) in a scalar register.
__device__ __forceinline__ i32x8 decode_f4(uint32_t w0, uint32_t w1, uint32_t two22) {
    i32x4 r;
    r[0] = (int)((w0 & 0xAAAAAAAAu) + two22);
    r[1] = (int)shl1_add(w0 & 0x55555555u, two22);
    r[2] = (int)((w1 & 0xAAAAAAAAu) + two22);
    r[3] = (int)shl1_add(w1 & 0x55555555u, two22);
    // the E2M1 form reads only the low four dwords: the others are left undefined
    return __builtin_shufflevector(r, r, 0, 1, 2, 3, -1, -1, -1, -1);
}

}  // namespace tbn
