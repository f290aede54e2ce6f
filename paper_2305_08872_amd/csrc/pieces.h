// An fp32 value as the exact sum of three bf16 pieces: see identity_split.hip.
#ifndef AMULET_PIECES_H
#define AMULET_PIECES_H
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace amulet {

// Two neighbouring values into three words of packed pieces; returns the OR of what remains of both.
// Two pieces are rounded, the third is what is left: |x - p0| <= 2^-8 |x|, |p2| <= 2^-17 |x|, in 7 bits of x's last place.
// 11 instructions, as with a second piece that is cut (v_cvt_pk_bf16_f32 as asm: the compiler would convert the single values a
// second time).
__device__ __forceinline__ uint32_t take_pieces(float x, float y, uint32_t &p0, uint32_t &p1, uint32_t &p2)
{
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(p0) : "v"(x), "v"(y));
    x -= __builtin_bit_cast(float, p0 << 16);
    y -= __builtin_bit_cast(float, p0 & 0xffff0000u);
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(p1) : "v"(x), "v"(y));
    x -= __builtin_bit_cast(float, p1 << 16);
    y -= __builtin_bit_cast(float, p1 & 0xffff0000u);
    const uint32_t vx = __builtin_bit_cast(uint32_t, x), vy = __builtin_bit_cast(uint32_t, y);
    p2 = __builtin_amdgcn_perm(vy, vx, 0x07060302u);
    return vx | vy;
}

}  // namespace amulet
#endif
