// FP4 (e2m1) operands of packed descriptor bits, shared by the FP4
// matchers.  Included inside namespace latch { namespace { ... } }.
//
// e2m1 holds 0 (0x0), +-0.5 (0x1 / 0x9), +-1 (0x2 / 0xa) and +-2 (0x4 / 0xc)
// exactly.  The 32 bits of a packed word become 32 nibbles in four dwords, bit
// 4 i + j in nibble i of dword j; train and query use the same map, so a
// product over K covers every bit once.  A train bit is 0 or c (c = 0.5, 1,
// 2, 2 for dwords j = 0..3) and the query bit it meets +1 / c or -1 / c.
#pragma once

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Train word -> its four FP4 dwords (0 or c per bit, c = 0.5, 1, 2, 2): the
// bits stay where they are as nibble bit 0, 1, 2, and bit 3 (the sign) moves
// down to bit 2.
__device__ __forceinline__ uint4 fp4_train(uint32_t w)
{
    return make_uint4(w & 0x11111111u, w & 0x22222222u, w & 0x44444444u, (w >> 1) & 0x44444444u);
}

// (a << n) | b in one instruction (b in a scalar register; the compiler turns
// the shift of a masked value into a shift, a mask and an or).
template <int n>
__device__ __forceinline__ uint32_t lshl_or(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "i"(n), "s"(b));
    return r;
}

// Query word -> its four FP4 dwords (+-1 / c per bit: +-2, +-1, +-0.5, +-0.5):
// the magnitude is constant and the nibble's sign is the inverted bit.
__device__ __forceinline__ uint4 fp4_query(uint32_t w)
{
    const uint32_t n = ~w;
    return make_uint4(lshl_or<3>(n & 0x11111111u, 0x44444444u), lshl_or<2>(n & 0x22222222u, 0x22222222u),
                      lshl_or<1>(n & 0x44444444u, 0x11111111u), (n & 0x88888888u) | 0x11111111u);
}

__device__ __forceinline__ v8i fp4_operand(uint4 f)
{
    v8i r = {};
    r[0] = (int)f.x;
    r[1] = (int)f.y;
    r[2] = (int)f.z;
    r[3] = (int)f.w;
    return r;
}

// c + a b over K = 128, 16 x 16, of FP4 operands.  Scales of zero select the
// instruction without block scales, which issues in half the time (the one with
// them is two instruction words and reads two more registers): with keys whose
// fraction holds the row instead of scaled products, matching 8000 x 1,000,000
// went from 1231 to 1176 us and 1920 x 1080 pixels within radius 4 from 107 to 103 us.
__device__ __forceinline__ v4f fp4_mfma(v8i a, v8i b, v4f c)
{
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);
}
