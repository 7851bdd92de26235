// Arithmetic on pairs of 16-bit lanes, shared by the extraction kernels.
// Included inside namespace latch { namespace { ... } }.
#pragma once

typedef short short2v __attribute__((ext_vector_type(2)));

constexpr uint32_t kPkMinus2 = 0xfffefffeu;       // -2 in both 16-bit halves

// c + a b per 16-bit half (v_pk_mad_i16; the compiler splits the multiply-add
// of 16-bit vectors into a shift, an add and a subtract).  b is uniform.
__device__ __forceinline__ short2v pk_mad_i16(short2v a, uint32_t b, short2v c)
{
    uint32_t r;
    asm("v_pk_mad_i16 %0, %1, %2, %3"
        : "=v"(r)
        : "v"(__builtin_bit_cast(uint32_t, a)), "s"(b), "v"(__builtin_bit_cast(uint32_t, c)));
    return __builtin_bit_cast(short2v, r);
}

// acc + a b of the low (high) halves, in 32 bits.
__device__ __forceinline__ int mad_i32_lo16(short2v a, short2v b, int acc)
{
    int r;
    asm("v_mad_i32_i16 %0, %1, %2, %3"
        : "=v"(r)
        : "v"(__builtin_bit_cast(uint32_t, a)), "v"(__builtin_bit_cast(uint32_t, b)), "v"(acc));
    return r;
}

__device__ __forceinline__ int mad_i32_hi16(short2v a, short2v b, int acc)
{
    int r;
    asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,1,0,0]"
        : "=v"(r)
        : "v"(__builtin_bit_cast(uint32_t, a)), "v"(__builtin_bit_cast(uint32_t, b)), "v"(acc));
    return r;
}
