// Values and loads that the compiler is to leave as written.  Included inside
// namespace latch { namespace { ... } } of each kernel file.
#pragma once

// v, as a value the compiler does not know, made where it is used: what
// follows from it is not kept in registers over a loop.
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// One ds_read_b64.  (Atomic, so that the compiler does not pair two of a patch's reads
// into a ds_read2_b64, which gfx950 serves 16 lanes and one address at a time: at best
// half the rate of two ds_read_b64, and bank-conflicted unless the 16-lane quarters,
// rather than the 32-lane halves, of a wavefront are spread over the banks.)
__device__ __forceinline__ uint64_t read_quad(const uint8_t *p)
{
    return __atomic_load_n(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED);
}
