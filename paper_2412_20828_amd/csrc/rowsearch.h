// The least two entries of a row in the order of the lane-per-frame kernels
// (gen_spec._min_steps).  On numbers the order does not matter, and the
// frame-per-workgroup kernels read a row in an order of their own; but a median
// with a NaN returns the least of the others, so that what a NaN entry does
// depends on the triple it is in.  Frames whose posteriors hold a NaN (NaN or
// contradicting infinite LLRs, overflow) take this search, and decode as in
// the lane-per-frame kernels bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bch {

__device__ __forceinline__ uint32_t med3i(uint32_t a, uint32_t b, uint32_t c)
{
    return __float_as_uint(__builtin_amdgcn_fmed3f(__uint_as_float(a), __uint_as_float(b), __uint_as_float(c)));
}

// w entries; get() returns the magnitude bits of the next one, columns ascending
template <class Get>
__device__ __forceinline__ uint2 ordered_search(int w, Get get)
{
    uint32_t u1 = 0x7f800000u, u2 = 0x7f800000u;
    auto triple = [&](uint32_t &m, uint32_t &s) {
        // one entry after the other: side by side their addresses take registers
        const uint32_t a = get();
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t b = get();
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t c = get();
        __builtin_amdgcn_sched_barrier(0);
        m = min(min(a, b), c);
        s = med3i(a, b, c);
    };
    int n = w / 3, rest = w - 3 * n;
    uint32_t ma, sa, mb, sb;
    if (n >= 2) {
        triple(ma, sa);
        triple(mb, sb);
        u1 = min(ma, mb);
        u2 = med3i(ma, mb, min(sa, sb));
        n -= 2;
#pragma unroll 1
        while (n >= 2) {
            triple(ma, sa);
            triple(mb, sb);
            u2 = min(med3i(u1, ma, mb), min(min(u2, sa), sb));
            u1 = min(min(u1, ma), mb);
            n -= 2;
        }
        if (n) {
            triple(ma, sa);
            u2 = med3i(u1, ma, min(u2, sa));
            u1 = min(u1, ma);
        }
    } else if (n == 1) {
        triple(u1, u2);
    } else if (rest == 2) {
        ma = get();
        mb = get();
        u1 = min(ma, mb);
        u2 = max(ma, mb);
        rest = 0;
    }
#pragma unroll 1
    for (; rest > 0; rest--) {
        const uint32_t x = get();
        u2 = med3i(u1, u2, x);
        u1 = min(u1, x);
    }
    return make_uint2(u1, u2);
}

}  // namespace bch
