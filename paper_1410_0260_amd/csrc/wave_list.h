// A sorted list of (distance, id) entries kept across the 64 lanes of a wave
// (lane t: the t-th smallest), in increasing (distance, id) order.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace askit {

__device__ __forceinline__ bool wl_before(double d1, int32_t i1, double d2, int32_t i2)
{
    return d1 < d2 || (d1 == d2 && i1 < i2);
}

// compare-exchange with lane ^ o: the smaller entry stays in the lane whose
// bit o is clear (up) or set (not up)
__device__ __forceinline__ void wl_exchange(double &d, int32_t &i, int o, bool up)
{
    const double od = __shfl_xor(d, o);
    const int32_t oi = __shfl_xor(i, o);
    const bool low = ((threadIdx.x & o) == 0) == up;      // this lane keeps the smaller
    const bool take = low ? wl_before(od, oi, d, i) : wl_before(d, i, od, oi);
    d = take ? od : d;
    i = take ? oi : i;
}

// the 64 smallest of the list and of another ascending list (cd, ci)
__device__ __forceinline__ void wl_merge_sorted(double &ld, int32_t &li, double cd, int32_t ci)
{
    const int lane = threadIdx.x & 63;
    const double rd = __shfl(cd, 63 - lane);
    const int32_t ri = __shfl(ci, 63 - lane);
    if (wl_before(rd, ri, ld, li)) {
        ld = rd;
        li = ri;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wl_exchange(ld, li, o, true);
}

// Merges the entries (D, j) of the lanes in `in` (none of them in the list
// yet): up to WL_SERIAL one by one, each by a ballot and a shift, more by a
// bitonic sort of the batch and one merge.
constexpr int WL_SERIAL = 16;

__device__ __forceinline__ void wl_insert(double &ld, int32_t &li, double D, int32_t j, bool in)
{
    const int lane = threadIdx.x & 63;
    uint64_t m = __ballot(in);
    if (__popcll(m) <= WL_SERIAL) {
        while (m) {
            const int b = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const double cd = __shfl(D, b);
            const int32_t cj = __shfl(j, b);
            const int pos = __popcll(__ballot(wl_before(ld, li, cd, cj)));
            const double ud = __shfl_up(ld, 1);
            const int32_t ui = __shfl_up(li, 1);
            if (lane >= pos) {
                ld = lane == pos ? cd : ud;
                li = lane == pos ? cj : ui;
            }
        }
        return;
    }
    double cd = in ? D : __longlong_as_double(0x7ff0000000000000ll);
    int32_t ci = in ? j : 0x7fffffff;
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
        for (int o = k >> 1; o > 0; o >>= 1) wl_exchange(cd, ci, o, (lane & k) == 0);
    wl_merge_sorted(ld, li, cd, ci);
}

}  // namespace askit
