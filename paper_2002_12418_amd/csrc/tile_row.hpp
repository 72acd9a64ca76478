// One row of an input tile: A consecutive values of a row of the image, zeros where they lie left or right of it.
#pragma once
#include <hip/hip_runtime.h>
#include "bf16_parts.hpp"

namespace mnnconv {

// x of x_bytes bytes (below 2 GiB), element `first` of it the first of the row, column x0 of an image W wide; lanes that are not `ok` get zeros.
// 16- and 8-byte loads at 4-byte alignment, the same for rows that hang over an edge: what they read of the neighbouring row is cleared afterwards.
template <int A>
__device__ __forceinline__ void load_tile_row(const float* x, unsigned x_bytes, int first, int x0, int W, bool ok, float (&d)[A])
{
    const bool leaves = ok && (first < 0 || first + A > (int)(x_bytes / 4u));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)x_bytes, 0x00020000);
    const unsigned off = ok && !leaves ? (unsigned)first * 4u : kOutsideBytes;
    int j = 0;
#pragma unroll
    for (; j + 4 <= A; j += 4) {
        const uintx4 v = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 4 * j), 0, 0));
        d[j] = __uint_as_float(v.x); d[j + 1] = __uint_as_float(v.y);
        d[j + 2] = __uint_as_float(v.z); d[j + 3] = __uint_as_float(v.w);
    }
    if (j + 2 <= A) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(off + 4 * j), 0, 0);
        d[j] = __uint_as_float(v[0]); d[j + 1] = __uint_as_float(v[1]);
        j += 2;
    }
    if (j < A) d[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off + 4 * j), 0, 0));
    if (__builtin_amdgcn_ballot_w64(leaves) != 0) {       // a row whose loads would leave the tensor: element by element
#pragma unroll
        for (int e = 0; e < A; ++e) {
            const unsigned oe = leaves && (unsigned)(x0 + e) < (unsigned)W ? (unsigned)(first + e) * 4u : kOutsideBytes;
            const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)oe, 0, 0));
            d[e] = leaves ? v : d[e];
        }
    }
#pragma unroll
    for (int e = 0; e < A; ++e) d[e] = (unsigned)(x0 + e) < (unsigned)W ? d[e] : 0.f;
}

}  // namespace mnnconv
