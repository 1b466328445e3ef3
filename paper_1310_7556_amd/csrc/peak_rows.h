// Row arithmetic shared by the row-window peak kernels: a wavefront holds a
// row of 64 * C cells, lane i cells C*i .. C*i + C - 1 as 16-bit pairs.
#pragma once

#include "hough_internal.h"

namespace hough {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pmax(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}

// a - b per 16-bit half, wrapping: bit 15 of a half is set iff b > a there
// (both at most 17)
__device__ __forceinline__ uint32_t psub(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b));
}

__device__ __forceinline__ uint32_t popc_pair(uint32_t w)
{
    return uint32_t(__popc(w & 0xFFFFu)) | (uint32_t(__popc(w >> 16)) << 16);
}

// lane i receives lane i - 1's value, lane 0 lane 63's (a wave-wide rotate
// right by one lane)
__device__ __forceinline__ uint32_t from_left(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x13C, 0xF, 0xF, false));
}

// lane i receives lane i + 1's value, lane 63 lane 0's (rotate left)
__device__ __forceinline__ uint32_t from_right(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x134, 0xF, 0xF, false));
}

// the lane's C cells of row r (r clamped into the grid; the caller zeroes
// rows outside it)
template <int C>
__device__ __forceinline__ void load_row(const uint16_t *__restrict__ ev, int r, uint32_t n_qpt, uint32_t lane,
                                         uint32_t (&w)[C / 2])
{
    const uint32_t rr = uint32_t(min(max(r, 0), int(n_qpt) - 1));
    const uint16_t *p = ev + size_t(rr) * (64u * C) + size_t(lane) * C;
    if constexpr (C == 4) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        w[0] = v.x;
        w[1] = v.y;
    } else {
#pragma unroll
        for (int g = 0; g < C / 8; ++g) {
            const uint4 v = reinterpret_cast<const uint4 *>(p)[g];
            w[4 * g] = v.x;
            w[4 * g + 1] = v.y;
            w[4 * g + 2] = v.z;
            w[4 * g + 3] = v.w;
        }
    }
}

// popcount pairs, lr and h of one row (see the header)
template <int C>
__device__ __forceinline__ void row_maxima(const uint32_t (&raw)[C / 2], uint32_t t2, uint32_t (&pc)[C / 2],
                                           uint32_t (&lr)[C / 2], uint32_t (&h)[C / 2])
{
    constexpr int D = C / 2;
#pragma unroll
    for (int d = 0; d < D; ++d) pc[d] = popc_pair(raw[d]);
    const uint32_t lft = from_left(pc[D - 1]);     // high half: the cell before the lane's first
    const uint32_t rgt = from_right(pc[0]);        // low half: the cell after the lane's last
    // s[d] = (cell 2d - 1, cell 2d): the left neighbours of pair d and the
    // right neighbours of pair d - 1
    uint32_t s[D + 1];
    s[0] = __builtin_amdgcn_alignbit(pc[0], lft, 16);
#pragma unroll
    for (int d = 1; d < D; ++d) s[d] = __builtin_amdgcn_alignbit(pc[d], pc[d - 1], 16);
    s[D] = __builtin_amdgcn_alignbit(rgt, pc[D - 1], 16);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lr[d] = pmax(pmax(s[d], s[d + 1]), t2);
        h[d] = pmax(lr[d], pc[d]);
    }
}

}  // namespace hough
