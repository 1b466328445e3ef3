// Walks over an event's hits in device code.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hough {

__device__ __forceinline__ void event_range(const uint64_t *offs, uint32_t e, uint64_t n_hits,
                                            uint64_t &b, uint64_t &end)
{
    b = min(offs[e], n_hits);
    end = min(offs[e + 1], n_hits);
    if (end < b) end = b;
}

// Calls f(layer, phi, index) for every hit of [b, end); with `vec` (layer
// 4-byte and phi 16-byte aligned) the aligned middle is read four hits per
// load.
template <class F>
__device__ __forceinline__ void indexed_hits(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi,
                                             uint64_t b, uint64_t end, uint32_t t, uint32_t nt, bool vec, F &&f)
{
    uint64_t tail = b;
    if (vec) {
        const uint64_t a = min((b + 3) & ~uint64_t(3), end);
        if (t < a - b) f(uint32_t(layer[b + t]), phi[b + t], b + t);
        const uint64_t nq = (end - a) >> 2;
        const uint32_t *l4 = reinterpret_cast<const uint32_t *>(layer + a);
        const uint4 *p4 = reinterpret_cast<const uint4 *>(phi + a);
#pragma unroll 2
        for (uint64_t q = t; q < nq; q += nt) {
            const uint32_t lw = l4[q];
            const uint4 pw = p4[q];
            const uint64_t i = a + 4 * q;
            f(lw & 0xFFu, pw.x, i);
            f((lw >> 8) & 0xFFu, pw.y, i + 1);
            f((lw >> 16) & 0xFFu, pw.z, i + 2);
            f(lw >> 24, pw.w, i + 3);
        }
        tail = a + (nq << 2);
    }
    for (uint64_t i = tail + t; i < end; i += nt) f(uint32_t(layer[i]), phi[i], i);
}

constexpr uint32_t kBoundsQuads = 4;                 // four-hit loads in flight per thread

// Calls take(layer, phi) for every hit of [b, end); with `vec` as above, and kBoundsQuads loads are issued before the first
// is used (calls past the end have layer 255).
template <class F>
__device__ __forceinline__ void batched_hits(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi,
                                             uint64_t b, uint64_t end, uint32_t t, uint32_t nt, bool vec, F &&take)
{
    uint64_t tail = b;
    if (vec) {
        const uint64_t a = min((b + 3) & ~uint64_t(3), end);
        if (t < a - b) take(uint32_t(layer[b + t]), phi[b + t]);
        const uint64_t nq = (end - a) >> 2;
        const uint32_t *l4 = reinterpret_cast<const uint32_t *>(layer + a);
        const uint4 *p4 = reinterpret_cast<const uint4 *>(phi + a);
        for (uint64_t q = t; q < nq; q += kBoundsQuads * nt) {
            uint32_t lw[kBoundsQuads];
            uint4 pw[kBoundsQuads];
#pragma unroll
            for (uint32_t i = 0; i < kBoundsQuads; ++i) {
                const uint64_t k = min(q + i * nt, nq - 1);
                lw[i] = q + i * nt < nq ? l4[k] : 0xFFFFFFFFu;
                pw[i] = p4[k];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t i = 0; i < kBoundsQuads; ++i) {
                take(lw[i] & 0xFFu, pw[i].x);
                take((lw[i] >> 8) & 0xFFu, pw[i].y);
                take((lw[i] >> 16) & 0xFFu, pw[i].z);
                take(lw[i] >> 24, pw[i].w);
            }
        }
        tail = a + (nq << 2);
    }
    for (uint64_t i = tail + t; i < end; i += nt) take(uint32_t(layer[i]), phi[i]);
}

// The table entry of a bucket with hits in [mn, mx] (mn > mx: empty) before a
// bucket whose smallest is nn (nx < nn: empty).
__device__ __forceinline__ uint2 bounds_entry(uint32_t mn, uint32_t mx, uint32_t nn, uint32_t nx, uint32_t wmask)
{
    const uint32_t lo = mn <= mx ? (mx & wmask) + 1u : 0u;           // may equal W: never empty
    const uint32_t hi = nn <= nx ? (nn & wmask) : wmask;
    return hi >= lo ? make_uint2(lo, hi - lo) : make_uint2(0xFFFFFFFFu, 0u);
}

}  // namespace hough
