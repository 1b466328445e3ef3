// Step 1 of the transform in its row form (Section 4, first step; the
// Discussion's A[B[i]] += 1 in layer-mask form): the direct form's decision
// (k_vote_direct.hip: bin p of a row with offset o = J W + f is occupied iff
// (f - lo_j) mod 2^32 > span_j, j = J + p), arranged for grids and batches
// that do not keep the chip busy for long, where the chain of loads in front
// of the arithmetic decides.
//
// A wavefront takes R consecutive rows and 256 cells of them, four
// consecutive cells per lane.  Before any arithmetic it loads, for every
// layer, the table entries of the lane's cells at the rows' smaller J, five
// consecutive entries: J is monotone along the rows and rarely changes within
// R of them, and at J + 1 cell k's entry is cell k + 1's at J.  All layers'
// loads are in flight together; the rows then take entries k or k + 1 from
// registers (a layer whose J spans more is loaded row by row).  Row offsets
// come from a table by row, 64 contiguous bytes of scalars each.
//
// Bound by that chain: 1024 x 1024 cells take 9.8 us and 512 x 512 under 8,
// where a launch that does nothing takes 4.5 (rank form, tile by tile: 32 and
// 18; direct form: 12 and 10).  Four layers' entries at a time: all ten of a
// ten-layer grid take the same 7 to 10 us with 150 registers for 82.
#include <algorithm>

#include "device_hits.h"
#include "hough_internal.h"

namespace hough {

namespace {

constexpr uint32_t kRowsThreads = 256, kRowsWaves = kRowsThreads / 64;
// What a workgroup that finds the table itself takes: (layer, bucket) entries
// (20 KB of LDS), mean hits per event, and hits in all (one event may hold
// them all, and every workgroup walks its whole event).
constexpr uint32_t kRowsOwnEntries = 2560, kRowsOwnHits = 8192, kRowsOwnHitsAll = 32768;

// m[k] = 2 m[k] + [(f - e[k].lo) mod 2^32 > e[k].span] for four cells, f
// wave-uniform: a subtract, a subtract whose borrow is the comparison, an add
// with that borrow as carry, the four chains interleaved (as in
// k_vote_direct.hip).
__device__ __forceinline__ void shift_in4(uint32_t (&m)[4], uint32_t f, const uint2 &e0, const uint2 &e1,
                                          const uint2 &e2, const uint2 &e3)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t d0, d1, d2, d3;
    uint64_t c0, c1, c2, c3;
    asm("v_sub_u32 %4, %12, %13\n\t"
        "v_sub_u32 %5, %12, %14\n\t"
        "v_sub_u32 %6, %12, %15\n\t"
        "v_sub_u32 %7, %12, %16\n\t"
        "v_sub_co_u32 %4, %8, %17, %4\n\t"
        "v_sub_co_u32 %5, %9, %18, %5\n\t"
        "v_sub_co_u32 %6, %10, %19, %6\n\t"
        "v_sub_co_u32 %7, %11, %20, %7\n\t"
        "v_addc_co_u32 %0, %8, %0, %0, %8\n\t"
        "v_addc_co_u32 %1, %9, %1, %1, %9\n\t"
        "v_addc_co_u32 %2, %10, %2, %2, %10\n\t"
        "v_addc_co_u32 %3, %11, %3, %3, %11"
        : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3),
          "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "s"(f), "v"(e0.x), "v"(e1.x), "v"(e2.x), "v"(e3.x), "v"(e0.y), "v"(e1.y), "v"(e2.y), "v"(e3.y));
#else
    const uint2 e[4] = {e0, e1, e2, e3};
    for (int k = 0; k < 4; ++k) m[k] = 2 * m[k] + (f - e[k].x > e[k].y ? 1u : 0u);
#endif
}

}  // namespace

namespace {

// Rows R tile .. R tile + R - 1 of event e, cells 256 group .. + 255, from the
// event's table etab.
template <int R>
__device__ __forceinline__ void rows_unit(const uint2 *etab, const uint32_t *__restrict__ row_off,
                                          const uint32_t *__restrict__ row_ok, uint32_t n_layers, uint32_t rows,
                                          uint32_t nphi, uint32_t shift, uint32_t e, uint32_t tile, uint32_t group,
                                          uint16_t *__restrict__ acc)
{
    constexpr int B = 4;                             // layers loaded together
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t r0 = tile * R, last = min(r0 + R, rows) - 1;
    const uint32_t p0 = group * 256 + lane * 4, pm = nphi - 1, wmask = (1u << shift) - 1u;
    // the rows' offsets, 16 layers each (rows past the last repeat it)
    const uint32_t *off[R];
    uint32_t ok[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t row = min(r0 + r, last);
        off[r] = row_off + size_t(row) * kMaxLayers;
        ok[r] = row_ok[row];
    }
    uint32_t mask[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) mask[r][k] = 0;

    // layers from the highest to the lowest, B at a time
    for (int top = int(n_layers) - 1; top >= 0; top -= B) {
        uint2 win[B][5];
        uint32_t base[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int l = max(top - i, 0);
            const uint32_t ja = off[0][l] >> shift, jb = off[R - 1][l] >> shift;
            base[i] = ((jb - ja) & pm) <= (pm >> 1) ? ja : jb;       // the smaller, modulo the circle
            const uint2 *tl = etab + size_t(l) * nphi;
#pragma unroll
            for (int k = 0; k < 5; ++k) win[i][k] = tl[(base[i] + p0 + k) & pm];
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            if (top - i < 0) break;           // uniform
            const int l = top - i;
            const uint2 *tl = etab + size_t(l) * nphi;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!((ok[r] >> l) & 1u)) {                 // uniform
#pragma unroll
                    for (int k = 0; k < 4; ++k) mask[r][k] *= 2;
                    continue;
                }
                const uint32_t o = off[r][l], f = o & wmask, dj = ((o >> shift) - base[i]) & pm;
                if (dj == 0) {                       // uniform, as the two below
                    shift_in4(mask[r], f, win[i][0], win[i][1], win[i][2], win[i][3]);
                } else if (dj == 1) {
                    shift_in4(mask[r], f, win[i][1], win[i][2], win[i][3], win[i][4]);
                } else {
                    uint2 w[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[k] = tl[((o >> shift) + p0 + k) & pm];
                    shift_in4(mask[r], f, w[0], w[1], w[2], w[3]);
                }
            }
        }
    }
    if (p0 < nphi) {
        uint16_t *dst = acc + (uint64_t(e) * rows + r0) * nphi + p0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r0 + r <= last) {
                const uint32_t w[2] = {mask[r][0] | (mask[r][1] << 16), mask[r][2] | (mask[r][3] << 16)};
                __builtin_memcpy(__builtin_assume_aligned(dst + size_t(r) * nphi, 4), w, 8);
            }
        }
    }
}

}  // namespace

template <int R>
__global__ void __launch_bounds__(kRowsThreads)
k_vote_rows(const uint2 *__restrict__ tab, const uint32_t *__restrict__ row_off, const uint32_t *__restrict__ row_ok,
            uint32_t n_layers, uint32_t rows, uint32_t nphi, uint32_t shift, uint32_t n_tiles, uint32_t n_groups,
            uint64_t n_units, uint16_t *__restrict__ acc)
{
    const uint64_t unit = uint64_t(blockIdx.x) * kRowsWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= n_units) return;
    const uint32_t group = uint32_t(unit % n_groups), tile = uint32_t(unit / n_groups % n_tiles);
    const uint32_t e = uint32_t(unit / n_groups / n_tiles);
    rows_unit<R>(tab + size_t(e) * n_layers * nphi, row_off, row_ok, n_layers, rows, nphi, shift, e, tile, group, acc);
}

// The same for events of few hits on small grids, in one launch: every
// workgroup finds the event's whole table itself, in LDS, from all of its
// hits.  Bound by its chain of LDS passes, which takes less than a second
// launch: bounds and vote of one event of 256 x 256 cells and 2000 hits 10.6 ->
// 8.9 us, of 64 x 128 11.2 -> 8.3.
template <int R>
__global__ void __launch_bounds__(kRowsThreads)
k_vote_rows_own(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi, const uint64_t *__restrict__ offs,
                uint64_t n_hits, int vec, const uint32_t *__restrict__ row_off, const uint32_t *__restrict__ row_ok,
                uint32_t n_layers, uint32_t rows, uint32_t nphi, uint32_t shift, uint32_t n_tiles, uint32_t n_groups,
                uint32_t wgs, uint16_t *__restrict__ acc)
{
    HOUGH_DYNAMIC_LDS(uint2, tab_s);                 // [L][nphi]: {min, max}, then {lo, span}
    const uint32_t t = threadIdx.x, e = blockIdx.x / wgs, entries = n_layers * nphi;
    const uint32_t unit = (blockIdx.x % wgs) * kRowsWaves + __builtin_amdgcn_readfirstlane(t >> 6);
    uint64_t b, end;
    event_range(offs, e, n_hits, b, end);
    for (uint32_t i = t; i < entries; i += kRowsThreads) tab_s[i] = make_uint2(0xFFFFFFFFu, 0u);
    __syncthreads();
    batched_hits(layer, phi, b, end, t, kRowsThreads, vec, [&](uint32_t l, uint32_t ph) {
        if (l < n_layers) {
            uint2 *x = &tab_s[l * nphi + (ph >> shift)];
            atomicMin(&x->x, ph);
            atomicMax(&x->y, ph);
        }
    });
    __syncthreads();
    uint2 out[kRowsOwnEntries / kRowsThreads];
#pragma unroll
    for (uint32_t k = 0; k < kRowsOwnEntries / kRowsThreads; ++k) {
        if (k * kRowsThreads >= entries) break;      // uniform
        const uint32_t i = min(t + k * kRowsThreads, entries - 1);
        const uint2 a = tab_s[i], n = tab_s[(i & ~(nphi - 1)) + ((i + 1) & (nphi - 1))];
        out[k] = bounds_entry(a.x, a.y, n.x, n.y, (1u << shift) - 1u);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kRowsOwnEntries / kRowsThreads; ++k) {
        if (k * kRowsThreads >= entries) break;
        if (t + k * kRowsThreads < entries) tab_s[t + k * kRowsThreads] = out[k];
    }
    __syncthreads();
    if (unit < n_tiles * n_groups)
        rows_unit<R>(tab_s, row_off, row_ok, n_layers, rows, nphi, shift, e, unit / n_groups, unit % n_groups, acc);
}

namespace {

template <int R>
void launch_rows_r(hough_ctx *c, const hough_hits *h, bool own, uint16_t *acc, hipStream_t s)
{
    const uint32_t E = h->n_events, n_tiles = (c->rows + R - 1) / R, n_groups = (c->spec.n_phi + 255) / 256;
    if (own) {
        const int vec = (reinterpret_cast<uintptr_t>(h->layer) & 3) == 0 && (reinterpret_cast<uintptr_t>(h->phi) & 15) == 0;
        const uint32_t wgs = (n_tiles * n_groups + kRowsWaves - 1) / kRowsWaves;
        hipLaunchKernelGGL(k_vote_rows_own<R>, dim3(E * wgs), dim3(kRowsThreads),
                           size_t(c->spec.n_layers) * c->spec.n_phi * 8, s, h->layer, h->phi, h->event_offsets,
                           h->n_hits, vec, c->d_row_off, c->d_row_ok, c->spec.n_layers, c->rows, c->spec.n_phi,
                           c->shift, n_tiles, n_groups, wgs, acc);
    } else {
        const uint64_t n_units = uint64_t(E) * n_tiles * n_groups;
        const dim3 grid(uint32_t((n_units + kRowsWaves - 1) / kRowsWaves));
        hipLaunchKernelGGL(k_vote_rows<R>, grid, dim3(kRowsThreads), 0, s, c->d_dir_tab, c->d_row_off, c->d_row_ok,
                           c->spec.n_layers, c->rows, c->spec.n_phi, c->shift, n_tiles, n_groups, n_units, acc);
    }
}

}  // namespace

// The default for few events (those whose bounds are found layer by layer)
// and up to 2^22 cells.  Bounds and vote together, here against the better of
// the rank and direct forms with the same bounds: 1 x 256 x 256 cells 10.4 us
// against 12.5, 1024 x 1024 13.0 against 15.4, 1024 x 2048 16.6 against 24.2,
// 16 x 512 x 512 (2^22) 21.4 against 20.7 to 23.8, 24 x 512 x 512 29.3 against
// 24.2, 37 x 512 x 512 40 against 28: past the line the rank form's one
// staging of a tile's tables for many cells costs less than five entries per
// lane and layer for every few rows.
bool rows_vote_default(const hough_ctx *c, uint32_t n_events)
{
    return c->d_row_off && direct_vote_usable(c) && bounds_by_layer(c, n_events) &&
           uint64_t(n_events) * c->rows * c->spec.n_phi <= kRowsCellsMax;
}

hipError_t launch_vote_rows(hough_ctx *c, const hough_hits *h, uint16_t *acc, hipStream_t s)
{
    const uint32_t E = h->n_events;
    // one launch where finding the table again in every workgroup is cheap
    // (both ways in us: 256 x 256 cells 2000 hits 8.9 / 10.6, 8000 hits 9.8 /
    // 10.8, 16,000 11.5 / 10.5; 512 x 512 cells 6000 hits 11.2 / 11.1; 16
    // events of 256 x 256 and 2000 hits 10.6 / 11.5)
    const bool own = uint64_t(c->spec.n_layers) * c->spec.n_phi <= kRowsOwnEntries &&
                     h->n_hits <= std::min(uint64_t(kRowsOwnHits) * E, uint64_t(kRowsOwnHitsAll));
    if (!own) {
        const hipError_t err = launch_vote_bounds(c, h, s);
        if (err != hipSuccess) return err;
    }
    // rows per wave: eight share the loads best, but sixteen waves per compute
    // unit come first (16 events of 512 x 512: 17.1 us at four rows, 19.6 at
    // eight); two rows need no more entries than one (1024 x 1024: 9.8 us at
    // two, 11.7 at one)
    const uint64_t waves = uint64_t(E) * c->rows * ((c->spec.n_phi + 255) / 256);
    uint32_t R = 8;
    while (R > 2 && waves / R < 16 * uint64_t(c->n_cu)) R >>= 1;
    KernelTimer t;
    prof_begin(c, own ? "vote_rows_own" : "vote_rows", s, &t);
    switch (R) {
    case 2: launch_rows_r<2>(c, h, own, acc, s); break;
    case 4: launch_rows_r<4>(c, h, own, acc, s); break;
    default: launch_rows_r<8>(c, h, own, acc, s); break;
    }
    prof_end(c, s, &t);
    return hipGetLastError();
}

}  // namespace hough
