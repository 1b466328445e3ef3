// Step 2 of the transform (Section 4, second step) in one launch: the row-
// window form of the peak search (peak_rows.h, k_peaks_rows.hip) with every
// strip's rows kept in registers, so that a strip is read once, counted,
// placed and written.
//
// A wavefront owns a strip of R consecutive q/pT rows of one event (and one
// d0 plane): it reads them with a halo row on either side (and, with a d0
// axis, the same rows of the planes beside it), decides every cell and keeps
// the decisions as bits.  A workgroup of four strips publishes its count and
// finds its place by a decoupled look-back over the workgroups before it:
// wave 0 reads 64 predecessors' states at a time, each {empty, count, or
// count of everything up to it}, and adds counts until it meets a sum.  Then
// each row's peaks are compacted in cell order through LDS and stored.
//
// The states have to be empty when a launch begins: launches alternate
// between two arrays (the parity of a launch count kept on the device, so
// that a replayed graph alternates too), and each clears what the one before
// it filled.  A workgroup waits only for workgroups of smaller number, and
// takes its number from a counter when it starts running, so the smallest
// number still at work never waits and every wait ends.  That counter serves
// one workgroup per 12 ns, hence eight strips per workgroup on large grids.
//
// Bound by HBM on batches (2 bytes per cell read, 8 bytes per peak written),
// by the chain load, count, look back, store on single events.  Against a
// count pass, a scan and a write pass: 4096 events of 512 x 512 (7.3e8 peaks)
// 1917 -> 1707 us (4.7 TB/s), 512 x 512 x 64 70 -> 58 us, one event of 256 x
// 256 15 -> 8 us, of 1024 x 1024 30 -> 10 us.  Fewer rows per strip cost more
// numbers: 4096 events with 8 and 4 rows 2164 and 3109 us (16: 1884), all
// with four strips per workgroup and two counters.
#include "peak_rows.h"

namespace hough {

namespace {

// entries of the counters, each in a cache line of its own
constexpr uint32_t kNumber = 0, kLaunches = 32, kLastGrid = 33;
static_assert(kPeakCounterBase + kLastGrid < kCounterDwords, "peak counters fit the counter array");

constexpr uint64_t kStateCount = uint64_t(1) << 62, kStateSum = uint64_t(2) << 62, kStateValue = kStateCount - 1;

__device__ __forceinline__ uint64_t state_load(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t load_counter(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void state_store(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the counts of workgroups 0 .. w - 1, by one wave (uniform result).
__device__ __forceinline__ uint64_t look_back(const uint64_t *state, uint32_t w, uint32_t lane)
{
    uint64_t sum = 0;
    for (int64_t top = int64_t(w) - 1; top >= 0; top -= 64) {
        const int64_t i = top - int64_t(lane);
        uint64_t v, sums;
        for (;;) {
            v = i >= 0 ? state_load(state + i) : kStateSum;      // before the first: the sum 0
            sums = __ballot((v & kStateSum) != 0);
            // the lanes up to the nearest sum have to be filled
            const uint64_t need = sums ? (sums & (~sums + 1)) - 1 : ~uint64_t(0);
            if ((__ballot(v == 0) & need) == 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        const uint32_t last = sums ? uint32_t(__builtin_ctzll(sums)) : 63u;
        uint64_t x = lane <= last ? v & kStateValue : 0u;
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        sum += x;
        if (sums) break;
    }
    return sum;
}

}  // namespace

template <int C, int R, bool D3, int WAVES>
__global__ void __launch_bounds__(64 * WAVES)
k_peaks_one(const uint16_t *__restrict__ acc, uint32_t n_events, uint32_t n_qpt, uint32_t n_d0, uint32_t n_strips,
            uint64_t n_tiles, uint32_t thr, uint64_t *__restrict__ states, uint64_t n_states,
            uint32_t *__restrict__ counters,
            uint64_t *__restrict__ poff, hough_peak *__restrict__ peaks, uint64_t capacity)
{
    constexpr int D = C / 2;
    constexpr int kCells = 64 * C;
    __shared__ uint2 rec_s[WAVES][kCells];
    __shared__ uint32_t wave_cnt[WAVES], number_s, parity_s;
    __shared__ uint64_t base_s;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        const uint32_t number = atomicAdd(counters + kNumber, 1u);
        const uint32_t parity = load_counter(counters + kLaunches) & 1u, filled = load_counter(counters + kLastGrid);
        uint64_t *other = states + (parity ? 0 : n_states);
        for (uint64_t i = number; i < filled; i += gridDim.x) state_store(other + i, 0);
        number_s = number;
        parity_s = parity;
    }
    __syncthreads();
    const uint32_t number = __builtin_amdgcn_readfirstlane(number_s);
    uint64_t *state = states + (__builtin_amdgcn_readfirstlane(parity_s) ? n_states : 0);
    const uint64_t tile = uint64_t(number) * WAVES + wave;
    const bool active = tile < n_tiles;
    const uint32_t planes = D3 ? n_d0 : 1u;
    const uint64_t per_event = uint64_t(planes) * n_strips;
    const uint32_t e = active ? uint32_t(tile / per_event) : 0u;
    const uint32_t rem = active ? uint32_t(tile % per_event) : 0u;
    const uint32_t dp = rem / n_strips;
    const int r0 = int(rem % n_strips) * R;
    const uint64_t plane = uint64_t(n_qpt) * kCells;
    const uint16_t *ev = acc + (uint64_t(e) * planes + dp) * plane;
    const uint32_t t2 = min(thr, 17u) * 0x00010001u;   // popcounts are <= 16

    uint32_t raw[R + 2][D];                          // rows r0 - 1 .. r0 + R, zeros outside the grid
    uint32_t bits[R];                                // bit j of row i: cell j of the lane is a peak
    uint32_t cnt = 0;
    if (active) {
        auto zero_outside = [&](int r, uint32_t (&w)[D]) {
            const uint32_t keep = r < 0 || r >= int(n_qpt) ? 0u : 0xFFFFFFFFu;     // uniform
#pragma unroll
            for (int d = 0; d < D; ++d) w[d] &= keep;
        };
#pragma unroll
        for (int i = 0; i < R + 2; ++i) load_row<C>(ev, r0 - 1 + i, n_qpt, lane, raw[i]);
        // nb of row r0 - 1 + i: the larger h of the neighbour planes' rows (a
        // missing plane or row counts as zeros; loads without branches, so
        // that they are all issued ahead)
        const bool has_m = D3 && dp > 0, has_p = D3 && dp + 1 < planes;
        const uint16_t *evm = has_m ? ev - plane : ev, *evp = has_p ? ev + plane : ev;
        const uint32_t keep_m = has_m ? 0xFFFFFFFFu : 0u, keep_p = has_p ? 0xFFFFFFFFu : 0u;
        uint32_t rawm[D3 ? R + 2 : 1][D], rawp[D3 ? R + 2 : 1][D];
        if constexpr (D3) {
#pragma unroll
            for (int i = 0; i < R + 2; ++i) {
                load_row<C>(evm, r0 - 1 + i, n_qpt, lane, rawm[i]);
                load_row<C>(evp, r0 - 1 + i, n_qpt, lane, rawp[i]);
            }
        }
        auto nb_of = [&](int i, uint32_t (&nb)[D]) {
            uint32_t pcx[D], lrx[D], hx[D], hy[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                rawm[i][d] &= keep_m;
                rawp[i][d] &= keep_p;
            }
            zero_outside(r0 - 1 + i, rawm[i]);
            zero_outside(r0 - 1 + i, rawp[i]);
            row_maxima<C>(rawm[i], t2, pcx, lrx, hx);
            row_maxima<C>(rawp[i], t2, pcx, lrx, hy);
#pragma unroll
            for (int d = 0; d < D; ++d) nb[d] = pmax(hx[d], hy[d]);
        };
        uint32_t hp[D], pcc[D], lrc[D], hc[D], nbp[D], nbc[D];
        {
            uint32_t pcx[D], lrx[D];
            zero_outside(r0 - 1, raw[0]);
            row_maxima<C>(raw[0], t2, pcx, lrx, hp);
            row_maxima<C>(raw[1], t2, pcc, lrc, hc);
            if (D3) {
                nb_of(0, nbp);
                nb_of(1, nbc);
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            uint32_t pcn[D], lrn[D], hn[D], nbn[D];
            zero_outside(r0 + i + 1, raw[i + 2]);
            row_maxima<C>(raw[i + 2], t2, pcn, lrn, hn);
            if (D3) nb_of(i + 2, nbn);
            uint32_t bt = 0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                uint32_t mx = pmax(pmax(hp[d], hn[d]), lrc[d]);
                if (D3) mx = pmax(mx, pmax(pmax(nbp[d], nbc[d]), nbn[d]));
                const uint32_t neg = psub(pcc[d], mx);       // bit 15 of a half: not a peak
                bt |= (((neg >> 15) & 1u) | ((neg >> 30) & 2u)) << (2 * d);
            }
            bt ^= C == 32 ? 0xFFFFFFFFu : (1u << (C & 31)) - 1u;
            bits[i] = r0 + i < int(n_qpt) ? bt : 0u;
            cnt += uint32_t(__popc(bits[i]));
#pragma unroll
            for (int d = 0; d < D; ++d) {
                hp[d] = hc[d];
                hc[d] = hn[d];
                pcc[d] = pcn[d];
                lrc[d] = lrn[d];
                if (D3) {
                    nbp[d] = nbc[d];
                    nbc[d] = nbn[d];
                }
            }
        }
    }
    uint32_t mine = cnt;
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if (lane == 0) wave_cnt[wave] = mine;
    __syncthreads();
    uint32_t all = 0, before = 0;
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) {
        before += w < wave ? wave_cnt[w] : 0u;
        all += wave_cnt[w];
    }
    if (wave == 0) {
        if (lane == 0 && number > 0) state_store(state + number, kStateCount | all);
        const uint64_t sum = look_back(state, number, lane);
        if (lane == 0) {
            state_store(state + number, kStateSum | (sum + all));
            base_s = sum;
            // the last number's sum means that every workgroup has filled
            // its state, and so has read the counters
            if (number == gridDim.x - 1) {
                counters[kNumber] = 0;
                counters[kLaunches] += 1;
                counters[kLastGrid] = gridDim.x;
            }
        }
    }
    __syncthreads();
    uint64_t running = base_s + before;
    if (active && rem == 0 && lane == 0) poff[e] = running;
    if (active && tile == n_tiles - 1 && lane == 0) poff[n_events] = running + mine;

    // (the popcounts are taken again below: kept from above, they would take
    // as many registers as the cells)
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int i = 1; i <= R; ++i)
#pragma unroll
        for (int d = 0; d < D; ++d) asm volatile("" : "+v"(raw[i][d]));
#endif

    uint2 *rec = rec_s[wave];
    uint2 *out = reinterpret_cast<uint2 *>(peaks);
    if (active) {
        const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t bt = bits[i], n = uint32_t(__popc(bt));
            uint32_t o = 0, total = 0;
#pragma unroll
            for (int b = 0; (1 << b) <= C; ++b) {
                const uint64_t m = __ballot((n >> b) & 1u);
                o += uint32_t(__popcll(m & lt)) << b;
                total += uint32_t(__popcll(m)) << b;
            }
            if (total == 0) continue;                // uniform
            const uint32_t cell0 = (dp * n_qpt + uint32_t(r0 + i)) * uint32_t(kCells) + lane * C;
#pragma unroll
            for (int j = 0; j < C; ++j) {
                if ((bt >> j) & 1u) {
                    const uint32_t m = (raw[i + 1][j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
                    rec[o++] = make_uint2(cell0 + j, m | (uint32_t(__popc(m)) << 16));
                }
            }
            // the wave's records are in LDS before any lane reads them back
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (uint32_t k = lane; k < total; k += 64) {
                const uint64_t pos = running + k;
                if (pos < capacity) out[pos] = rec[k];
            }
            running += total;
            // and read back before the next row overwrites them
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

namespace {

template <int C, int R, bool D3, int WAVES>
void launch_one(hipStream_t s, const uint16_t *acc, uint32_t n_events, const hough_ctx *c, uint32_t n_strips,
                uint64_t n_tiles, uint64_t *poff, hough_peak *peaks, uint64_t capacity)
{
    const uint32_t grid = uint32_t((n_tiles + WAVES - 1) / WAVES);
    hipLaunchKernelGGL((k_peaks_one<C, R, D3, WAVES>), dim3(grid), dim3(64 * WAVES), 0, s, acc, n_events,
                       c->spec.n_qpt, c->spec.n_d0, n_strips, n_tiles, c->spec.threshold, c->d_peak_state,
                       c->n_peak_state, c->d_counters + kPeakCounterBase, poff, peaks, capacity);
}

// Strips from which a workgroup takes 8 (n_phi 512) or 16 (n_phi 256) of
// them instead of 4, so that the number counter keeps up: 512 events of 256 x
// 256, 8192 strips, 67 us with 4, 60 with 8, 54 with 16 (58 in three passes).
constexpr uint64_t kManyStrips = 4096;

// Rows per strip at most: what the registers hold.
constexpr int most_rows(int cells, bool d3)
{
    return d3 ? (cells >= 16 ? 2 : 32 / cells) : (cells >= 32 ? 4 : cells <= 8 ? 16 : 8);
}

// Rows per strip: as many as that, fewer while the chip is short of strips.
uint32_t one_rows(const hough_ctx *c, uint32_t n_events)
{
    uint32_t R = uint32_t(most_rows(int(c->spec.n_phi / 64), c->spec.n_d0 > 1));
    while (R > 2 && uint64_t(n_events) * c->spec.n_d0 * ((c->spec.n_qpt + R - 1) / R) < uint64_t(c->n_cu) * 8) R /= 2;
    return R;
}

}  // namespace

// The default peak search (no peak knob set by hand) of n_phi 256, 512, 1024
// and 2048.
bool peaks_one_usable(const hough_ctx *c, const uint16_t *acc, uint32_t n_events)
{
    const uint32_t C = c->spec.n_phi / 64;
    if (c->tun.peak_algo != 0 || c->tun.peak_rows != 0 || n_events == 0 || !c->d_peak_state) return false;
    if (c->spec.n_phi % 64 != 0 || (C != 4 && C != 8 && C != 16 && C != 32)) return false;
    return reinterpret_cast<uintptr_t>(acc) % (C == 4 ? 8 : 16) == 0;
}

uint64_t peaks_one_states(const hough_grid_spec &g, uint64_t max_events)
{
    return (max_events * g.n_d0 * ((g.n_qpt + 1) / 2) + 3) / 4;
}

hipError_t launch_peaks_one(hough_ctx *c, const uint16_t *acc, uint32_t n_events, hough_peak *peaks, uint64_t capacity,
                            uint64_t *poff, hipStream_t s)
{
    const uint32_t C = c->spec.n_phi / 64, R = one_rows(c, n_events);
    const uint32_t n_strips = (c->spec.n_qpt + R - 1) / R;
    const uint64_t n_tiles = uint64_t(n_events) * c->spec.n_d0 * n_strips;
    if (n_tiles > 0xFFFFFFFFull / 64) return hipErrorInvalidConfiguration;
    const bool d3 = c->spec.n_d0 > 1;
    // (cells per lane, rows, rows with a d0 axis) of the instances; R is one of them
    auto go = [&](auto cc, auto rr) {
        constexpr int kC = decltype(cc)::value, kR = decltype(rr)::value;
        constexpr int kR3 = std::min(kR, most_rows(kC, true)), kR1 = std::min(kR, most_rows(kC, false));
        constexpr int kMany = kC == 4 ? 16 : kC == 8 ? 8 : 4;
        const bool many = n_tiles >= kManyStrips;
        if (d3 && many)
            launch_one<kC, kR3, true, kMany>(s, acc, n_events, c, n_strips, n_tiles, poff, peaks, capacity);
        else if (d3)
            launch_one<kC, kR3, true, 4>(s, acc, n_events, c, n_strips, n_tiles, poff, peaks, capacity);
        else if (many)
            launch_one<kC, kR1, false, kMany>(s, acc, n_events, c, n_strips, n_tiles, poff, peaks, capacity);
        else
            launch_one<kC, kR1, false, 4>(s, acc, n_events, c, n_strips, n_tiles, poff, peaks, capacity);
    };
    auto rows = [&](auto cc) {
        using std::integral_constant;
        if (R == 16) return go(cc, integral_constant<int, 16>{});
        if (R == 8) return go(cc, integral_constant<int, 8>{});
        if (R == 4) return go(cc, integral_constant<int, 4>{});
        return go(cc, integral_constant<int, 2>{});
    };
    KernelTimer t;
    prof_begin(c, "peaks_one", s, &t);
    if (C == 4) rows(std::integral_constant<int, 4>{});
    else if (C == 8) rows(std::integral_constant<int, 8>{});
    else if (C == 16) rows(std::integral_constant<int, 16>{});
    else rows(std::integral_constant<int, 32>{});
    prof_end(c, s, &t);
    return hipGetLastError();
}

}  // namespace hough
