// Step 2 of the transform (Section 4, second step) in one launch: the row-
// window form of the peak search (peak_rows.h, k_peaks_rows.hip) with every
// strip's rows kept in registers, so that a strip is read once, counted,
// placed and written.
//
// A wavefront owns a strip of R consecutive q/pT rows of one event (and one
// d0 plane): it reads them with a halo row on either side (and, with a d0
// axis, the same rows of the planes beside it), decides every cell and keeps
// the decisions as bits.  A workgroup of several strips finds its place by a
// decoupled look-back over the workgroups before it (look_back.h); then each
// row's peaks are compacted in cell order through LDS and stored.
//
// Bound by HBM on batches (2 bytes per cell read, 8 bytes per peak written),
// by the chain load, count, look back, store on single events.  Against a
// count pass, a scan and a write pass: 4096 events of 512 x 512 (7.3e8 peaks)
// 1917 -> 1707 us (4.7 TB/s), 512 x 512 x 64 70 -> 58 us, one event of 256 x
// 256 15 -> 8 us, of 1024 x 1024 30 -> 10 us.  Fewer rows per strip cost more
// numbers: 4096 events with 8 and 4 rows 2164 and 3109 us (16: 1884), all
// with four strips per workgroup and two counters.
#include "look_back.h"
#include "peak_rows.h"

namespace hough {

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
    __shared__ uint32_t wave_cnt[WAVES], join_s[2];
    __shared__ uint64_t base_s;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t *state;
    const uint32_t number = look_back_join(states, n_states, counters, join_s, state);
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
        const uint64_t sum = look_back_place(state, counters, number, all, lane);
        if (lane == 0) base_s = sum;
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
    return max_events * g.n_d0 * ((g.n_qpt + 1) / 2);    // the counting form's workgroups, of at least two rows
}

// Local maxima of a counting accumulator in one launch.  A strip is R
// consecutive q/pT rows of one event (and d0 plane); a wave takes 256 cells of
// them, four per lane, and a workgroup one or several whole strips; neighbours across lanes by wave rotates, those of the first
// and last lane (and across the phi0 wrap) by one more load per row.  The
// rows' counts per wave give the cell order within the workgroup, the
// look-back its place.  Bound by the chain load, count, look back, store:
// 2048 x 2048 cells (16.8 MB): 16 us, where LDS tiles read in three passes took
// 121 us.
template <int R, bool D3>
__global__ void __launch_bounds__(1024)
k_peaks_count_one(const uint32_t *__restrict__ counts, uint32_t n_events, uint32_t n_qpt, uint32_t n_d0, uint32_t nphi,
                  uint32_t n_strips, uint64_t n_tiles, uint32_t thr, uint64_t *__restrict__ states, uint64_t n_states,
                  uint32_t *__restrict__ counters, uint64_t *__restrict__ poff, uint2 *__restrict__ peaks,
                  uint64_t capacity)
{
    __shared__ uint32_t cnt_s[R * 16], pre_s[R * 16], join_s[2];
    __shared__ uint64_t base_s;
    const uint32_t lane = threadIdx.x & 63, waves = nphi >> 8, parts = blockDim.x / (nphi >> 2);
    const uint32_t at = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = at % waves, part = at / waves;
    uint64_t *state;
    const uint32_t number = look_back_join(states, n_states, counters, join_s, state);
    const uint32_t planes = D3 ? n_d0 : 1u;
    const uint64_t tile = min(uint64_t(number) * parts + part, n_tiles - 1);
    const bool active = uint64_t(number) * parts + part < n_tiles;
    const uint32_t st = uint32_t(tile % n_strips), dp = uint32_t(tile / n_strips % planes);
    const uint32_t e = uint32_t(tile / n_strips / planes);
    const int r0 = int(st) * R;
    const uint64_t plane = uint64_t(n_qpt) * nphi;
    const uint32_t *ev = counts + (uint64_t(e) * planes + dp) * plane;
    const bool has_m = D3 && dp > 0, has_p = D3 && dp + 1 < planes;
    const uint32_t p0 = wave * 256 + lane * 4;
    const uint32_t edge = (lane == 63 ? wave * 256 + 256 : wave * 256 + nphi - 1) & (nphi - 1);

    struct Row {
        uint32_t v[4], x;                            // the lane's cells; the wave's neighbour cell on the lane's side
    };
    auto load = [&](const uint32_t *pl, int r) {
        const uint32_t *row = pl + uint64_t(min(max(r, 0), int(n_qpt) - 1)) * nphi;
        const uint4 a = *reinterpret_cast<const uint4 *>(row + p0);
        return Row{{a.x, a.y, a.z, a.w}, row[edge]};
    };
    // lr: the larger neighbour in the row; h: that and the cell itself
    // (everything 0 when the row is absent)
    auto maxima = [&](Row &w, bool present, uint32_t (&lr)[4], uint32_t (&h)[4]) {
        const uint32_t keep = present ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) w.v[j] &= keep;
        w.x &= keep;
        // the rotates with every lane active, then the choice
        const uint32_t fl = from_left(w.v[3]), fr = from_right(w.v[0]);
        const uint32_t l = lane == 0 ? w.x : fl, r = lane == 63 ? w.x : fr;
        lr[0] = max(l, w.v[1]);
        lr[1] = max(w.v[0], w.v[2]);
        lr[2] = max(w.v[1], w.v[3]);
        lr[3] = max(w.v[2], r);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = max(lr[j], w.v[j]);
    };
    Row row[R + 2], rowm[D3 ? R + 2 : 1], rowp[D3 ? R + 2 : 1];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        row[i] = load(ev, r0 - 1 + i);
        if constexpr (D3) {
            rowm[i] = load(has_m ? ev - plane : ev, r0 - 1 + i);
            rowp[i] = load(has_p ? ev + plane : ev, r0 - 1 + i);
        }
    }
    auto inside = [&](int i) { return r0 - 1 + i >= 0 && r0 - 1 + i < int(n_qpt); };
    // strips past the last one have no peaks
    auto beside = [&](int i, uint32_t (&nb)[4]) {     // the larger h of the neighbour planes' row i
        uint32_t lr[4], hm[4], hq[4];
        if constexpr (D3) {
            maxima(rowm[i], has_m && inside(i), lr, hm);
            maxima(rowp[i], has_p && inside(i), lr, hq);
#pragma unroll
            for (int j = 0; j < 4; ++j) nb[j] = max(hm[j], hq[j]);
        }
    };
    uint32_t bits[R], hp[4], lrc[4], hc[4], nbp[4], nbc[4], lrx[4];
    maxima(row[0], inside(0), lrx, hp);
    maxima(row[1], inside(1), lrc, hc);
    beside(0, nbp);
    beside(1, nbc);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        uint32_t lrn[4], hn[4], nbn[4];
        maxima(row[i + 2], inside(i + 2), lrn, hn);
        beside(i + 2, nbn);
        bits[i] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t mx = max(max(hp[j], hn[j]), lrc[j]);
            if (D3) mx = max(mx, max(max(nbp[j], nbc[j]), nbn[j]));
            const uint32_t v = row[i + 1].v[j];
            bits[i] |= (v >= thr && v >= mx && active && inside(i + 1) ? 1u : 0u) << j;
            hp[j] = hc[j];
            hc[j] = hn[j];
            lrc[j] = lrn[j];
            nbp[j] = nbc[j];
            nbc[j] = nbn[j];
        }
    }
    // the lane's place in its wave's part of each row
    uint32_t place[R];
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t n = uint32_t(__popc(bits[i]));
        const uint64_t b0 = __ballot(n & 1u), b1 = __ballot(n & 2u), b2 = __ballot(n & 4u);
        place[i] = uint32_t(__popcll(b0 & lt)) + 2 * uint32_t(__popcll(b1 & lt)) + 4 * uint32_t(__popcll(b2 & lt));
        if (lane == 0)
            cnt_s[(part * R + i) * waves + wave] = uint32_t(__popcll(b0)) + 2 * uint32_t(__popcll(b1)) + 4 * uint32_t(__popcll(b2));
    }
    __syncthreads();
    if (at == 0) {
        const uint32_t n = parts * R * waves;        // at most 64: 16 waves of four rows
        const uint32_t c = lane < n ? cnt_s[lane] : 0u;
        uint32_t inc = c;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d, 64);
            inc += lane >= d ? y : 0u;
        }
        if (lane < n) pre_s[lane] = inc - c;
        const uint32_t all = uint32_t(__builtin_amdgcn_readlane(int(inc), 63));
        const uint64_t sum = look_back_place(state, counters, number, all, lane);
        if (lane == 0) {
            base_s = sum;
            if (number == gridDim.x - 1) poff[n_events] = sum + all;
        }
    }
    __syncthreads();
    const uint64_t base = base_s;
    if (active && st == 0 && dp == 0 && wave == 0 && lane == 0) poff[e] = base + pre_s[part * R * waves];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        uint64_t pos = base + pre_s[(part * R + i) * waves + wave] + place[i];
        const uint32_t cell = (dp * n_qpt + uint32_t(r0 + i)) * nphi + p0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if ((bits[i] >> j) & 1u) {
                if (pos < capacity) peaks[pos] = make_uint2(cell + j, row[i + 1].v[j]);
                ++pos;
            }
        }
    }
}

// The default counting peak search for n_phi 256 to 4096.
bool peaks_count_one_usable(const hough_ctx *c, const uint32_t *counts, uint32_t n_events)
{
    const uint32_t n = c->spec.n_phi;
    return c->tun.peak_rows == 0 && n_events != 0 && c->d_peak_state && n >= 256 && n <= 4096 &&
           (reinterpret_cast<uintptr_t>(counts) & 15) == 0;
}

hipError_t launch_peaks_count_one(hough_ctx *c, const uint32_t *counts, uint32_t n_events, uint2 *peaks,
                                  uint64_t capacity, uint64_t *poff, hipStream_t s)
{
    const uint32_t nphi = c->spec.n_phi, n_qpt = c->spec.n_qpt, n_d0 = c->spec.n_d0;
    // four rows per workgroup, two while that leaves compute units idle
    const uint64_t four = uint64_t(n_events) * n_d0 * ((n_qpt + 3) / 4);
    const uint32_t R = four >= uint64_t(c->n_cu) ? 4 : 2;
    const uint32_t n_strips = (n_qpt + R - 1) / R;
    const uint64_t n_tiles = uint64_t(n_events) * n_d0 * n_strips;
    // short rows: several strips per workgroup once there are many (16 waves)
    const uint32_t parts = n_tiles >= 4 * uint64_t(c->n_cu) ? std::max(1u, 4096 / nphi) : 1u;
    const uint64_t wgs = (n_tiles + parts - 1) / parts;
    const uint32_t threads = parts * (nphi / 4);
    if (wgs > 0xFFFFFFFFull / threads) return hipErrorInvalidConfiguration;
    KernelTimer t;
    prof_begin(c, "peaks_count_one", s, &t);
    auto go = [&](auto rr, auto dd) {
        hipLaunchKernelGGL((k_peaks_count_one<decltype(rr)::value, decltype(dd)::value>), dim3(uint32_t(wgs)),
                           dim3(threads), 0, s, counts, n_events, n_qpt, n_d0, nphi, n_strips, n_tiles,
                           c->spec.threshold, c->d_peak_state, c->n_peak_state, c->d_counters + kPeakCounterBase, poff, peaks, capacity);
    };
    using std::integral_constant;
    if (R == 4 && n_d0 > 1) go(integral_constant<int, 4>{}, std::true_type{});
    else if (R == 4) go(integral_constant<int, 4>{}, std::false_type{});
    else if (n_d0 > 1) go(integral_constant<int, 2>{}, std::true_type{});
    else go(integral_constant<int, 2>{}, std::false_type{});
    prof_end(c, s, &t);
    return hipGetLastError();
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
