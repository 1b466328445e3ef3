// Candidate confirmation, first part: plateau clusters of the peak list.
//
// The non-strict local-maximum rule keeps every cell of a flat-topped ridge,
// so one track yields several adjacent peaks (Section 4 leaves the
// confirmation of candidates to later, more expensive computations).  Two
// peaks of one event are adjacent when their cells are neighbours in the
// local-maximum neighbourhood (3x3, 3x3x3 with a d0 axis; phi0 periodic);
// a cluster is a connected component of that relation.
//
// GPU form: lock-free union-find over peak-list indices.  A root is always
// hooked under a smaller index, so parent[i] <= i, a tree's root is its
// smallest member, and no cycle can form.
//   tile  -- a workgroup takes a tile of consecutive rows (of one event and
//            d0 plane): a contiguous range of the sorted peak list.  It
//            marks the tile's peaks in an LDS bitmap, a peak's index is its
//            rank in the bitmap, and rows are joined 32 cells at a time by
//            bit operations that leave one union per pair of touching runs;
//            the union-find runs in LDS, and parent[i] = the root within
//            the tile is written once;
//   seam  -- one wave per pair of neighbouring rows of different tiles (and
//            of different d0 planes) joins them the same way, in global
//            memory;
//   flat  -- parent[i] = root(i), found by a walk that writes nothing else;
//            per block of 4096 peaks, the root count;
//   scan  -- exclusive prefix of the block counts;
//   rank  -- roots get their global rank (= cluster index, ordered by first
//            peak) and initialise their cluster record;
//   acc   -- every peak replaces parent[i] by its cluster's index within
//            the event and adds its offsets to the cluster's sums (integer
//            sums, so the result does not depend on their order): first
//            over runs of adjacent lanes, then in an LDS table per block of
//            4096 peaks, so that a large cluster's record is updated once
//            per block.
// Rows of fewer than 64 or more than 8192 cells take the general form
// (init, link: a search per neighbour) in place of tile and seam.
// The parent array is the caller's per-peak label output; the ranks live in
// the context (max_peaks entries).
#include "hough_internal.h"

namespace hough {
namespace {

// The list passes (flat, rank, acc) take blocks of kClThreads * PER entries:
// few entries per thread while there are few blocks (a short list is bound
// by the serial steps of its blocks: 400,000 peaks, acc 46 us with 16 per
// thread on 98 blocks), 16 once there are more blocks than one pass of the
// scan's workgroup takes.
constexpr uint32_t kClThreads = 256, kClPerMax = 16, kClFewBlocks = 4096;

uint32_t cl_per(uint64_t n)
{
    for (uint32_t per : {1u, 4u})
        if (n <= uint64_t(kClFewBlocks) * kClThreads * per) return per;
    return kClPerMax;
}

struct ClParams {
    const uint2 *pk;         // peak records: x = cell, y = mask | popcount << 16
    const uint64_t *poff;    // [E + 1] event peak offsets
    uint32_t E;
    uint64_t cap;            // peak capacity
    uint32_t *par;           // [cap] parent, finally the label
    uint32_t *rank;          // [cap] cluster index of each root
    uint32_t *part;          // [nb] roots per block
    const uint64_t *part_off;// [nb + 1] their exclusive prefix
    uint64_t nb;
    hough_cluster *cl;
    uint64_t cl_cap;
    uint64_t *coff;          // [E + 1] event cluster offsets
    uint32_t n_phi, log2_phi, n_qpt, n_d0;
};

__device__ __forceinline__ uint64_t n_stored(const ClParams &P)
{
    return min(P.poff[P.E], P.cap);
}

// Largest event e with start(e) <= i (offsets ascending, as hough_peaks
// writes them).
__device__ __forceinline__ uint32_t event_of(const ClParams &P, uint64_t n, uint64_t i)
{
    uint32_t lo = 0, hi = P.E;
    while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (min(P.poff[m], n) <= i) lo = m;
        else hi = m;
    }
    return lo;
}

__device__ __forceinline__ uint32_t ld_par(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_par(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x with path halving.  Every parent is <= its child and a root is
// its own parent, so the walk strictly descends and ends.  (An entry above
// its index, which only a list that is not sorted leaves unset, also ends
// it: no walk leaves the list.)
__device__ uint32_t cl_find(uint32_t *par, uint32_t x)
{
    uint32_t next = ld_par(par + x);
    while (next < x) {
        const uint32_t nn = ld_par(par + next);
        if (nn < next) st_par(par + x, nn);
        x = next;
        next = nn;
    }
    return x;
}

// Root of x without writing.  The flattening pass uses this walk: a halving
// store from another thread could otherwise overwrite parent[x] after x's
// own thread has set it to the root, leaving an ancestor that is no root.
__device__ uint32_t cl_root(const uint32_t *par, uint32_t x)
{
    uint32_t next = ld_par(par + x);
    while (next < x) {
        x = next;
        next = ld_par(par + x);
    }
    return x;
}

// Unite the trees of a and b, hooking the larger root under the smaller.  A
// failed CAS means another thread hooked b meanwhile; every hook removes one
// of at most n roots, so the retries are bounded and the loop ends.
__device__ void cl_unite(uint32_t *par, uint32_t a, uint32_t b)
{
    for (;;) {
        a = cl_find(par, a);
        b = cl_find(par, b);
        if (a == b) return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        uint32_t expect = b;
        if (__hip_atomic_compare_exchange_strong(par + b, &expect, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
        if (expect > b) return;                      // unset: the list is not sorted
        b = expect;
    }
}

__global__ void __launch_bounds__(256) k_cl_init(ClParams P)
{
    const uint64_t n = n_stored(P);
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
        P.par[i] = uint32_t(i);
}

__global__ void __launch_bounds__(256) k_cl_link(ClParams P)
{
    const uint64_t n = n_stored(P);
    const uint32_t pmask = P.n_phi - 1;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x) {
        const uint32_t e = event_of(P, n, i);
        const uint64_t lo = min(P.poff[e], n);
        const uint64_t hi = max(min(P.poff[e + 1], n), lo);
        const uint32_t c = P.pk[i].x;
        const uint32_t p = c & pmask, row = c >> P.log2_phi;
        const uint32_t k = row % P.n_qpt, d = row / P.n_qpt;
        // first index in [b, t) whose cell is >= key (cells ascend)
        auto lower = [&](uint64_t b, uint64_t t, uint32_t key) {
            while (b < t) {
                const uint64_t m = (b + t) >> 1;
                if (P.pk[m].x < key) b = m + 1;
                else t = m;
            }
            return b;
        };
        // one neighbour cell c2, wherever it is: after i when larger (at
        // most c2 - c places on), before i when smaller (phi0 wrap)
        auto try_cell = [&](uint32_t c2) {
            uint64_t b, t;
            if (c2 > c) {
                b = i + 1;
                t = min(hi, i + 1 + uint64_t(c2 - c));
            } else if (c2 < c) {
                const uint64_t back = uint64_t(c - c2);
                b = i - lo > back ? i - back : lo;
                t = i;
            } else {
                return;
            }
            if (b >= t) return;
            const uint64_t j = lower(b, t, c2);
            if (j < t && P.pk[j].x == c2) cl_unite(P.par, uint32_t(i), uint32_t(j));
        };
        // three consecutive cells ca .. ca + 2 of a later row (no wrap inside):
        // one search, then at most three list entries
        auto try_triple = [&](uint32_t ca) {
            const uint64_t t = min(hi, i + 1 + uint64_t(ca + 2 - c));
            if (i + 1 >= t) return;
            for (uint64_t q = lower(i + 1, t, ca); q < t; ++q) {
                if (P.pk[q].x > ca + 2) break;
                cl_unite(P.par, uint32_t(i), uint32_t(q));
            }
        };
        auto try_row = [&](uint32_t rbase) {
            if (p != 0 && p != pmask) {
                try_triple(rbase | (p - 1));
            } else {
                try_cell(rbase | ((p - 1) & pmask));
                try_cell(rbase | p);
                try_cell(rbase | ((p + 1) & pmask));
            }
        };
        if (p != pmask) {
            if (i + 1 < hi && P.pk[i + 1].x == c + 1) cl_unite(P.par, uint32_t(i), uint32_t(i + 1));
        } else {
            try_cell(row << P.log2_phi);                // (k, 0) across the wrap
        }
        if (k + 1 < P.n_qpt) try_row((row + 1) << P.log2_phi);
        if (d + 1 < P.n_d0) {
            for (int dk = -1; dk <= 1; ++dk) {
                const int k2 = int(k) + dk;
                if (k2 < 0 || k2 >= int(P.n_qpt)) continue;
                try_row(((d + 1) * P.n_qpt + uint32_t(k2)) << P.log2_phi);
            }
        }
    }
}

// First index of [lo, hi) whose cell is >= key (cells ascend), 64 probes per
// step: uniform over the wave, every lane active.
__device__ __forceinline__ uint64_t wave_lower(const uint2 *pk, uint64_t lo, uint64_t hi, uint64_t key, uint32_t lane)
{
    while (hi - lo > 64) {
        const uint64_t step = (hi - lo + 63) >> 6;
        const uint64_t q = lo + lane * step;
        const uint32_t c = uint32_t(__popcll(__ballot(q < hi && pk[q].x < key)));
        if (c == 0) return lo;
        hi = min(hi, lo + c * step);
        lo = lo + (c - 1) * step + 1;
    }
    return lo + uint32_t(__popcll(__ballot(lo + lane < hi && pk[lo + lane].x < key)));
}

// Bits of the words of two rows, `a` and its neighbour `b`, at whose
// positions one union joins a run of a with a run of b that touches it:
// the first cell of each stretch both rows hold (`over`; cell 0 always,
// so that two full rows are joined too), and a cell of a whose only
// neighbours across are diagonal ones (`right`, `left`).  al, ar, bl, br:
// the rows shifted so that bit p holds cell p - 1 (l) or p + 1 (r).
struct Joins {
    uint32_t over, right, left;
};

__device__ __forceinline__ Joins row_joins(const uint32_t *a, const uint32_t *b, uint32_t w, uint32_t wr)
{
    const uint32_t wp = w ? w - 1 : wr - 1, wn = w + 1 < wr ? w + 1 : 0;
    const uint32_t av = a[w], bv = b[w];
    const uint32_t al = (av << 1) | (a[wp] >> 31), ar = (av >> 1) | (a[wn] << 31);
    const uint32_t bl = (bv << 1) | (b[wp] >> 31), br = (bv >> 1) | (b[wn] << 31);
    Joins j;
    j.over = av & bv & ~(al & bl & (w ? 0xFFFFFFFFu : 0xFFFFFFFEu));
    j.right = av & br & ~bv & ~ar;
    j.left = av & bl & ~bv & ~al;
    return j;
}

__device__ __forceinline__ uint32_t bit_rank(const uint32_t *bits, const uint32_t *pre, uint32_t cell)
{
    return pre[cell >> 5] + uint32_t(__popc(bits[cell >> 5] & ((1u << (cell & 31)) - 1u)));
}

// Exclusive prefix of the words' bit counts, by one wave; n a multiple of 2, up to 256.
__device__ __forceinline__ void bit_prefix(const uint32_t *bits, uint32_t *pre, uint32_t n, uint32_t lane)
{
    const uint32_t per = (n + 63) >> 6, b = min(lane * per, n), e = min(b + per, n);
    uint32_t s = 0;
    for (uint32_t i = b; i < e; ++i) s += uint32_t(__popc(bits[i]));
    uint32_t inc = s;
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        inc += lane >= d ? y : 0u;
    }
    uint32_t run = inc - s;
    for (uint32_t i = b; i < e; ++i) {
        pre[i] = run;
        run += uint32_t(__popc(bits[i]));
    }
}

__device__ __forceinline__ uint32_t tile_find(const uint32_t *par, uint32_t x)
{
    uint32_t next = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (next != x) {
        x = next;
        next = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return x;
}

// As cl_unite, in LDS: a minimum that finds its node no longer a root goes
// on with the parent it found; parents only decrease, so the loop ends.
__device__ __forceinline__ void tile_unite(uint32_t *par, uint32_t a, uint32_t b)
{
    for (;;) {
        a = tile_find(par, a);
        b = tile_find(par, b);
        if (a == b) return;
        const uint32_t lo = min(a, b), hi = max(a, b);
        const uint32_t old = atomicMin(&par[hi], lo);
        if (old == hi) return;
        a = lo;
        b = old;
    }
}

// A tile holds at most kTileCells cells: 50 KB of LDS, three workgroups per
// compute unit.  Bound by the LDS (bitmap, walks); 64 events of 512 x 512,
// 11.4M peaks: 99 us plus 47 us of seams (0.1 ms of traffic at 1.2 TB/s),
// where a search per neighbour and unions in global memory took 4.4 ms --
// in components of 180,000 peaks nearly every union contended for the same
// few roots; here a tile's unions stay in LDS and the global ones are one
// row in 16.
constexpr uint32_t kTileCells = 8192, kTileThreads = 512;

__global__ void __launch_bounds__(kTileThreads) k_cl_tile(ClParams P, uint32_t T, uint32_t tiles, uint64_t items)
{
    __shared__ uint32_t par[kTileCells];
    __shared__ uint16_t at[kTileCells];              // cell within the tile
    __shared__ uint32_t bits[kTileCells / 32], pre[kTileCells / 32];
    __shared__ uint64_t range[2];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint64_t n = n_stored(P);
  for (uint64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const uint32_t kt = uint32_t(item % tiles), d = uint32_t(item / tiles % P.n_d0);
    const uint32_t e = uint32_t(item / tiles / P.n_d0);
    const uint64_t lo = min(P.poff[e], n), hi = max(min(P.poff[e + 1], n), lo);
    const uint32_t rows = min(T, P.n_qpt - kt * T);
    const uint64_t key0 = uint64_t(d * P.n_qpt + kt * T) << P.log2_phi, cells = uint64_t(rows) << P.log2_phi;
    const uint32_t wr = P.n_phi >> 5, words = rows * wr;
    if (wave < 2) {
        const uint64_t x = wave_lower(P.pk, lo, hi, wave ? key0 + cells : key0, lane);
        if (lane == 0) range[wave] = x;
    }
    for (uint32_t i = t; i < words; i += kTileThreads) bits[i] = 0;
    __syncthreads();
    const uint64_t base = range[0];
    // a sorted list has at most one peak per cell
    const uint32_t cnt = uint32_t(min(range[1] > base ? range[1] - base : uint64_t(0), cells));
    for (uint32_t j = t; j < cnt; j += kTileThreads) {
        const uint32_t c = min(uint32_t(P.pk[base + j].x - key0), uint32_t(cells) - 1);
        atomicOr(&bits[c >> 5], 1u << (c & 31));
        at[j] = uint16_t(c);
        par[j] = j;
    }
    __syncthreads();
    if (wave == 0) bit_prefix(bits, pre, words, lane);
    __syncthreads();
    // every peak under the first peak of its run within its word, or, when
    // the run enters from the word before, under that word's last peak
    for (uint32_t j = t; j < cnt; j += kTileThreads) {
        const uint32_t c = at[j], w = c >> 5, b = c & 31;
        const uint32_t gaps = ~bits[w] & ((1u << b) - 1u);
        const uint32_t first = gaps ? 32u - uint32_t(__clz(gaps)) : 0u;
        uint32_t x = bit_rank(bits, pre, (w << 5) + first);
        if (first == 0 && (w & (wr - 1)) != 0 && (bits[w - 1] >> 31)) x = max(x, 1u) - 1;
        par[j] = min(x, j);
    }
    __syncthreads();
    // two threads per word of a row and the row after it
    for (uint32_t i = t; i < 2 * words; i += kTileThreads) {
        const uint32_t w = i >> 1, half = (i & 1u) ? 0xFFFF0000u : 0x0000FFFFu;
        const uint32_t r = w / wr, wc = w & (wr - 1);
        const uint32_t *a = bits + r * wr;
        if (wc == 0 && (i & 1u) == 0 && (a[0] & 1u) && (a[wr - 1] >> 31))        // across the phi0 wrap
            tile_unite(par, bit_rank(bits, pre, w << 5), bit_rank(bits, pre, ((w + wr) << 5) - 1));
        if (r + 1 >= rows) continue;
        const uint32_t row0 = r << P.log2_phi, row1 = row0 + P.n_phi, pm = P.n_phi - 1;
        const Joins q = row_joins(a, a + wr, wc, wr);
        for (uint32_t m = (q.over | q.right | q.left) & half; m; m &= m - 1) {
            const uint32_t b = uint32_t(__ffs(m)) - 1, p = (wc << 5) + b;
            const uint32_t x = bit_rank(bits, pre, row0 + p);
            if ((q.over >> b) & 1u) tile_unite(par, x, bit_rank(bits, pre, row1 + p));
            if ((q.right >> b) & 1u) tile_unite(par, x, bit_rank(bits, pre, row1 + ((p + 1) & pm)));
            if ((q.left >> b) & 1u) tile_unite(par, x, bit_rank(bits, pre, row1 + ((p - 1) & pm)));
        }
    }
    __syncthreads();
    for (uint32_t j = t; j < cnt; j += kTileThreads) P.par[base + j] = uint32_t(base + tile_find(par, j));
    __syncthreads();                                 // the LDS is reused by the next item
  }
}

// One workgroup per pair of rows: with dd == 0 the last row of a tile and
// the row after it, else row k of a d0 plane and row k + dk, dk = -1, 0, 1,
// of the next plane.  Latency bounds it (searches, then dependent walks
// towards the roots), so the searches run side by side, one per wave, and a
// thread joins an eighth of a word: 1024 x 1024 grid, 127 seams, 52 us with
// one wave per seam.
constexpr uint32_t kSeamThreads = 256;

__global__ void __launch_bounds__(kSeamThreads)
k_cl_seam(ClParams P, uint32_t T, uint32_t seams, uint32_t dd, uint64_t items)
{
    HOUGH_DYNAMIC_LDS(uint32_t, lds);                // bits and prefix of the two rows
    __shared__ uint64_t at[4];                       // their first and end list indices
    const uint32_t t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t wr = P.n_phi >> 5;
    const uint64_t n = n_stored(P);
  for (uint64_t item = blockIdx.x; item < items; item += gridDim.x) {
    uint32_t row[2], e;
    if (dd == 0) {
        const uint64_t ed = item / seams;
        e = uint32_t(ed / P.n_d0);
        row[0] = uint32_t(ed % P.n_d0) * P.n_qpt + uint32_t(item % seams + 1) * T - 1;
        row[1] = row[0] + 1;
    } else {
        const uint64_t per = uint64_t(P.n_d0 - 1) * P.n_qpt * 3, x = item % per;
        e = uint32_t(item / per);
        const uint32_t k = uint32_t(x / 3 % P.n_qpt), d = uint32_t(x / 3 / P.n_qpt);
        const int k2 = int(k) + int(x % 3) - 1;
        if (k2 < 0 || k2 >= int(P.n_qpt)) continue;
        row[0] = d * P.n_qpt + k;
        row[1] = (d + 1) * P.n_qpt + uint32_t(k2);
    }
    const uint64_t lo = min(P.poff[e], n), hi = max(min(P.poff[e + 1], n), lo);
    for (uint32_t i = t; i < 2 * wr; i += kSeamThreads) lds[i] = 0;
    const uint64_t x = wave_lower(P.pk, lo, hi, uint64_t(row[wave >> 1] + (wave & 1u)) << P.log2_phi, lane);
    if (lane == 0) at[wave] = x;
    __syncthreads();
    // an empty row joins nothing (every thread sees the same bounds)
    const bool both = at[0] < at[1] && at[2] < at[3];
    if (both) {
        for (uint32_t s = 0; s < 2; ++s) {
            const uint64_t key = uint64_t(row[s]) << P.log2_phi, end = min(at[2 * s + 1], at[2 * s] + P.n_phi);
            for (uint64_t i = at[2 * s] + t; i < end; i += kSeamThreads) {
                const uint32_t off = uint32_t(P.pk[i].x - key) & (P.n_phi - 1);
                atomicOr(&lds[s * wr + (off >> 5)], 1u << (off & 31));
            }
        }
        __syncthreads();
        if (wave < 2) bit_prefix(lds + wave * wr, lds + (2 + wave) * wr, wr, lane);
        __syncthreads();
        const uint32_t pm = P.n_phi - 1;
        const uint32_t *bits[2] = {lds, lds + wr}, *pre[2] = {lds + 2 * wr, lds + 3 * wr};
        const uint32_t b0 = uint32_t(at[0]), b1 = uint32_t(at[2]);
        for (uint32_t i = t; i < 8 * wr; i += kSeamThreads) {
            const uint32_t w = i >> 3;
            const Joins q = row_joins(bits[0], bits[1], w, wr);
            for (uint32_t m = (q.over | q.right | q.left) & (0xFu << (4 * (i & 7u))); m; m &= m - 1) {
                const uint32_t b = uint32_t(__ffs(m)) - 1, p = (w << 5) + b;
                const uint32_t y = b0 + bit_rank(bits[0], pre[0], p);
                if ((q.over >> b) & 1u) cl_unite(P.par, y, b1 + bit_rank(bits[1], pre[1], p));
                if ((q.right >> b) & 1u) cl_unite(P.par, y, b1 + bit_rank(bits[1], pre[1], (p + 1) & pm));
                if ((q.left >> b) & 1u) cl_unite(P.par, y, b1 + bit_rank(bits[1], pre[1], (p - 1) & pm));
            }
        }
    }
    __syncthreads();                                 // the LDS is reused by the next item
  }
}

// Roots per block of list entries, parents flattened.
template <uint32_t PER>
__global__ void __launch_bounds__(kClThreads) k_cl_flat(ClParams P)
{
    __shared__ uint32_t wsum[kClThreads / 64];
    const uint64_t n = n_stored(P);
    const uint64_t base = uint64_t(blockIdx.x) * (kClThreads * PER);
    uint32_t roots = 0;
    if (base < n) {
#pragma unroll 4
        for (uint32_t j = 0; j < PER; ++j) {
            const uint64_t i = base + uint64_t(j) * kClThreads + threadIdx.x;
            if (i < n) {
                const uint32_t r = cl_root(P.par, uint32_t(i));
                st_par(P.par + i, r);
                roots += r == uint32_t(i);
            }
        }
    }
    for (uint32_t off = 32; off > 0; off >>= 1) roots += __shfl_down(roots, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = roots;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (uint32_t w = 0; w < kClThreads / 64; ++w) s += wsum[w];
        P.part[blockIdx.x] = s;
    }
}

// Event of list entry i >= i0, given the event e0 of i0 (a block's entries
// lie in few events).
__device__ __forceinline__ uint32_t event_from(const ClParams &P, uint64_t n, uint64_t i, uint32_t e0)
{
    while (e0 + 1 < P.E && min(P.poff[e0 + 1], n) <= i) ++e0;
    return e0;
}

// Global rank of every root (in list order) and its cluster record.
template <uint32_t PER>
__global__ void __launch_bounds__(kClThreads) k_cl_rank(ClParams P)
{
    constexpr uint32_t kWaves = kClThreads / 64;
    __shared__ uint32_t wsum[PER * kWaves];
    const uint64_t n = n_stored(P);
    const uint64_t base = uint64_t(blockIdx.x) * (kClThreads * PER);
    if (base >= n) return;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t bal[PER];
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint64_t i = base + uint64_t(j) * kClThreads + threadIdx.x;
        bal[j] = __ballot(i < n && P.par[i] == uint32_t(i));
        if (lane == 0) wsum[j * kWaves + wave] = uint32_t(__popcll(bal[j]));
    }
    __syncthreads();
    uint64_t run = P.part_off[blockIdx.x];
    const uint32_t e0 = event_of(P, n, base);
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        uint32_t before = 0, total = 0;
        for (uint32_t w = 0; w < kWaves; ++w) {
            before += w < wave ? wsum[j * kWaves + w] : 0u;
            total += wsum[j * kWaves + w];
        }
        if ((bal[j] >> lane) & 1u) {
            const uint64_t i = base + uint64_t(j) * kClThreads + threadIdx.x;
            const uint64_t r = run + before + uint32_t(__popcll(bal[j] & ((uint64_t(1) << lane) - 1)));
            P.rank[i] = uint32_t(r);
            if (r < P.cl_cap) {
                const uint32_t e = event_from(P, n, i, e0);
                const uint2 rec = P.pk[i];
                hough_cluster h;
                h.first = uint32_t(i - min(P.poff[e], n));
                h.popcount = uint16_t(rec.y >> 16);
                h.mask_or = uint16_t(rec.y);
                h.n_peaks = 1;
                h.sum_dk = 0;
                h.sum_dp = 0;
                h.sum_dd = 0;
                P.cl[r] = h;
            }
        }
        run += total;
    }
}

// Adds a partial sum to a cluster's record.  n_peaks (low word, never
// carries) and sum_dk (high word) in one add.
// m: the members' mask bits that the root's mask lacks.
__device__ __forceinline__ void cl_add(hough_cluster *h, unsigned long long cnt_dk, int32_t dp, int32_t dd, uint32_t m)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(&h->n_peaks), cnt_dk);
    if (dp) atomicAdd(&h->sum_dp, dp);
    if (dd) atomicAdd(&h->sum_dd, dd);
    if (m) atomicOr(reinterpret_cast<uint32_t *>(&h->popcount), m << 16);
}

// Labels (cluster index within the event), member sums, event offsets.  Runs of adjacent lanes in one cluster (a
// flat plateau along phi0 is a run of consecutive list entries) are summed
// by segmented shuffles, and each run's last lane adds the run to the
// block's table of cluster sums in LDS (to the record itself when four
// probes find no slot); the table is added to the records at the end.
// Without the table every run of a large cluster updates its one record:
// 64 events of 512 x 512, 11.4M peaks, 547 us; with it 98 us.  (A read of
// the record's mask before the OR, past the L2, cost 40 of 65 us on a short
// list: the root's mask decides instead.)
constexpr uint32_t kClSlots = 512;

template <uint32_t PER>
__global__ void __launch_bounds__(kClThreads) k_cl_acc(ClParams P)
{
    __shared__ uint32_t key_s[kClSlots], mask_s[kClSlots];
    __shared__ unsigned long long cnt_s[kClSlots];
    __shared__ int32_t dp_s[kClSlots], dd_s[kClSlots];
    const uint64_t n = n_stored(P);
    const uint64_t total = P.part_off[P.nb];
    const uint64_t g0 = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x, gs = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t e = g0; e <= P.E; e += gs) {
        const uint64_t s = min(P.poff[e], n);
        P.coff[e] = s < n ? P.rank[s] : total;
    }
    const uint64_t base = uint64_t(blockIdx.x) * (kClThreads * PER);
    if (base >= n) return;                           // uniform over the block
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    for (uint32_t i = threadIdx.x; i < kClSlots; i += kClThreads) {
        key_s[i] = kNone;
        mask_s[i] = 0;
        cnt_s[i] = 0;
        dp_s[i] = 0;
        dd_s[i] = 0;
    }
    __syncthreads();
    const uint32_t pmask = P.n_phi - 1, lane = threadIdx.x & 63;
    const int32_t half = int32_t(P.n_phi >> 1);
    const uint64_t lanes_below = lane == 63 ? ~uint64_t(0) : (uint64_t(2) << lane) - 1;
    const uint32_t e0 = event_of(P, n, base);
    for (uint32_t j = 0; j < PER; ++j) {
        const uint64_t i = base + uint64_t(j) * kClThreads + threadIdx.x;
        uint32_t key = kNone, cnt = 0, m = 0;
        int32_t dk = 0, dp = 0, dd = 0;
        if (i < n) {
            const uint32_t e = event_from(P, n, i, e0);
            const uint64_t lo = min(P.poff[e], i);
            const uint32_t r = P.par[i];
            const uint32_t cid = P.rank[r];
            P.par[i] = cid - P.rank[lo];
            if (r != uint32_t(i) && cid < P.cl_cap) {
                const uint2 rec = P.pk[i], root = P.pk[r];
                const uint32_t c = rec.x, cr = root.x;
                const uint32_t row = c >> P.log2_phi, rowr = cr >> P.log2_phi;
                key = cid;
                cnt = 1;
                if (P.n_d0 > 1) {
                    dk = int32_t(row % P.n_qpt) - int32_t(rowr % P.n_qpt);
                    dd = int32_t(row / P.n_qpt) - int32_t(rowr / P.n_qpt);
                } else {
                    dk = int32_t(row) - int32_t(rowr);
                }
                dp = int32_t((c - cr) & pmask);
                if (dp >= half) dp -= int32_t(P.n_phi);
                m = rec.y & ~root.y & 0xFFFFu;
            }
        }
        // segmented inclusive sums over runs of equal keys
        const uint32_t prev = __shfl_up(key, 1, 64);
        const uint64_t heads = __ballot(lane == 0 || prev != key);
        const uint32_t start = 63u - uint32_t(__clzll(heads & lanes_below));
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t c2 = __shfl_up(cnt, d, 64), m2 = __shfl_up(m, d, 64);
            const int32_t k2 = __shfl_up(dk, d, 64), p2 = __shfl_up(dp, d, 64);
            const int32_t d2 = P.n_d0 > 1 ? __shfl_up(dd, d, 64) : 0;
            if (lane >= start + d) {
                cnt += c2;
                m |= m2;
                dk += k2;
                dp += p2;
                dd += d2;
            }
        }
        const bool tail = lane == 63 || ((heads >> (lane + 1)) & 1u);
        if (tail && key != kNone) {
            const unsigned long long cd = (static_cast<unsigned long long>(uint32_t(dk)) << 32) | cnt;
            uint32_t s = (key * 2654435761u) >> 23;
            bool put = false;
            for (uint32_t probe = 0; probe < 4 && !put; ++probe, s = (s + 1) & (kClSlots - 1)) {
                const uint32_t was = atomicCAS(&key_s[s], kNone, key);
                if (was == kNone || was == key) {
                    atomicAdd(&cnt_s[s], cd);
                    if (dp) atomicAdd(&dp_s[s], dp);
                    if (dd) atomicAdd(&dd_s[s], dd);
                    if (m) atomicOr(&mask_s[s], m);
                    put = true;
                }
            }
            if (!put) cl_add(P.cl + key, cd, dp, dd, m);
        }
    }
    __syncthreads();
    for (uint32_t s = threadIdx.x; s < kClSlots; s += kClThreads)
        if (key_s[s] != kNone) cl_add(P.cl + key_s[s], cnt_s[s], dp_s[s], dd_s[s], mask_s[s]);
}

uint32_t grid_for(const hough_ctx *c, uint64_t n)
{
    return uint32_t(std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, uint64_t(c->n_cu) * 16)));
}

}  // namespace

uint64_t cluster_blocks(uint64_t n)
{
    return (n + uint64_t(kClThreads) * cl_per(n) - 1) / (uint64_t(kClThreads) * cl_per(n));
}

// a call with a smaller list may take more, shorter blocks
uint64_t cluster_blocks_max(uint64_t n)
{
    return n ? std::max<uint64_t>(cluster_blocks(n), kClFewBlocks) : 0;
}

hipError_t launch_clusters(hough_ctx *c, const hough_peak *peaks, uint64_t peak_capacity, const uint64_t *poff,
                           uint32_t n_events, uint32_t *labels, hough_cluster *clusters, uint64_t capacity,
                           uint64_t *coff, hipStream_t s)
{
    if (n_events == 0) return launch_fill_u32(c, reinterpret_cast<uint32_t *>(coff), 0u, 2, s);
    ClParams P{};
    P.pk = reinterpret_cast<const uint2 *>(peaks);
    P.poff = poff;
    P.E = n_events;
    P.cap = peak_capacity;
    P.par = labels;
    P.rank = c->d_cl_rank;
    P.part = c->d_cl_part;
    P.part_off = c->d_cl_part_off;
    P.nb = cluster_blocks(peak_capacity);
    P.cl = clusters;
    P.cl_cap = capacity;
    P.coff = coff;
    P.n_phi = c->spec.n_phi;
    P.log2_phi = c->log2_phi;
    P.n_qpt = c->spec.n_qpt;
    P.n_d0 = c->spec.n_d0;
    KernelTimer t;
    const uint32_t nphi = c->spec.n_phi;
    if (nphi >= 64 && nphi <= kTileCells) {
        // rows per tile: as many as the LDS holds
        const uint32_t T = std::min(kTileCells / nphi, c->spec.n_qpt);
        const uint32_t tiles = (c->spec.n_qpt + T - 1) / T;
        const uint64_t planes = uint64_t(n_events) * c->spec.n_d0;
        auto grid = [](uint64_t items) { return dim3(uint32_t(std::min<uint64_t>(items, 1u << 20))); };
        prof_begin(c, "cluster_link", s, &t);
        hipLaunchKernelGGL(k_cl_tile, grid(planes * tiles), dim3(kTileThreads), 0, s, P, T, tiles, planes * tiles);
        const size_t lds = size_t(nphi / 32) * 16;
        if (const uint64_t m = planes * (tiles - 1))
            hipLaunchKernelGGL(k_cl_seam, grid(m), dim3(kSeamThreads), lds, s, P, T, tiles - 1, 0u, m);
        if (const uint64_t m = uint64_t(n_events) * (c->spec.n_d0 - 1) * c->spec.n_qpt * 3)
            hipLaunchKernelGGL(k_cl_seam, grid(m), dim3(kSeamThreads), lds, s, P, T, 1u, 1u, m);
        prof_end(c, s, &t);
    } else {
        const uint32_t g = grid_for(c, peak_capacity);
        prof_begin(c, "cluster_init", s, &t);
        hipLaunchKernelGGL(k_cl_init, dim3(g), dim3(256), 0, s, P);
        prof_end(c, s, &t);
        prof_begin(c, "cluster_link", s, &t);
        hipLaunchKernelGGL(k_cl_link, dim3(g), dim3(256), 0, s, P);
        prof_end(c, s, &t);
    }
    const uint32_t per = cl_per(peak_capacity);
    auto pick = [&](auto one, auto four, auto most) { return per == 1 ? one : per == 4 ? four : most; };
    if (P.nb) {
        prof_begin(c, "cluster_flat", s, &t);
        hipLaunchKernelGGL(pick(k_cl_flat<1>, k_cl_flat<4>, k_cl_flat<kClPerMax>), dim3(uint32_t(P.nb)),
                           dim3(kClThreads), 0, s, P);
        prof_end(c, s, &t);
    }
    hipError_t e = launch_scan_counts(c, c->d_cl_part, P.nb, c->d_cl_part_off, 0, nullptr, s);
    if (e != hipSuccess) return e;
    if (P.nb) {
        prof_begin(c, "cluster_rank", s, &t);
        hipLaunchKernelGGL(pick(k_cl_rank<1>, k_cl_rank<4>, k_cl_rank<kClPerMax>), dim3(uint32_t(P.nb)),
                           dim3(kClThreads), 0, s, P);
        prof_end(c, s, &t);
    }
    prof_begin(c, "cluster_acc", s, &t);
    hipLaunchKernelGGL(pick(k_cl_acc<1>, k_cl_acc<4>, k_cl_acc<kClPerMax>),
                       dim3(std::max<uint32_t>(uint32_t(P.nb), 1u)), dim3(kClThreads), 0, s, P);
    prof_end(c, s, &t);
    return hipGetLastError();
}

}  // namespace hough
