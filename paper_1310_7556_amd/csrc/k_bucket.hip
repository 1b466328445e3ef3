// Hit ingest: per-event counting sorts that group hits by layer (so a vote
// wavefront works on one layer at a time and the layer bit and the offset
// of a row are wave-uniform), and, for the rz stage and the cluster fit, the
// hit index: hits by (layer, coarse azimuth bucket), so the member hits of a
// candidate cell are found in a few buckets.  Order inside a group is
// unspecified: votes are OR/count updates and every result is independent of
// hit order.
#include "device_hits.h"
#include "hough_internal.h"

namespace hough {

// One workgroup per event: layer histogram, prefix, scatter.
__global__ void __launch_bounds__(1024)
k_bucket_layers(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi,
                const uint64_t *__restrict__ offs, uint64_t n_hits, uint32_t n_layers,
                uint32_t *__restrict__ out_phi, uint32_t *__restrict__ layer_off)
{
    __shared__ uint32_t cnt[kMaxLayers], cur[kMaxLayers];
    const uint32_t e = blockIdx.x, t = threadIdx.x;
    uint64_t b, end;
    event_range(offs, e, n_hits, b, end);
    if (t < kMaxLayers) cnt[t] = 0;
    __syncthreads();
    for (uint64_t i = b + t; i < end; i += blockDim.x) {
        const uint32_t l = layer[i];
        if (l < n_layers) atomicAdd(&cnt[l], 1u);
    }
    __syncthreads();
    if (t == 0) {
        uint32_t run = 0;
        uint32_t *lo = layer_off + size_t(e) * (n_layers + 1);
        for (uint32_t l = 0; l < n_layers; ++l) {
            cur[l] = run;
            lo[l] = run;
            run += cnt[l];
        }
        lo[n_layers] = run;
    }
    __syncthreads();
    for (uint64_t i = b + t; i < end; i += blockDim.x) {
        const uint32_t l = layer[i];
        if (l < n_layers) {
            const uint32_t pos = atomicAdd(&cur[l], 1u);
            out_phi[b + pos] = phi[i];
        }
    }
}

// Split form of the layer sort for batches of few events: event e is cut
// into K parts of consecutive hits, one 256-thread workgroup each.
// k_layer_count counts a part's hits per layer (one ballot per layer per 64
// hits, no atomics); k_split_plan (one wave per event) turns the parts'
// counts into the event's layer offsets and each part's first position per
// layer; k_layer_scatter places a part's hits in input order.  The result
// is a stable counting sort, so the order inside a layer is the input order.
constexpr uint32_t kSplitThreads = 256;

__device__ __forceinline__ void part_range(const uint64_t *offs, uint32_t e, uint32_t k, uint32_t K, uint64_t n,
                                           uint64_t &pb, uint64_t &pe)
{
    uint64_t b, end;
    event_range(offs, e, n, b, end);
    const uint64_t len = end - b;
    pb = b + len * k / K;
    pe = b + len * (k + 1) / K;
}

__global__ void __launch_bounds__(kSplitThreads)
k_layer_count(const uint8_t *__restrict__ layer, const uint64_t *__restrict__ offs, uint64_t n_hits,
              uint32_t n_layers, uint32_t K, uint32_t *__restrict__ part_cnt)
{
    __shared__ uint32_t wc[kSplitThreads / 64][kMaxLayers];
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    uint64_t pb, pe;
    part_range(offs, blockIdx.x / K, blockIdx.x % K, K, n_hits, pb, pe);
    uint32_t cnt[kMaxLayers];
#pragma unroll
    for (uint32_t q = 0; q < kMaxLayers; ++q) cnt[q] = 0;
    for (uint64_t i0 = pb + wave * 64; i0 < pe; i0 += kSplitThreads) {
        const uint64_t i = i0 + lane;
        const uint32_t l = i < pe ? layer[i] : 0xFFu;
#pragma unroll
        for (uint32_t q = 0; q < kMaxLayers; ++q)
            if (q < n_layers) cnt[q] += uint32_t(__popcll(__ballot(l == q)));
    }
    if (lane == 0) {
#pragma unroll
        for (uint32_t q = 0; q < kMaxLayers; ++q) wc[wave][q] = cnt[q];
    }
    __syncthreads();
    if (t < n_layers) {
        uint32_t s = 0;
        for (uint32_t w = 0; w < kSplitThreads / 64; ++w) s += wc[w][t];
        part_cnt[size_t(blockIdx.x) * kSplitBins + t] = s;
    }
}

// One wave per event: for each of the event's bins (layers) in order, the
// bin's start is the sum of all earlier bins, and part k's first position
// in bin v is the start plus the counts of parts 0..k-1 in v.  bin_off
// receives the n_bins + 1 starts (relative to the event) when not null.
__global__ void __launch_bounds__(64)
k_split_plan(const uint32_t *__restrict__ part_cnt, uint32_t n_bins, uint32_t K, uint32_t *__restrict__ part_base,
             uint32_t *__restrict__ bin_off)
{
    const uint32_t e = blockIdx.x, lane = threadIdx.x;
    uint32_t run = 0;
    for (uint32_t v = 0; v < n_bins; ++v) {
        const uint32_t x = lane < K ? part_cnt[(size_t(e) * K + lane) * kSplitBins + v] : 0u;
        uint32_t incl = x;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            incl += lane >= d ? y : 0u;
        }
        if (lane < K) part_base[(size_t(e) * K + lane) * kSplitBins + v] = run + incl - x;
        if (bin_off && lane == 0) bin_off[size_t(e) * (n_bins + 1) + v] = run;
        run += __shfl(incl, 63, 64);
    }
    if (bin_off && lane == 0) bin_off[size_t(e) * (n_bins + 1) + n_bins] = run;
}

__global__ void __launch_bounds__(kSplitThreads)
k_layer_scatter(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi,
                const uint64_t *__restrict__ offs, uint64_t n_hits, uint32_t n_layers, uint32_t K,
                const uint32_t *__restrict__ part_base, uint32_t *__restrict__ out_phi)
{
    __shared__ uint32_t wc[kSplitThreads / 64][kMaxLayers];
    __shared__ uint32_t base[kMaxLayers];
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t e = blockIdx.x / K;
    uint64_t b, end, pb, pe;
    event_range(offs, e, n_hits, b, end);
    part_range(offs, e, blockIdx.x % K, K, n_hits, pb, pe);
    if (t < n_layers) base[t] = part_base[size_t(blockIdx.x) * kSplitBins + t];
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1ull;
    // rounds of 256 consecutive hits, wave w taking the w-th 64
    for (uint64_t r0 = pb; r0 < pe; r0 += kSplitThreads) {
        const uint64_t i = r0 + t;
        const bool ok = i < pe;
        const uint32_t l = ok ? layer[i] : 0xFFu;
        const uint32_t ph = ok ? phi[i] : 0u;
        uint32_t rank = 0;
#pragma unroll
        for (uint32_t q = 0; q < kMaxLayers; ++q) {
            if (q < n_layers) {
                const uint64_t m = __ballot(l == q);
                if (lane == 0) wc[wave][q] = uint32_t(__popcll(m));
                if (l == q) rank = uint32_t(__popcll(m & lt));
            }
        }
        __syncthreads();
        if (l < n_layers) {
            uint32_t pos = base[l] + rank;
            for (uint32_t w = 0; w < wave; ++w) pos += wc[w][l];
            out_phi[b + pos] = ph;
        }
        __syncthreads();
        if (t < n_layers) {
            uint32_t s = 0;
            for (uint32_t w = 0; w < kSplitThreads / 64; ++w) s += wc[w][t];
            base[t] += s;
        }
        __syncthreads();
    }
}

// Exclusive prefix of n LDS counters in place, by all NT threads (a multiple
// of 64); returns the total.  wsum: NT / 64 entries of LDS.
template <uint32_t NT>
__device__ uint32_t block_prefix(uint32_t *v, uint32_t n, uint32_t *wsum)
{
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t per = (n + NT - 1) / NT, b = min(t * per, n), e = min(b + per, n);
    uint32_t s = 0;
    for (uint32_t i = b; i < e; ++i) s += v[i];
    uint32_t inc = s;
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        inc += lane >= d ? y : 0u;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t run = inc - s, total = 0;
    for (uint32_t w = 0; w < NT / 64; ++w) {
        run += w < wave ? wsum[w] : 0u;
        total += wsum[w];
    }
    for (uint32_t i = b; i < e; ++i) {
        const uint32_t x = v[i];
        v[i] = run;
        run += x;
    }
    __syncthreads();
    return total;
}

// The hit index: `out` holds the event's hits by (layer, bucket), the bucket
// being the top `bits` bits of phi -- phi alone, or {phi, z} records, which a
// member search reads with one load -- and bucket_off[(e * L + l) * (NB + 1)
// + i] is the start of bucket i relative to the event start.
template <bool Z>
struct IndexRec {
    using type = uint32_t;
    static __device__ __forceinline__ type make(uint32_t ph, const int32_t *, uint64_t) { return ph; }
    static __device__ __forceinline__ uint32_t phi(type r) { return r; }
};
template <>
struct IndexRec<true> {
    using type = uint2;
    static __device__ __forceinline__ type make(uint32_t ph, const int32_t *z, uint64_t i)
    {
        return make_uint2(ph, uint32_t(z[i]));
    }
    static __device__ __forceinline__ uint32_t phi(type r) { return r.x; }
};

// Whole form: one workgroup per (event, layer), in one launch.  It reads all
// of the event's hits twice (they stay in the L2: 5 bytes per hit and layer)
// and sorts its layer's; the layer's start is the number of hits in lower
// layers.
constexpr uint32_t kIndexThreads = 1024;

template <bool Z>
__global__ void __launch_bounds__(kIndexThreads)
k_hit_index(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi, const int32_t *__restrict__ z,
            const uint64_t *__restrict__ offs, uint64_t n_hits, uint32_t n_layers, uint32_t bits, int vec,
            typename IndexRec<Z>::type *__restrict__ out, uint32_t *__restrict__ bucket_off)
{
    __shared__ uint32_t hist[1u << kMaxBucketBits];
    __shared__ uint32_t wsum[kIndexThreads / 64];
    __shared__ uint32_t base_s;
    const uint32_t e = blockIdx.x / n_layers, l = blockIdx.x % n_layers, t = threadIdx.x;
    const uint32_t nb = 1u << bits, sh = 32 - bits;
    uint64_t b, end;
    event_range(offs, e, n_hits, b, end);
    for (uint32_t i = t; i < nb; i += kIndexThreads) hist[i] = 0;
    if (t == 0) base_s = 0;
    __syncthreads();
    uint32_t lower = 0;
    indexed_hits(layer, phi, b, end, t, kIndexThreads, vec, [&](uint32_t hl, uint32_t ph, uint64_t) {
        if (hl == l) atomicAdd(&hist[ph >> sh], 1u);
        lower += hl < l ? 1u : 0u;
    });
    for (uint32_t d = 32; d > 0; d >>= 1) lower += __shfl_down(lower, d, 64);
    if ((t & 63) == 0) atomicAdd(&base_s, lower);
    __syncthreads();
    const uint32_t total = block_prefix<kIndexThreads>(hist, nb, wsum), base = base_s;
    uint32_t *bo = bucket_off + (size_t(e) * n_layers + l) * (nb + 1);
    for (uint32_t i = t; i < nb; i += kIndexThreads) bo[i] = base + hist[i];
    if (t == 0) bo[nb] = base + total;
    __syncthreads();
    indexed_hits(layer, phi, b, end, t, kIndexThreads, vec, [&](uint32_t hl, uint32_t ph, uint64_t i) {
        if (hl == l) out[b + base + atomicAdd(&hist[ph >> sh], 1u)] = IndexRec<Z>::make(ph, z, i);
    });
}

// Split form: an event's hits are cut into K parts and sorted by (layer,
// sector), a sector being the top bits of the bucket (16 of them, so that a
// bin's hits suit one small workgroup), then each bin by bucket.
// k_sector_count counts a part's hits per bin; k_sector_plan (one workgroup
// per event) turns the counts into the bins' starts and each part's place in
// them; k_sector_scatter moves the hits; k_sector_sort sorts a bin.  Both
// moves sort in LDS first, so that memory is written in runs (written hit by
// hit, 16 events of 150,000 hits took 77 us: every 4-byte store was a request
// of its own).
__global__ void __launch_bounds__(kSplitThreads)
k_sector_count(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi, const uint64_t *__restrict__ offs,
               uint64_t n_hits, uint32_t n_layers, uint32_t sbits, uint32_t K, int vec, uint32_t *__restrict__ part_cnt)
{
    __shared__ uint32_t hist[kSectorBins];
    const uint32_t t = threadIdx.x;
    uint64_t pb, pe;
    part_range(offs, blockIdx.x / K, blockIdx.x % K, K, n_hits, pb, pe);
    hist[t] = 0;
    __syncthreads();
    indexed_hits(layer, phi, pb, pe, t, kSplitThreads, vec, [&](uint32_t l, uint32_t ph, uint64_t) {
        if (l < n_layers) atomicAdd(&hist[(l << sbits) + (ph >> (32 - sbits))], 1u);
    });
    __syncthreads();
    part_cnt[size_t(blockIdx.x) * kSectorBins + t] = hist[t];
}

// part_cnt[k][bin] becomes the part's first position in the bin, relative to
// the event; bin_off[e][0 .. kSectorBins]: the bins' starts.  Bound by the
// walk over the event's parts, so four threads share a bin, each a quarter of
// them, sixteen loads together (one event of 60,000 hits, 58 parts, 7.4 -> 3.8
// us; 16 events of 100 to 10,000 tracks 9.0 -> 6.7; one event of 600,000 hits,
// the whole index 54 -> 49).
constexpr uint32_t kPlanShares = 4, kPlanThreads = kPlanShares * kSectorBins, kPlanBatch = 16;

__global__ void __launch_bounds__(kPlanThreads)
k_sector_plan(uint32_t K, uint32_t *__restrict__ part_cnt, uint32_t *__restrict__ bin_off)
{
    __shared__ uint32_t share_s[kPlanShares][kSectorBins], tot[kSectorBins];
    __shared__ uint32_t wsum[kPlanThreads / 64];
    const uint32_t bin = threadIdx.x % kSectorBins, share = threadIdx.x / kSectorBins;
    const uint32_t k0 = K * share / kPlanShares, k1 = K * (share + 1) / kPlanShares;
    uint32_t *pc = part_cnt + size_t(blockIdx.x) * K * kSectorBins + bin;
    auto batch = [&](uint32_t k, uint32_t (&x)[kPlanBatch]) {
#pragma unroll
        for (uint32_t u = 0; u < kPlanBatch; ++u) x[u] = pc[size_t(min(k + u, k1 - 1)) * kSectorBins];
    };
    uint32_t s = 0, x[kPlanBatch];
    for (uint32_t k = k0; k < k1; k += kPlanBatch) {
        batch(k, x);
#pragma unroll
        for (uint32_t u = 0; u < kPlanBatch; ++u) s += k + u < k1 ? x[u] : 0u;
    }
    share_s[share][bin] = s;
    __syncthreads();
    uint32_t all = 0, run = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPlanShares; ++i) {
        run += i < share ? share_s[i][bin] : 0u;
        all += share_s[i][bin];
    }
    if (share == 0) tot[bin] = all;
    __syncthreads();
    all = block_prefix<kPlanThreads>(tot, kSectorBins, wsum);
    run += tot[bin];
    uint32_t *bo = bin_off + size_t(blockIdx.x) * (kSectorBins + 1);
    if (share == 0) bo[bin] = run;
    if (threadIdx.x == 0) bo[kSectorBins] = all;
    for (uint32_t k = k0; k < k1; k += kPlanBatch) {
        if (k1 - k0 > kPlanBatch) batch(k, x);       // else still there
#pragma unroll
        for (uint32_t u = 0; u < kPlanBatch; ++u) {
            if (k + u < k1) pc[size_t(k + u) * kSectorBins] = run;
            run += x[u];
        }
    }
}

// Rounds of kScatterRound hits: each hit's rank in its bin from an LDS
// counter, the bins' places in the round from a prefix, the records placed
// in LDS and copied out in that order.
constexpr uint32_t kScatterPer = 8, kScatterRound = kSplitThreads * kScatterPer;

template <bool Z>
__global__ void __launch_bounds__(kSplitThreads)
k_sector_scatter(const uint8_t *__restrict__ layer, const uint32_t *__restrict__ phi, const int32_t *__restrict__ z,
                 const uint64_t *__restrict__ offs, uint64_t n_hits, uint32_t n_layers, uint32_t sbits, uint32_t K,
                 const uint32_t *__restrict__ part_base, typename IndexRec<Z>::type *__restrict__ out)
{
    using Rec = typename IndexRec<Z>::type;
    static_assert(kSectorBins == kSplitThreads, "one bin per thread");
    __shared__ Rec rec[kScatterRound];
    __shared__ uint8_t rec_bin[kScatterRound];
    __shared__ uint32_t cnt[kSectorBins], to[kSectorBins];
    __shared__ uint32_t wsum[kSplitThreads / 64];
    const uint32_t t = threadIdx.x, e = blockIdx.x / K;
    uint64_t b, end, pb, pe;
    event_range(offs, e, n_hits, b, end);
    part_range(offs, e, blockIdx.x % K, K, n_hits, pb, pe);
    uint32_t next = part_base[size_t(blockIdx.x) * kSectorBins + t];     // bin t's next position
    for (uint64_t r0 = pb; r0 < pe; r0 += kScatterRound) {
        uint32_t bin[kScatterPer], rank[kScatterPer];
        Rec v[kScatterPer];
        cnt[t] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < kScatterPer; ++u) {
            const uint64_t i = r0 + u * kSplitThreads + t;
            bin[u] = kSectorBins;
            v[u] = Rec{};
            if (i < pe) {
                const uint32_t l = layer[i], ph = phi[i];
                v[u] = IndexRec<Z>::make(ph, z, i);
                if (l < n_layers) bin[u] = (l << sbits) + (ph >> (32 - sbits));
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kScatterPer; ++u) rank[u] = bin[u] < kSectorBins ? atomicAdd(&cnt[bin[u]], 1u) : 0u;
        __syncthreads();
        const uint32_t mine = cnt[t];
        const uint32_t total = block_prefix<kSplitThreads>(cnt, kSectorBins, wsum);
        to[t] = next - cnt[t];                       // bin t's place in memory less its place in the round
        next += mine;
#pragma unroll
        for (uint32_t u = 0; u < kScatterPer; ++u) {
            if (bin[u] < kSectorBins) {
                const uint32_t p = cnt[bin[u]] + rank[u];
                rec[p] = v[u];
                rec_bin[p] = uint8_t(bin[u]);
            }
        }
        __syncthreads();
        for (uint32_t p = t; p < total; p += kSplitThreads) out[b + (to[rec_bin[p]] + p)] = rec[p];
        __syncthreads();
    }
}

// One workgroup per (event, layer, sector).  A bin of at most kSortMax hits
// is placed in LDS and copied out; a larger one is written hit by hit.
constexpr uint32_t kSortMax = 2048;

template <bool Z>
__global__ void __launch_bounds__(kSplitThreads)
k_sector_sort(const typename IndexRec<Z>::type *__restrict__ in, const uint64_t *__restrict__ offs, uint64_t n_hits,
              const uint32_t *__restrict__ bin_off, uint32_t n_layers, uint32_t bits, uint32_t sbits,
              typename IndexRec<Z>::type *__restrict__ out, uint32_t *__restrict__ bucket_off)
{
    using Rec = typename IndexRec<Z>::type;
    __shared__ Rec rec[kSortMax];
    __shared__ uint32_t hist[1u << (kMaxBucketBits - kSectorBits)];
    __shared__ uint32_t wsum[kSplitThreads / 64];
    const uint32_t t = threadIdx.x, bins = n_layers << sbits, bin = blockIdx.x % bins, e = blockIdx.x / bins;
    const uint32_t l = bin >> sbits, sector = bin & ((1u << sbits) - 1u);
    const uint32_t nb = 1u << bits, sh = 32 - bits, own = 1u << (bits - sbits);
    uint64_t b, end;
    event_range(offs, e, n_hits, b, end);
    const uint32_t *so = bin_off + size_t(e) * (kSectorBins + 1) + bin;
    const uint32_t s0 = so[0], s1 = so[1];
    for (uint32_t i = t; i < own; i += kSplitThreads) hist[i] = 0;
    __syncthreads();
    for (uint32_t i = s0 + t; i < s1; i += kSplitThreads)
        atomicAdd(&hist[(IndexRec<Z>::phi(in[b + i]) >> sh) & (own - 1u)], 1u);
    __syncthreads();
    block_prefix<kSplitThreads>(hist, own, wsum);
    uint32_t *bo = bucket_off + (size_t(e) * n_layers + l) * (nb + 1) + sector * own;
    for (uint32_t i = t; i < own; i += kSplitThreads) bo[i] = s0 + hist[i];
    if (t == 0 && sector == (1u << sbits) - 1u) bo[own] = s1;
    __syncthreads();
    const bool staged = s1 - s0 <= kSortMax;         // uniform over the workgroup
    for (uint32_t i = s0 + t; i < s1; i += kSplitThreads) {
        const Rec v = in[b + i];
        const uint32_t p = atomicAdd(&hist[(IndexRec<Z>::phi(v) >> sh) & (own - 1u)], 1u);
        if (staged) rec[p] = v;
        else out[b + s0 + p] = v;
    }
    if (!staged) return;
    __syncthreads();
    for (uint32_t i = t; i < s1 - s0; i += kSplitThreads) out[b + s0 + i] = rec[i];
}

// Events ordered longest first (coarse: log2 size with 3 mantissa bits) for
// a longest-processing-time-first work queue.  One workgroup.
__global__ void __launch_bounds__(1024)
k_event_order(const uint64_t *__restrict__ offs, uint64_t n_hits, uint32_t n_events,
              uint32_t *__restrict__ order)
{
    __shared__ uint32_t hist[256];
    const uint32_t t = threadIdx.x;
    auto key = [&](uint32_t e) {
        uint64_t b, end;
        event_range(offs, e, n_hits, b, end);
        const uint64_t sz = end - b;
        if (sz == 0) return 255u;
        const uint32_t lg = 63 - __clzll(sz);
        const uint32_t sub = lg >= 3 ? uint32_t(sz >> (lg - 3)) & 7u : uint32_t(sz << (3 - lg)) & 7u;
        return 255u - min(lg * 8 + sub, 255u);        // descending size
    };
    for (uint32_t i = t; i < 256; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    for (uint32_t e = t; e < n_events; e += blockDim.x) atomicAdd(&hist[key(e)], 1u);
    __syncthreads();
    // exclusive prefix sum of the 256 bins: four per lane of the first wave,
    // then a wave scan of the lanes' totals
    if (t < 64) {
        const uint32_t h0 = hist[4 * t], h1 = hist[4 * t + 1], h2 = hist[4 * t + 2], h3 = hist[4 * t + 3];
        const uint32_t tot = h0 + h1 + h2 + h3;
        uint32_t inc = tot;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t v = __shfl_up(inc, d, 64);
            if (t >= d) inc += v;
        }
        const uint32_t ex = inc - tot;
        hist[4 * t] = ex;
        hist[4 * t + 1] = ex + h0;
        hist[4 * t + 2] = ex + h0 + h1;
        hist[4 * t + 3] = ex + h0 + h1 + h2;
    }
    __syncthreads();
    for (uint32_t e = t; e < n_events; e += blockDim.x) order[atomicAdd(&hist[key(e)], 1u)] = e;
}

hipError_t launch_bucket_layers(hough_ctx *c, const hough_hits *h, hipStream_t s)
{
    if (h->n_events == 0) return hipSuccess;
    KernelTimer t;
    prof_begin(c, "bucket_layers", s, &t);
    if (const uint32_t K = split_parts(c, h->n_events)) {
        const uint32_t parts = h->n_events * K, L = c->spec.n_layers;
        hipLaunchKernelGGL(k_layer_count, dim3(parts), dim3(kSplitThreads), 0, s, h->layer, h->event_offsets,
                           h->n_hits, L, K, c->d_part_cnt);
        hipError_t err = launch_split_plan(h->n_events, L, K, c->d_part_cnt, c->d_part_base, c->d_layer_off, s);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(k_layer_scatter, dim3(parts), dim3(kSplitThreads), 0, s, h->layer, h->phi,
                           h->event_offsets, h->n_hits, L, K, c->d_part_base, c->d_phi_a);
        prof_end(c, s, &t);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_bucket_layers, dim3(h->n_events), dim3(1024), 0, s, h->layer, h->phi, h->event_offsets,
                       h->n_hits, c->spec.n_layers, c->d_phi_a, c->d_layer_off);
    prof_end(c, s, &t);
    return hipGetLastError();
}

hipError_t launch_split_plan(uint32_t n_events, uint32_t n_bins, uint32_t K, const uint32_t *part_cnt,
                             uint32_t *part_base, uint32_t *bin_off, hipStream_t s)
{
    if (n_events == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_plan, dim3(n_events), dim3(64), 0, s, part_cnt, n_bins, K, part_base, bin_off);
    return hipGetLastError();
}

// The whole form is used up to these mean hits per event and hits in all:
// above them its rereading of every event per layer costs more than the
// split form's three more launches.  Whole / split form in us: one event of
// 20,000 hits 12.9 / 19.2, of 60,000 27 / 18.5; 16 events of 20,000 14 / 23;
// 64 events of 25,000 58 / 36.
constexpr uint64_t kIndexWholeHits = 32768, kIndexWholeTotal = 1u << 19;

namespace {

template <bool Z>
void launch_index(hough_ctx *c, const hough_hits *h, hipStream_t s)
{
    using Rec = typename IndexRec<Z>::type;
    const uint32_t E = h->n_events, L = c->spec.n_layers, bits = c->bucket_bits;
    const int vec = (reinterpret_cast<uintptr_t>(h->layer) & 3) == 0 && (reinterpret_cast<uintptr_t>(h->phi) & 15) == 0;
    Rec *out = reinterpret_cast<Rec *>(c->d_hit_b), *mid = reinterpret_cast<Rec *>(c->d_phi_a);
    if (h->n_hits <= kIndexWholeTotal && h->n_hits / E <= kIndexWholeHits) {
        hipLaunchKernelGGL(k_hit_index<Z>, dim3(E * L), dim3(kIndexThreads), 0, s, h->layer, h->phi, h->z_um,
                           h->event_offsets, h->n_hits, L, bits, vec, out, c->d_bucket_off);
        return;
    }
    const uint32_t K = index_parts(c, E, h->n_hits), sbits = std::min(kSectorBits, bits);
    hipLaunchKernelGGL(k_sector_count, dim3(E * K), dim3(kSplitThreads), 0, s, h->layer, h->phi, h->event_offsets,
                       h->n_hits, L, sbits, K, vec, c->d_sec_part);
    hipLaunchKernelGGL(k_sector_plan, dim3(E), dim3(kPlanThreads), 0, s, K, c->d_sec_part, c->d_sec_off);
    hipLaunchKernelGGL(k_sector_scatter<Z>, dim3(E * K), dim3(kSplitThreads), 0, s, h->layer, h->phi, h->z_um,
                       h->event_offsets, h->n_hits, L, sbits, K, c->d_sec_part, mid);
    hipLaunchKernelGGL(k_sector_sort<Z>, dim3(E * (L << sbits)), dim3(kSplitThreads), 0, s, mid, h->event_offsets,
                       h->n_hits, c->d_sec_off, L, bits, sbits, out, c->d_bucket_off);
}

}  // namespace

hipError_t launch_hit_index(hough_ctx *c, const hough_hits *h, bool with_z, hipStream_t s)
{
    if (h->n_events == 0) return hipSuccess;
    KernelTimer t;
    prof_begin(c, "hit_index", s, &t);
    if (with_z) launch_index<true>(c, h, s);
    else launch_index<false>(c, h, s);
    prof_end(c, s, &t);
    return hipGetLastError();
}

hipError_t launch_event_order(hough_ctx *c, const hough_hits *h, hipStream_t s)
{
    KernelTimer t;
    prof_begin(c, "event_order", s, &t);
    hipLaunchKernelGGL(k_event_order, dim3(1), dim3(1024), 0, s, h->event_offsets, h->n_hits,
                       h->n_events, c->d_order);
    prof_end(c, s, &t);
    return hipGetLastError();
}

}  // namespace hough
