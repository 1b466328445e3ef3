// Candidate confirmation, second part: a track fit per plateau cluster.
//
// For a beam-line grid (no d0 axis) a hit (r, phi) lies on the track
// (q/pT, phi0) when y cos phi0 - x sin phi0 + rho r^2 / 2 = 0 with
// x = r cos phi, y = r sin phi and rho = 0.299792458e-3 B q/pT (the track
// model of the offset tables with d0 = 0).  Rotated by a reference azimuth
// phi_ref close to the track and divided by cos(phi0 - phi_ref) this is
// linear: y' = t x' - alpha r^2 with t = tan(phi0 - phi_ref) and
// alpha = rho / (2 cos(phi0 - phi_ref)).  Least squares over the members
// gives the 2x2 normal equations, solved by Cramer's rule.
//
// Members are the hits that voted into the cluster's first peak cell; the
// reference azimuth is the centre of that cell's phi0 bin.  Sixteen lanes
// (a DPP row) per cluster, four clusters per wave: a cell holds tens of
// members, in one window of azimuth buckets per layer (hits sorted by
// (layer, bucket) per event), and lane l finds layer l's window.  Pass 1
// sums x'^2, x' r^2, r^4, x' y', y' r^2 over the members, pass 2 the squared
// residuals of the solution.  With z (grids with an rz stage), the residual
// pass also sums the members' (arc length, z) and a third pass takes the
// residuals of the least-squares line z = z0 + cot(theta) s, s the
// transverse arc length (2 / rho) asin(rho r / 2) along the fitted circle:
// the helix.  fp64 throughout, row sums by a fixed butterfly.
//
// Bound by instructions and by the chain of dependent loads (cluster, peak,
// buckets, hits).  A wave per cluster left most lanes idle and evaluated
// sincos and asin twice per member: 64 events of 512 x 512, 250,000
// clusters, 870 us.  Here the first 64 scanned hits stay in registers
// between the passes, sine and cosine are Taylor polynomials after an exact
// reduction of the integer azimuth, and the arc length is evaluated once per
// layer: 145 us; the 1024 x 1024 event with z (50,000 clusters): 206 -> 30 us.
#include "hough_internal.h"

namespace hough {
namespace {

struct FitParams {
    const uint32_t *hit;          // hits by (layer, azimuth bucket) per event: phi, or with the
                                  // longitudinal fit {phi, z (um)}
    const uint32_t *bucket_off;   // [E][L][NB + 1] relative to the event start
    uint32_t bucket_bits;
    const uint64_t *hoff;         // [E + 1] hit offsets
    uint64_t n_hits;
    const uint2 *pk;              // peak records
    uint64_t peak_cap;
    const uint64_t *poff;         // [E + 1]
    const hough_cluster *cl;
    uint64_t cl_cap;
    const uint64_t *coff;         // [E + 1]
    uint32_t E;
    hough_fit *out;
    const uint32_t *O;            // [L][n_qpt]
    const uint8_t *V;
    double r_mm[kMaxLayers];
    uint32_t n_layers, n_qpt, n_phi, log2_phi, shift;
    double qpt_lo, qpt_w;         // bin width (qpt_hi - qpt_lo) / n_qpt
    double inv_curv;              // 1 / (0.299792458e-3 B)
};

// Value of the lane n places on in the row of 16 (rotated).
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x120 | N, 0xF, 0xF, false));
}

template <int N>
__device__ __forceinline__ double row_ror(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t r = uint64_t(row_ror<N>(uint32_t(u))) | (uint64_t(row_ror<N>(uint32_t(u >> 32))) << 32);
    return __builtin_bit_cast(double, r);
}

// Sum over the row of 16 lanes, the same bits in each (every step adds the
// same two partial sums in both of the lanes that hold them).
template <typename T>
__device__ __forceinline__ T row_sum(T v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return v;
}

// Sine and cosine of the azimuth d (a signed turn fraction of 2^-32): the
// quadrant is taken off exactly in integers, then the Taylor series up to
// x^17 and x^16, whose remainders for |x| <= pi/4 are below 1e-19 and 2e-18.
__device__ __forceinline__ void turn_sincos(int32_t d, double &sn, double &cs)
{
    const uint32_t q = (uint32_t(d) + 0x20000000u) >> 30;
    const double x = double(int32_t(uint32_t(d) - (q << 30))) * (6.283185307179586476925286766559 / 4294967296.0);
    const double x2 = x * x;
    double s = 1.0 / 355687428096000.0, c = 1.0 / 20922789888000.0;
    s = fma(s, x2, -1.0 / 1307674368000.0);
    c = fma(c, x2, -1.0 / 87178291200.0);
    s = fma(s, x2, 1.0 / 6227020800.0);
    c = fma(c, x2, 1.0 / 479001600.0);
    s = fma(s, x2, -1.0 / 39916800.0);
    c = fma(c, x2, -1.0 / 3628800.0);
    s = fma(s, x2, 1.0 / 362880.0);
    c = fma(c, x2, 1.0 / 40320.0);
    s = fma(s, x2, -1.0 / 5040.0);
    c = fma(c, x2, -1.0 / 720.0);
    s = fma(s, x2, 1.0 / 120.0);
    c = fma(c, x2, 1.0 / 24.0);
    s = fma(s, x2, -1.0 / 6.0);
    c = fma(c, x2, -0.5);
    s = fma(s * x2, x, x);
    c = fma(c, x2, 1.0);
    const double a = (q & 1u) ? c : s, b = (q & 1u) ? s : c;
    sn = (q & 2u) ? -a : a;
    cs = ((q + 1u) & 2u) ? -b : b;
}

// One layer's window of the member search: hit index = scan index + (scan
// index < split ? add1 : add2) (two ranges when it wraps past 2 pi), and
// the layer's offset at the cell's row.
struct LayerWindow {
    uint32_t add1, add2, split, o;
};

constexpr uint32_t kFitThreads = 256, kFitRows = kFitThreads / 16;
constexpr uint32_t kFitKept = 4;          // scanned hits per lane kept between the passes

// Z: the longitudinal line is fitted too; a separate instance
// keeps the transverse-only kernel's register count (and occupancy) down.
template <bool Z>
__global__ void __launch_bounds__(kFitThreads) k_fit(FitParams P)
{
    __shared__ LayerWindow win_s[kFitRows][kMaxLayers];
    __shared__ uint32_t start_s[kFitRows][kMaxLayers];   // first scan index of each layer's window
    __shared__ double arc_s[kFitRows][kMaxLayers];
    __shared__ double r_s[kMaxLayers];
    const uint32_t lane = threadIdx.x & 15, row = threadIdx.x >> 4;
    if (threadIdx.x < kMaxLayers) r_s[threadIdx.x] = threadIdx.x < P.n_layers ? P.r_mm[threadIdx.x] : 0.0;
    __syncthreads();
    LayerWindow *win = win_s[row];
    uint32_t *start = start_s[row];
    double *arcs = arc_s[row];
    const uint64_t n_cl = min(P.coff[P.E], P.cl_cap);
    const double two_pi = 6.283185307179586476925286766559;
    const double turn_rad = two_pi / 4294967296.0;
    const uint32_t pmask = P.n_phi - 1;
    const uint32_t nb = 1u << P.bucket_bits, bs = 32 - P.bucket_bits;
    auto hit_at = [&](uint64_t h) { return Z ? reinterpret_cast<const uint2 *>(P.hit)[h] : make_uint2(P.hit[h], 0u); };
    uint32_t e = 0;
    // whole waves step together; the rows past the last cluster do nothing
    for (uint64_t c0 = uint64_t(blockIdx.x) * kFitRows + (row & ~3u); c0 < n_cl; c0 += uint64_t(gridDim.x) * kFitRows) {
        const uint64_t c = c0 + (row & 3u);
        const bool act = c < n_cl;
        hough_cluster rec{};
        uint64_t eb = 0;
        uint32_t cell = 0;
        bool ok = false;
        if (act) {
            // event of cluster c: largest e with start(e) <= c; c ascends
            uint32_t hi = P.E;
            while (hi - e > 1) {
                const uint32_t m = (e + hi) >> 1;
                if (min(P.coff[m], n_cl) <= c) e = m;
                else hi = m;
            }
            rec = P.cl[c];
            const uint64_t pe0 = min(P.poff[e], P.peak_cap), pe1 = min(max(P.poff[e + 1], P.poff[e]), P.peak_cap);
            const uint64_t gi = pe0 + rec.first;
            ok = gi < pe1 && rec.n_peaks > 0;
            if (ok) cell = P.pk[gi].x;
            eb = min(P.hoff[e], P.n_hits);
        }
        const uint32_t p = cell & pmask, k = (cell >> P.log2_phi) % P.n_qpt;
        // lane l: the window of layer l
        uint32_t o = 0, hs1 = 0, len1 = 0, hs2 = 0, len2 = 0;
        if (ok && lane < P.n_layers) {
            const size_t ti = size_t(lane) * P.n_qpt + k;
            if (P.V[ti]) {
                const uint64_t W = uint64_t(1) << P.shift, BW = uint64_t(1) << bs;
                o = P.O[ti];
                const uint32_t st = o + (p << P.shift);
                const uint32_t b0 = st >> bs;
                const uint32_t nbk = min(uint32_t(((uint64_t(st) & (BW - 1)) + W - 1) / BW + 1), nb);
                const uint32_t *bl = P.bucket_off + (size_t(e) * P.n_layers + lane) * (nb + 1);
                const uint32_t e1 = b0 + nbk;
                hs1 = bl[b0];
                if (e1 <= nb) {
                    len1 = bl[e1] - hs1;
                } else {
                    len1 = bl[nb] - hs1;
                    hs2 = bl[0];
                    len2 = bl[e1 - nb] - hs2;
                }
            }
        }
        const uint32_t len = len1 + len2;
        uint32_t incl = len;
        incl += uint32_t(__builtin_amdgcn_update_dpp(0, int(incl), 0x111, 0xF, 0xF, false));   // row_shr:1
        incl += uint32_t(__builtin_amdgcn_update_dpp(0, int(incl), 0x112, 0xF, 0xF, false));   // row_shr:2
        incl += uint32_t(__builtin_amdgcn_update_dpp(0, int(incl), 0x114, 0xF, 0xF, false));   // row_shr:4
        incl += uint32_t(__builtin_amdgcn_update_dpp(0, int(incl), 0x118, 0xF, 0xF, false));   // row_shr:8
        const uint32_t excl = incl - len;
        start[lane] = excl;
        win[lane] = LayerWindow{hs1 - excl, hs2 - excl - len1, excl + len1, o};
        const uint32_t T = uint32_t(__shfl(int(incl), 15, 16));
        // the rows' LDS is written and read by the row's own wave only
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // scanned hit gi < T: its layer, azimuth and (Z) z; true for a member
        auto layer_of = [&](uint32_t gi) {
            uint32_t l = 0;
#pragma unroll
            for (uint32_t st = 8; st > 0; st >>= 1) l += start[l + st] <= gi ? st : 0u;
            return l;
        };
        const uint32_t ref = (p << P.shift) + (1u << (P.shift - 1));
        double kx[kFitKept], ky[kFitKept], kz[kFitKept];
        uint32_t kl[kFitKept];                            // layer, kMaxLayers: not a member
        {
            uint32_t ph[kFitKept], oo[kFitKept];
            int32_t zi[kFitKept];
#pragma unroll
            for (uint32_t i = 0; i < kFitKept; ++i) {
                const uint32_t gi = i * 16 + lane;
                kl[i] = kMaxLayers;
                ph[i] = oo[i] = 0;
                zi[i] = 0;
                if (gi < T) {
                    const uint32_t l = layer_of(gi);
                    const LayerWindow w = win[l];
                    const uint64_t h = eb + (gi + (gi < w.split ? w.add1 : w.add2));
                    const uint2 ht = hit_at(h);
                    ph[i] = ht.x;
                    zi[i] = int32_t(ht.y);
                    oo[i] = w.o;
                    kl[i] = l;
                }
            }
#pragma unroll
            for (uint32_t i = 0; i < kFitKept; ++i) {
                if (((ph[i] - oo[i]) >> P.shift) != p) kl[i] = kMaxLayers;
                kx[i] = ky[i] = kz[i] = 0.0;
                if (kl[i] < kMaxLayers) {
                    double sa, ca;
                    turn_sincos(int32_t(ph[i] - ref), sa, ca);
                    const double r = r_s[kl[i]];
                    kx[i] = r * ca;
                    ky[i] = r * sa;
                    if (Z) kz[i] = double(zi[i]) * 1e-3;
                }
            }
        }
        // visit(layer, x', y', z) for every member of this lane: the kept
        // ones, then those past 16 kFitKept scanned hits, evaluated anew
        auto for_members = [&](auto &&visit) {
#pragma unroll
            for (uint32_t i = 0; i < kFitKept; ++i)
                if (kl[i] < kMaxLayers) visit(kl[i], kx[i], ky[i], kz[i]);
            for (uint32_t gi = 16 * kFitKept + lane; gi < T; gi += 16) {
                const uint32_t l = layer_of(gi);
                const LayerWindow w = win[l];
                const uint64_t h = eb + (gi + (gi < w.split ? w.add1 : w.add2));
                const uint2 ht = hit_at(h);
                const uint32_t ph = ht.x;
                if (((ph - w.o) >> P.shift) != p) continue;
                double sa, ca;
                turn_sincos(int32_t(ph - ref), sa, ca);
                const double r = r_s[l];
                visit(l, r * ca, r * sa, Z ? double(int32_t(ht.y)) * 1e-3 : 0.0);
            }
        };
        double sxx = 0, sxw = 0, sww = 0, sxy = 0, syw = 0;
        uint32_t m = 0;
        for_members([&](uint32_t l, double x, double y, double) {
            const double r = r_s[l], wr = r * r;
            sxx += x * x;
            sxw += x * wr;
            sww += wr * wr;
            sxy += x * y;
            syw += y * wr;
            ++m;
        });
        sxx = row_sum(sxx);
        sxw = row_sum(sxw);
        sww = row_sum(sww);
        sxy = row_sum(sxy);
        syw = row_sum(syw);
        m = row_sum(m);
        hough_fit f{};
        if (ok) {
            const double n = double(rec.n_peaks);
            const double kc = double(k) + double(rec.sum_dk) / n;
            const double pc = double(p) + double(rec.sum_dp) / n;
            f.qpt_c = P.qpt_lo + (kc + 0.5) * P.qpt_w;
            const double turns = (pc + 0.5) / double(P.n_phi);
            double fr = turns - trunc(turns);                 // exact, as fmod by 1
            if (fr < 0) fr += 1.0;
            f.phi0_c = two_pi * fr;
            f.n_hits = m;
        }
        const double det = sxx * sww - sxw * sxw;
        const bool fit = ok && m >= 3 && det > 1e-12 * sxx * sww;
        const double t = (sxy * sww - sxw * syw) / det;
        const double alpha = (sxw * sxy - sxx * syw) / det;
        const double cosp = 1.0 / sqrt(1.0 + t * t);
        const double qpt = 2.0 * alpha * cosp * P.inv_curv;
        if (Z) {
            // arc length from the perigee along the fitted circle, layer `lane`
            const double r = r_s[lane], x = 0.5 * (qpt / P.inv_curv) * r;
            arcs[lane] = x == 0.0 ? r : r * (asin(x) / x);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        double ss = 0, s1 = 0, s2 = 0, sz = 0, ssz = 0;
        for_members([&](uint32_t l, double x, double y, double zm) {
            const double r = r_s[l];
            const double res = (y - t * x + alpha * (r * r)) * cosp;
            ss += res * res;
            if (Z) {
                const double s = arcs[l];
                s1 += s;
                s2 += s * s;
                sz += zm;
                ssz += s * zm;
            }
        });
        ss = row_sum(ss);
        if (Z) {
            s1 = row_sum(s1);
            s2 = row_sum(s2);
            sz = row_sum(sz);
            ssz = row_sum(ssz);
            // the line z = z0 + cot s through the members
            const double dm = double(m), detz = dm * s2 - s1 * s1;
            const double z0 = (s2 * sz - s1 * ssz) / detz;
            const double ct = (dm * ssz - s1 * sz) / detz;
            double sr = 0;
            for_members([&](uint32_t l, double, double, double zm) {
                const double res = zm - z0 - ct * arcs[l];
                sr += res * res;
            });
            sr = row_sum(sr);
            if (fit && detz > 1e-12 * dm * s2) {
                f.cot = ct;
                f.z0_mm = z0;
                f.rms_z_mm = sqrt(sr / m);
                f.status_z = 1;
            }
        }
        if (fit) {
            // in (-pi/2, 5 pi/2): one turn added or taken off (exactly)
            double ph0 = double(ref) * turn_rad + atan(t);
            if (ph0 >= two_pi) ph0 -= two_pi;
            if (ph0 < 0) ph0 += two_pi;
            f.phi0 = ph0;
            f.qpt = qpt;
            f.rms_mm = sqrt(ss / m);
            f.status = 1;
        }
        if (act && lane == 0) P.out[c] = f;
    }
}

}  // namespace

hipError_t launch_fit(hough_ctx *c, const hough_hits *h, const hough_peak *peaks, uint64_t peak_capacity,
                      const uint64_t *poff, const hough_cluster *clusters, uint64_t capacity, const uint64_t *coff,
                      hough_fit *out, hipStream_t s)
{
    if (h->n_events == 0 || capacity == 0) return hipSuccess;
    // the longitudinal line needs z, bucketed with the azimuths (rz grids)
    const bool with_z = c->spec.n_z0 > 0 && h->z_um != nullptr;
    const hipError_t err = launch_hit_index(c, h, with_z, s);
    if (err != hipSuccess) return err;
    FitParams P{};
    P.hit = c->d_hit_b;
    P.bucket_off = c->d_bucket_off;
    P.bucket_bits = c->bucket_bits;
    P.hoff = h->event_offsets;
    P.n_hits = h->n_hits;
    P.pk = reinterpret_cast<const uint2 *>(peaks);
    P.peak_cap = peak_capacity;
    P.poff = poff;
    P.cl = clusters;
    P.cl_cap = capacity;
    P.coff = coff;
    P.E = h->n_events;
    P.out = out;
    P.O = c->d_O;
    P.V = c->d_V;
    for (uint32_t l = 0; l < c->spec.n_layers && l < kMaxLayers; ++l) P.r_mm[l] = c->spec.layer_r_mm[l];
    P.n_layers = c->spec.n_layers;
    P.n_qpt = c->spec.n_qpt;
    P.n_phi = c->spec.n_phi;
    P.log2_phi = c->log2_phi;
    P.shift = c->shift;
    P.qpt_lo = c->spec.qpt_lo;
    P.qpt_w = (c->spec.qpt_hi - c->spec.qpt_lo) / c->spec.n_qpt;
    P.inv_curv = 1.0 / (0.299792458e-3 * c->spec.b_tesla);
    const uint64_t blocks = std::min<uint64_t>((capacity + kFitRows - 1) / kFitRows, uint64_t(c->n_cu) * 16);
    KernelTimer t;
    prof_begin(c, "cluster_fit", s, &t);
    if (with_z)
        hipLaunchKernelGGL(k_fit<true>, dim3(uint32_t(std::max<uint64_t>(blocks, 1))), dim3(256), 0, s, P);
    else
        hipLaunchKernelGGL(k_fit<false>, dim3(uint32_t(std::max<uint64_t>(blocks, 1))), dim3(256), 0, s, P);
    prof_end(c, s, &t);
    return hipGetLastError();
}

}  // namespace hough
