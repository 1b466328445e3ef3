"""Performance cases of the track finder: the work its users have it do,
through the binding's public calls, over the range of sizes they use.

Every case is one of six kinds of call sequence:

  find     vote, then the peak search (a trigger without confirmation);
  refine   vote, peak search, rz refinement of every candidate;
  serve    a serving micro-batch: gather the events out of a resident pool,
           vote, peak search, rz refinement of the best 1024 candidates;
  replay   one launch of a captured HIP graph of vote and peak search over a
           batch of events (offline processing);
  confirm  plateau clusters of a peak list at hand and the track fit of every
           cluster;
  count    the counting accumulator and its local maxima.

Sizes come from the workloads of the benchmark and the tests: 10-layer
barrel, 3.8 T, grids from 256 x 256 to 2048 x 2048 and 512 x 512 x 64, 10
to 10,000 tracks per event, 1 to 4096 events per call.  Contexts carry the
autotuner's cached parameters where it has an entry for the workload, the
library's defaults elsewhere, as the benchmark runs them.
"""
import math

import numpy as np
import torch

from paper_1310_7556_amd import hough as H
from paper_1310_7556_amd import tune

BARREL_R_MM = (40.0, 70.0, 110.0, 250.0, 340.0, 430.0, 520.0, 610.0, 700.0, 800.0)
WIDE_R_MM = tuple(110.0 * i for i in range(1, 11))      # the paper's toy detector (counting form)
B_TESLA = 3.8
C_LIGHT = 0.299792458e-3
Z_ACCEPT_MM = 1200.0
D0_MM = 100.0
SERVE_CANDIDATES = 1024
POOL_EVENTS = 64
TWO_PI = 2.0 * math.pi


def _case(name, kind, n_qpt, n_phi, events, tracks, noise, spread="fixed", n_d0=1, rz=False, threshold=8):
    """tracks: per event (the median when spread is "lognormal", the lower
    end of a log-uniform range up to 100 times as many, at most 10,000, when
    it is "loguniform"); noise: noise hits per track hit."""
    return dict(name=name, kind=kind, n_qpt=n_qpt, n_phi=n_phi, n_d0=n_d0, rz=rz, threshold=threshold,
                events=events, tracks=tracks, noise=noise, spread=spread)


def listed():
    return [
        # smallest call: one sparse event on a coarse grid, bound by launches and latency
        _case("event_256", "find", 256, 256, 1, 100, 1.0),
        # the benchmark's headline: one dense event, every candidate refined in rz
        _case("event_1024_rz", "refine", 1024, 1024, 1, 1000, 1.0, rz=True),
        # odd sizes: a row count that is no multiple of any tile, an rz grid, few tracks
        _case("event_odd_rz", "refine", 389, 512, 1, 150, 3.0, rz=True),
        # displaced tracks: a third grid axis (at 1500 tracks the cells are not all full)
        _case("event_512_d0", "find", 512, 512, 1, 1500, 1.0, n_d0=64, threshold=7),
        # serving at low rate: one event per call, and at high rate: a full micro-batch
        _case("serve_1", "serve", 512, 512, 1, 1000, 5.0, rz=True),
        _case("serve_16", "serve", 512, 512, 16, 100, 5.0, spread="loguniform", rz=True),
        # offline processing: a small ragged batch and the benchmark's full one, as graphs
        _case("batch_37", "replay", 512, 512, 37, 300, 5.0, spread="lognormal"),
        _case("batch_4096", "replay", 512, 512, 4096, 300, 5.0, spread="lognormal"),
        # confirmation: the dense single event with z (helix), a saturated
        # batch (circle), and the clusters of a small event
        _case("confirm_1024_rz", "confirm", 1024, 1024, 1, 1000, 1.0, rz=True),
        _case("confirm_batch_64", "confirm", 512, 512, 64, 300, 5.0, spread="lognormal"),
        _case("confirm_256", "confirm", 256, 256, 1, 100, 1.0),
        # the paper's own form: counts on its 2048 x 2048 grid
        _case("count_2048", "count", 2048, 2048, 1, 1000, 0.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["find", "find", "refine", "serve", "replay", "confirm", "count"])
    noise = round(rng.uniform(0.0, 5.0), 2)
    if kind == "find":
        if rng.random() < 0.4:                            # with a d0 axis
            n_phi = rng.choice([256, 512])
            return _nameless(kind, _log_int(rng, 64, 512), n_phi, 1, _log_int(rng, 100, 3 * n_phi),
                             round(noise / 5, 2), n_d0=rng.randint(2, 64), threshold=7)
        return _nameless(kind, _log_int(rng, 64, 1024), rng.choice([256, 512, 1024, 2048]), 1,
                         _log_int(rng, 50, 3000), noise)
    if kind == "refine":
        n_phi = rng.choice([256, 512, 1024])
        return _nameless(kind, _log_int(rng, 64, 1000), n_phi, 1, _log_int(rng, 50, n_phi), round(noise / 5, 2), rz=True)
    if kind == "serve":
        return _nameless(kind, 512, 512, rng.randint(1, 16), _log_int(rng, 100, 1000), 5.0, rz=True)
    if kind == "replay":
        return _nameless(kind, _log_int(rng, 100, 512), rng.choice([256, 512]), _log_int(rng, 2, 1024),
                         _log_int(rng, 50, 400), noise, spread="lognormal")
    if kind == "confirm":
        if rng.random() < 0.5:
            n_phi = rng.choice([256, 512, 1024])
            return _nameless(kind, _log_int(rng, 128, 1000), n_phi, 1, _log_int(rng, 50, n_phi), round(noise / 5, 2),
                             rz=rng.random() < 0.5)
        return _nameless(kind, _log_int(rng, 128, 512), 512, rng.randint(2, 48), _log_int(rng, 50, 300), noise,
                         spread="lognormal")
    return _nameless(kind, _log_int(rng, 256, 2048), rng.choice([512, 1024, 2048]), 1, _log_int(rng, 100, 1000), 0.0)


def _nameless(*args, **kw):
    c = _case("", *args, **kw)
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------

def _spec(case):
    """The grid spec of a case, the same dict as the benchmark's for its workloads."""
    d0_lo, d0_hi = (-D0_MM, D0_MM) if case["n_d0"] > 1 else (0.0, 0.0)
    radii = WIDE_R_MM if case["kind"] == "count" else BARREL_R_MM
    s = dict(n_layers=len(radii), layer_r_mm=list(radii), b_tesla=B_TESLA, n_qpt=case["n_qpt"], qpt_lo=-1.0,
             qpt_hi=1.0, n_phi=case["n_phi"], n_d0=case["n_d0"], d0_lo_mm=d0_lo, d0_hi_mm=d0_hi,
             threshold=case["threshold"], n_z0=0, z0_lo_um=0, z0_hi_um=0, n_cot=0, cot_lo=0.0, cot_hi=0.0,
             rz_max_candidates=SERVE_CANDIDATES if case["kind"] == "serve" else 0)
    if case["rz"]:
        s.update(n_z0=256, z0_lo_um=-200000, z0_hi_um=200000, n_cot=256, cot_lo=-1.2, cot_hi=1.2)
    return s


def _event_tracks(case, rng, n):
    if case["spread"] == "lognormal":
        t = case["tracks"] * np.exp(0.8 * rng.standard_normal(n))
    elif case["spread"] == "loguniform":
        lo = math.log(case["tracks"])
        t = np.exp(rng.uniform(lo, lo + math.log(100.0), n))
    else:
        return np.full(n, case["tracks"], np.int64)
    return np.clip(np.rint(t), 10, 10000).astype(np.int64)


def _hits(case, seed, n_events):
    """Seeded events on the GPU: helix tracks crossing the barrel, smeared,
    plus uniform noise, shuffled within each event.  Returns layer (uint8),
    phi (uint32 turn fraction in int32), z (int32, um) and event offsets."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    nt = _event_tracks(case, np.random.default_rng(seed), n_events)
    ev = torch.from_numpy(np.repeat(np.arange(n_events, dtype=np.int64), nt)).to(dev)
    spec = _spec(case)
    r = torch.tensor(spec["layer_r_mm"], dtype=torch.float64, device=dev)[None, :]
    T, L = len(ev), spec["n_layers"]

    def uniform(lo, hi, n=T):
        return torch.rand(n, generator=g, device=dev, dtype=torch.float64) * (hi - lo) + lo

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev, dtype=torch.float64)

    kappa, phi0, cot = uniform(-1, 1)[:, None], uniform(0, TWO_PI)[:, None], torch.sinh(uniform(-1, 1))[:, None]
    z0 = 50.0 * normal(T, 1)
    d0 = torch.zeros_like(z0)
    if case["n_d0"] > 1:                                  # a fifth of the tracks is displaced
        d0 = torch.where(uniform(0, 1)[:, None] < 0.2, uniform(-D0_MM, D0_MM)[:, None], d0)
    rho = C_LIGHT * B_TESLA * kappa
    denom = 1.0 - rho * d0
    chord = torch.sqrt(torch.clamp((r * r - d0 * d0) / denom, min=0.0))
    half = torch.asin(torch.clamp(rho * chord / 2, -1.0, 1.0))
    x = -d0 * torch.sin(phi0) + chord * torch.cos(phi0 - half)
    y = d0 * torch.cos(phi0) + chord * torch.sin(phi0 - half)
    s = torch.where(rho == 0, chord, 2 * half / torch.where(rho == 0, torch.ones_like(rho), rho))
    sigma = 0.4 if case["kind"] == "count" else 0.02
    phi = torch.atan2(y, x) + normal(T, L) * (sigma / r)
    z = z0 + cot * s + 0.05 * normal(T, L)
    ok = (r > d0.abs()) & (z.abs() < Z_ACCEPT_MM)
    event = ev[:, None].expand(T, L)[ok]
    layer = torch.arange(L, device=dev).expand(T, L)[ok]
    turn = torch.floor(torch.remainder(phi[ok] / TWO_PI, 1.0) * 2.0 ** 32 + 0.5).to(torch.int64)
    zum = torch.floor(z[ok] * 1000.0 + 0.5).to(torch.int32)

    per_event = torch.bincount(event, minlength=n_events)
    n_noise = (per_event * case["noise"]).to(torch.int64)
    noise_event = torch.repeat_interleave(torch.arange(n_events, device=dev), n_noise)
    M = len(noise_event)
    event = torch.cat([event, noise_event])
    layer = torch.cat([layer, torch.randint(0, L, (M,), generator=g, device=dev)])
    turn = torch.cat([turn, torch.randint(0, 1 << 32, (M,), generator=g, device=dev)])
    zum = torch.cat([zum, torch.randint(-1200000, 1200000, (M,), generator=g, device=dev).to(torch.int32)])

    order = torch.argsort(event + torch.rand(len(event), generator=g, device=dev, dtype=torch.float64))
    offsets = np.zeros(n_events + 1, np.uint64)
    np.cumsum(torch.bincount(event, minlength=n_events).cpu().numpy(), out=offsets[1:])
    return layer.to(torch.uint8)[order], _to_i32(turn)[order], zum[order], offsets


def _to_i32(turn):
    """uint32 turn fractions held in int64, as the bits of int32."""
    t = turn & 0xFFFFFFFF
    return torch.where(t >= 1 << 31, t - (1 << 32), t).to(torch.int32)


def _pool_batch(case, seed):
    """A serving micro-batch: which pool events it takes, in arrival order."""
    return np.random.default_rng(seed + 1).permutation(POOL_EVENTS)[:case["events"]]


def _pool(case, seed):
    """The pool's hits and the micro-batch's source offsets, lengths and offsets."""
    layer, phi, z, off = _hits(case, seed, POOL_EVENTS)
    pick = _pool_batch(case, seed)
    o = off.astype(np.int64)
    lens = (o[1:] - o[:-1])[pick]
    dst = np.zeros(len(pick) + 1, np.int64)
    np.cumsum(lens, out=dst[1:])
    return (layer, phi, z, off), o[:-1][pick], lens, dst


def prepare(case, seed):
    spec, E = _spec(case), case["events"]
    st = dict(kind=case["kind"], E=E)
    if case["kind"] == "serve":
        pool, src, lens, dst = _pool(case, seed)
        n = int(dst[-1])
        st["pool"] = H.DeviceHits(*pool)
        st["src"], st["lens"], st["dst"] = (torch.from_numpy(a).cuda() for a in (src, lens, dst))
        empty = [torch.zeros(n, dtype=t, device="cuda") for t in (torch.uint8, torch.int32, torch.int32)]
        hits = H.DeviceHits(*empty, dst.astype(np.uint64))
    else:
        hits = H.DeviceHits(*_hits(case, seed, E))
    cells = spec["n_d0"] * spec["n_qpt"] * spec["n_phi"]
    cap = E * cells
    ctx = H.HoughContext(spec, max_events=E, max_hits=max(hits.n_hits, 1),
                         max_peaks=cap if case["kind"] == "confirm" else 0)
    tuning = tune.cached(spec, E, hits.n_hits)
    if tuning:
        ctx.set_tuning(**tuning)
    st.update(ctx=ctx, hits=hits, cap=cap, peaks=ctx.new_peaks(cap).zero_(), poff=ctx.new_offsets(E).zero_())
    if case["kind"] == "count":
        st["counts"] = ctx.new_counts(E).zero_()
        return st
    st["acc"] = ctx.new_acc(E).zero_()
    if case["kind"] in ("refine", "serve"):
        st["rcap"] = E * SERVE_CANDIDATES if case["kind"] == "serve" else cap
        st["rz"], st["roff"] = ctx.new_rz(st["rcap"]).zero_(), ctx.new_offsets(E).zero_()
    elif case["kind"] == "confirm":
        ctx.vote(hits, st["acc"])
        ctx.peaks(st["acc"], E, capacity=cap, peaks=st["peaks"], offsets=st["poff"])
        st["ccap"] = max(1, cap // 4)
        st["labels"], st["coff"] = ctx.new_labels(cap).zero_(), ctx.new_offsets(E).zero_()
        st["clusters"] = ctx.new_clusters(st["ccap"]).zero_()
        st["fits"] = ctx.new_fits(st["ccap"]).zero_()
    elif case["kind"] == "replay":
        torch.cuda.synchronize()
        st["graph"] = ctx.graph_capture(hits, st["acc"], st["peaks"], cap, st["poff"], stream=torch.cuda.Stream())
    return st


def run(st):
    kind, ctx, E = st["kind"], st["ctx"], st["E"]
    if kind == "replay":
        st["graph"].launch()
        return dict(acc=st["acc"], peaks=st["peaks"], poff=st["poff"])
    if kind == "count":
        ctx.vote_count(st["hits"], st["counts"])
        ctx.peaks_count(st["counts"], E, capacity=st["cap"], peaks=st["peaks"], offsets=st["poff"])
        return dict(counts=st["counts"], peaks=st["peaks"], poff=st["poff"])
    if kind == "confirm":
        ctx.peak_clusters(st["peaks"], st["poff"], E, peak_capacity=st["cap"], capacity=st["ccap"],
                          labels=st["labels"], out=st["clusters"], offsets=st["coff"])
        ctx.cluster_fit(st["hits"], st["peaks"], st["poff"], st["clusters"], st["coff"], peak_capacity=st["cap"],
                        capacity=st["ccap"], out=st["fits"])
        # a fit record is 8 float64 followed by 4 uint32
        return dict(labels=st["labels"], clusters=st["clusters"], coff=st["coff"], fit=st["fits"][:, :8],
                    fit_status=st["fits"].view(torch.int32)[:, 16:])
    if kind == "serve":
        h = st["hits"]
        H.gather_events(st["pool"], st["src"], st["lens"], st["dst"], E, h.layer, h.phi, h.z)
    ctx.vote(st["hits"], st["acc"])
    ctx.peaks(st["acc"], E, capacity=st["cap"], peaks=st["peaks"], offsets=st["poff"])
    out = dict(acc=st["acc"], peaks=st["peaks"], poff=st["poff"])
    if kind in ("refine", "serve"):
        ctx.rz_refine(st["hits"], st["peaks"], st["poff"], peak_capacity=st["cap"], capacity=st["rcap"],
                      out=st["rz"], offsets=st["roff"])
        out.update(rz=st["rz"], roff=st["roff"])
    return out


# ---- what a pass cannot do without ------------------------------------------

def _mean_tracks(case):
    if case["spread"] == "lognormal":
        return case["tracks"] * math.exp(0.32)
    if case["spread"] == "loguniform":                   # mean of a log-uniform law over [t, 100 t]
        return case["tracks"] * 99.0 / math.log(100.0)
    return case["tracks"]


def work(case):
    """Hits read once, accumulators and records written once; the number of
    peaks is estimated from the mean occupancy (half of the cells at or above
    the threshold).  Operations: one decision per (cell, layer), 7 integer
    operations per (member, cot bin) vote of an rz candidate, about 60
    floating-point operations per member of a fitted cluster."""
    spec = _spec(case)
    L, E = spec["n_layers"], case["events"]
    cells = spec["n_d0"] * spec["n_qpt"] * spec["n_phi"]
    hits = _mean_tracks(case) * L * (1.0 + case["noise"])
    q = 1.0 - math.exp(-hits / L / spec["n_phi"])
    full = sum(math.comb(L, m) * q ** m * (1.0 - q) ** (L - m) for m in range(spec["threshold"], L + 1))
    peaks, members = 0.5 * full * cells, hits / spec["n_phi"]
    if case["kind"] == "confirm":
        clusters = peaks / 8
        return dict(bytes=E * (peaks * 12 + clusters * (24 + 80) + hits * 9),
                    flops=E * (peaks * 4 + clusters * members * 60))
    b, f = hits * 5 + peaks * 8, cells * L
    b += cells * (4 if case["kind"] == "count" else 2)
    if case["kind"] in ("refine", "serve"):
        cand = min(peaks, SERVE_CANDIDATES) if case["kind"] == "serve" else peaks
        b += hits * (4 if case["kind"] == "refine" else 13) + cand * 16
        f += cand * members * spec["n_cot"] * 7
    return dict(bytes=E * b, flops=E * f)


# ---- plain 64-bit evaluation ------------------------------------------------

EXACT_VOTES = 1e10        # hits x rows above which the plain vote takes too long


def _tables(spec):
    """O [L, D, K] (int64 turn fractions mod 2^32) and reachability V, in float64."""
    def centres(lo, hi, n):
        return lo + (np.arange(n) + 0.5) * (hi - lo) / n

    kap = centres(spec["qpt_lo"], spec["qpt_hi"], spec["n_qpt"])[None, None, :]
    d0 = centres(spec["d0_lo_mm"], spec["d0_hi_mm"], spec["n_d0"]) if spec["n_d0"] > 1 else np.zeros(1)
    d0 = d0[None, :, None]
    r = np.array(spec["layer_r_mm"])[:, None, None]
    rho = C_LIGHT * spec["b_tesla"] * kap
    den = r * (1.0 - rho * d0)
    with np.errstate(all="ignore"):
        arg = (d0 - 0.5 * rho * (r * r + d0 * d0)) / den
        ok = (1.0 - rho * d0 > 0) & (np.abs(arg) <= 1.0)
        a = np.arcsin(np.where(ok, arg, 0.0)) / TWO_PI * 4294967296.0
    rounded = np.where(a >= 0, np.floor(a + 0.5), np.ceil(a - 0.5)).astype(np.int64)
    return torch.from_numpy(rounded & 0xFFFFFFFF).cuda(), torch.from_numpy(ok).cuda()


def _plain_votes(spec, layer, phi, off, counting):
    """Layer masks or counts, [E, D, K, P], by one scatter per (event, layer)."""
    O, V = _tables(spec)
    L, D, K, P = spec["n_layers"], spec["n_d0"], spec["n_qpt"], spec["n_phi"]
    shift = 32 - int(math.log2(P))
    out = torch.zeros((len(off) - 1, D * K, P), dtype=torch.int32, device="cuda")
    ph = phi.to(torch.int64) & 0xFFFFFFFF
    base = (torch.arange(D * K, device="cuda") * P)[:, None]
    for e in range(len(off) - 1):
        a, b = int(off[e]), int(off[e + 1])
        for l in range(L):
            h = ph[a:b][layer[a:b] == l]
            o, v = O[l].reshape(-1, 1), V[l].reshape(-1)
            hit = torch.zeros(D * K * P, dtype=torch.int32, device="cuda")
            step = max(1, (1 << 28) // (D * K))
            for i in range(0, len(h), step):
                cell = ((((h[None, i:i + step] - o) & 0xFFFFFFFF) >> shift) + base)[v].reshape(-1)
                if counting:
                    hit += torch.bincount(cell, minlength=D * K * P).to(torch.int32)
                else:
                    hit[cell] = 1
            out[e] += (hit if counting else hit << l).reshape(D * K, P)
    return out.reshape(-1, D, K, P)


def _popcount(m):
    return sum((m >> i) & 1 for i in range(16))


def _neighbours(x, fill):
    """x shifted onto each of the 27 window offsets (its own included)."""
    def shift(t, dim, by):
        if by == 0:
            return t
        s = torch.roll(t, by, dim)
        s.select(dim, 0 if by > 0 else -1).fill_(fill)
        return s

    for dd in (-1, 0, 1) if x.shape[1] > 1 else (0,):
        a = shift(x, 1, dd)
        for dk in (-1, 0, 1):
            b = shift(a, 2, dk)
            for dp in (-1, 0, 1):
                yield torch.roll(b, dp, 3)


def _plain_peaks(value, threshold):
    """Peak flags of [E, D, K, P] values."""
    ok = value >= threshold
    for n in _neighbours(value, -1):
        ok &= value >= n
    return ok


def _plain_clusters(flag):
    """Smallest flat cell index of each peak's connected component (others
    hold the number of cells), by min-label hooking and pointer jumping."""
    n = flag.numel()
    lab = torch.where(flag, torch.arange(n, device="cuda").reshape(flag.shape), torch.full_like(flag, n, dtype=torch.int64))
    while True:
        low = lab
        for x in _neighbours(lab, n):
            low = torch.minimum(low, x)
        low = torch.where(flag, low, n).reshape(-1)
        new = torch.cat([lab.reshape(-1), torch.tensor([n], device="cuda")])
        new.scatter_reduce_(0, lab.reshape(-1), low, "amin")
        new[:n] = torch.minimum(new[:n], low)
        new[n] = n
        for _ in range(6):
            new = new[new]
        new = new[:n].reshape(flag.shape)
        if torch.equal(new, lab):
            return lab
        lab = new


def _fits(case, spec, hits, rec_cell, rec_event, n_peaks, sum_dk, sum_dp):
    """The least-squares helix of every cluster from its first peak's cell."""
    layer, phi, z, off = hits
    O, _ = _tables(spec)
    K, P = spec["n_qpt"], spec["n_phi"]
    W = 1 << (32 - int(math.log2(P)))
    k, p = (rec_cell // P) % K, rec_cell % P
    n = n_peaks.to(torch.float64)
    qpt_c = spec["qpt_lo"] + (k + sum_dk / n + 0.5) * ((spec["qpt_hi"] - spec["qpt_lo"]) / K)
    phi0_c = TWO_PI * torch.remainder((p + sum_dp / n + 0.5) / P, 1.0)
    ref = p * W + W // 2
    # members: per (event, layer) the sorted azimuths between the cell's edges
    ph = phi.to(torch.int64) & 0xFFFFFFFF
    event = torch.repeat_interleave(torch.arange(len(off) - 1, device="cuda"),
                                    torch.from_numpy(np.diff(off.astype(np.int64))).cuda())
    group = event * spec["n_layers"] + layer
    order = torch.argsort(group * (1 << 32) + ph)
    key, zs = (group * (1 << 32) + ph)[order], z[order].to(torch.float64) * 1e-3
    r_of = torch.tensor(spec["layer_r_mm"], dtype=torch.float64, device="cuda")
    owner, member = [], []
    for l in range(spec["n_layers"]):
        g = (rec_event * spec["n_layers"] + l) * (1 << 32)
        a = (O[l, 0][k] + p * W) & 0xFFFFFFFF
        for lo, hi in ((a, torch.clamp(a + W, max=1 << 32)), (torch.zeros_like(a), torch.clamp(a + W - (1 << 32), min=0))):
            i0, i1 = torch.searchsorted(key, g + lo), torch.searchsorted(key, g + hi)
            cnt = i1 - i0
            who = torch.repeat_interleave(torch.arange(len(cnt), device="cuda"), cnt)
            start = torch.cumsum(cnt, 0) - cnt
            owner.append(who)
            member.append(i0[who] + torch.arange(len(who), device="cuda") - start[who])
    owner, member = torch.cat(owner), torch.cat(member)
    C = len(rec_cell)

    def total(v):
        return torch.zeros(C, dtype=torch.float64, device="cuda").index_add_(0, owner, v)

    h = key[member] & 0xFFFFFFFF
    r = r_of[(key[member] >> 32) % spec["n_layers"]]
    d = (h - ref[owner]) & 0xFFFFFFFF
    ang = torch.where(d >= 1 << 31, d - (1 << 32), d).to(torch.float64) * (TWO_PI / 4294967296.0)
    x, y, w = r * torch.cos(ang), r * torch.sin(ang), r * r
    m = total(torch.ones_like(r))
    sxx, sxw, sww, sxy, syw = total(x * x), total(x * w), total(w * w), total(x * y), total(y * w)
    det = sxx * sww - sxw * sxw
    ok = (m >= 3) & (det > 1e-12 * sxx * sww)
    det = torch.where(ok, det, torch.ones_like(det))
    t, alpha = (sxy * sww - sxw * syw) / det, (sxw * sxy - sxx * syw) / det
    cosp = 1.0 / torch.sqrt(1.0 + t * t)
    curv = C_LIGHT * spec["b_tesla"]
    qpt = 2.0 * alpha * cosp / curv
    phi0 = torch.remainder(ref.to(torch.float64) * (TWO_PI / 4294967296.0) + torch.atan(t), TWO_PI)
    res = (y - t[owner] * x + alpha[owner] * w) * cosp[owner]
    rms = torch.sqrt(total(res * res) / torch.clamp(m, min=1))
    f = torch.zeros((C, 8), dtype=torch.float64, device="cuda")
    status = torch.zeros((C, 4), dtype=torch.int64, device="cuda")
    for j, v in enumerate((qpt, phi0)):
        f[:, j] = torch.where(ok, v, 0.0)
    f[:, 2], f[:, 3], f[:, 4] = qpt_c, phi0_c, torch.where(ok, rms, 0.0)
    status[:, 0], status[:, 1] = m.to(torch.int64), ok.to(torch.int64)
    if case["rz"]:
        half = 0.5 * (qpt * curv)[owner] * r
        s = torch.where(half == 0, r, r * torch.asin(torch.clamp(half, -1, 1)) / torch.where(half == 0, torch.ones_like(half), half))
        zz = zs[member]
        s1, s2, sz, ssz = total(s), total(s * s), total(zz), total(s * zz)
        det = m * s2 - s1 * s1
        okz = ok & (det > 1e-12 * m * s2)
        det = torch.where(okz, det, torch.ones_like(det))
        zero, cot = (s2 * sz - s1 * ssz) / det, (m * ssz - s1 * sz) / det
        rz = zz - zero[owner] - cot[owner] * s
        for j, v in enumerate((cot, zero, torch.sqrt(total(rz * rz) / torch.clamp(m, min=1)))):
            f[:, 5 + j] = torch.where(okz, v, 0.0)
        status[:, 2] = okz.to(torch.int64)
    return f, status


def _records(shape, *columns):
    out = torch.zeros(shape, dtype=torch.int64, device="cuda")
    for j, c in enumerate(columns):
        out[:len(c), j] = c
    return out


def exact(case, seed):
    spec, E = _spec(case), case["events"]
    cells = spec["n_d0"] * spec["n_qpt"] * spec["n_phi"]
    cap = E * cells
    if case["kind"] == "serve":
        (layer, phi, z, off), _, _, dst = _pool(case, seed)
        o = off.astype(np.int64)
        take = torch.cat([torch.arange(o[i], o[i + 1], device="cuda") for i in _pool_batch(case, seed)])
        hits = (layer[take], phi[take], z[take], dst.astype(np.uint64))
    else:
        hits = _hits(case, seed, E)
    if len(hits[0]) * (cells // spec["n_phi"]) > EXACT_VOTES:
        return None
    counting = case["kind"] == "count"
    acc = _plain_votes(spec, hits[0], hits[1], hits[3], counting)
    value = acc if counting else _popcount(acc)
    flag = _plain_peaks(value, spec["threshold"])
    where = torch.nonzero(flag.reshape(-1)).reshape(-1)
    edges = torch.arange(E + 1, device="cuda") * cells
    poff = torch.searchsorted(where, edges)
    if counting:
        return dict(counts=acc, peaks=_records((cap, 2), where % cells, value.reshape(-1)[where]), poff=poff)
    mask, pop = acc.reshape(-1)[where].to(torch.int64), value.reshape(-1)[where].to(torch.int64)
    if case["kind"] != "confirm":
        out = dict(acc=torch.where(acc >= 1 << 15, acc - (1 << 16), acc),
                   peaks=_records((cap, 2), where % cells, mask | pop << 16), poff=poff)
        if case["kind"] in ("refine", "serve"):
            out.update(rz=None, roff=torch.minimum(poff[1:] - poff[:-1], torch.tensor(
                SERVE_CANDIDATES if case["kind"] == "serve" else cap, device="cuda")).cumsum(0))
            out["roff"] = torch.cat([torch.zeros_like(out["roff"][:1]), out["roff"]])
        return out
    lab = _plain_clusters(flag).reshape(-1)[where]        # first cell of each peak's cluster
    first = torch.unique(lab)
    cid = torch.searchsorted(first, lab)
    C = len(first)
    coff = torch.searchsorted(first, edges)
    fev = first // cells
    P, K = spec["n_phi"], spec["n_qpt"]

    def total(v):
        return torch.zeros(C, dtype=torch.int64, device="cuda").index_add_(0, cid, v)

    dp = (where - lab) % P
    dp = torch.where(dp >= P // 2, dp - P, dp)
    n, dk = total(torch.ones_like(lab)), total((where // P) % K - (lab // P) % K)
    dd, sdp = total((where % cells) // (P * K) - (lab % cells) // (P * K)), total(dp)
    mor = sum((total((mask >> i) & 1) > 0).to(torch.int64) << i for i in range(16))
    at = torch.searchsorted(where, first)
    low32 = 0xFFFFFFFF
    clusters = _records((max(1, cap // 4), 3), (at - poff[fev]) | pop[at] << 32 | mor << 48, n | (dk & low32) << 32,
                        (sdp & low32) | (dd & low32) << 32)
    f, status = _fits(case, spec, hits, first % cells, fev, n, dk, sdp)
    labels = torch.zeros(cap, dtype=torch.int64, device="cuda")
    labels[:len(lab)] = cid - coff[where // cells]
    fit = torch.zeros((max(1, cap // 4), 8), dtype=torch.float64, device="cuda")
    fit[:C] = f
    return dict(labels=labels, clusters=clusters, coff=coff, fit=fit, fit_status=_records((max(1, cap // 4), 4), *status.T))
