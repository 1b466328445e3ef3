"""The hit index (hits by layer and azimuth bucket) under the rz stage and
the cluster fit, against the oracle: both forms around their dividing line,
bins past the LDS sort, few buckets, unaligned hit arrays, layers past the
detector's, empty events, and the index without z."""
import numpy as np
import pytest

import oracle
import synth
from test_clusters_gpu import check_fit
from test_gpu_parity import H, check_event, small_spec  # noqa: F401

pytestmark = pytest.mark.gpu


def event(rng, n, clustered=False, n_layers=10):
    layer = rng.integers(0, n_layers, n).astype(np.uint8)
    phi = rng.integers(0, 1 << 32, n, dtype=np.uint64)
    if clustered:                                     # half of the hits in a 64th of the circle, across 2 pi
        phi[::2] = (phi[::2] >> np.uint64(6)) - np.uint64(1 << 25)
    return layer, (phi & np.uint64(0xFFFFFFFF)).astype(np.uint32), rng.integers(-1_200_000, 1_200_000, n).astype(np.int32)


def run(H, spec, batch, shift=0):
    import torch
    n = batch.n_hits
    bufs = []
    for a, dt, view in ((batch.layer, torch.uint8, np.uint8), (batch.phi, torch.int32, np.int32), (batch.z, torch.int32, np.int32)):
        t = torch.zeros(n + shift, dtype=dt, device="cuda")[shift:]
        t.copy_(torch.from_numpy(np.ascontiguousarray(a).view(view)))
        bufs.append(t)
    hits = H.DeviceHits(*bufs, batch.offsets)
    ctx = H.HoughContext(spec, max_events=batch.n_events, max_hits=n)
    acc = ctx.vote(hits)
    pk, poff = ctx.peaks(acc, batch.n_events)
    rz, roff = ctx.rz_refine(hits, pk, poff)
    torch.cuda.synchronize()
    return dict(acc=acc, pk=pk, poff=poff, rz=rz, roff=roff)


@pytest.mark.parametrize("sizes,kw,opts", [
    ([32768], dict(n_phi=512, n_qpt=2), {}),                       # the last mean size of the whole form
    ([32800], dict(n_phi=512, n_qpt=2), {}),                       # the first of the split form
    ([40000, 0, 70000], dict(n_phi=512, n_qpt=1), dict(clustered=True)),   # bins past the LDS sort
    ([5000, 0, 70000, 120000], dict(n_phi=1024, n_qpt=1), {}),     # skewed events
    ([60000], dict(n_phi=2, n_qpt=1, n_cot=5), {}),                # fewer buckets than sectors
    ([33001, 41003], dict(n_phi=512, n_qpt=1), dict(shift=1)),     # unaligned arrays, split form
    ([3001, 403], dict(n_phi=128, n_qpt=3), dict(shift=1)),        # unaligned arrays, whole form
    ([50000], dict(n_phi=512, n_qpt=1), dict(layers=200)),         # hits of layers the detector lacks
    ([4000, 300], dict(n_phi=64, n_qpt=4), dict(layers=200)),
    ([480] * 1100, dict(n_phi=64, n_qpt=1, n_cot=3), {}),          # split form, one part per event
    ([300_000, 11], dict(n_phi=512, n_qpt=1, n_cot=3), {}),        # 146 parts per event
])
def test_rz_over_the_hit_index(H, sizes, kw, opts):  # noqa: F811
    spec = small_spec(**dict(dict(n_cot=20), **kw))
    rng = np.random.default_rng(sum(sizes))
    batch = synth.concat_events([event(rng, n, opts.get("clustered", False), opts.get("layers", 10)) for n in sizes])
    res = run(H, spec, batch, opts.get("shift", 0))
    tab = oracle.Tables(spec)
    for e in range(batch.n_events):
        check_event(H, tab, res, batch, e, rz=True)


@pytest.mark.parametrize("n", [3000, 40000])
def test_fit_without_z_over_the_hit_index(H, n):  # noqa: F811
    import torch
    spec = small_spec(n_phi=256, n_qpt=3)
    rng = np.random.default_rng(n)
    batch = synth.concat_events([event(rng, n), event(rng, n)])
    tab = oracle.Tables(spec)
    cap = 2 * tab.cells
    ctx = H.HoughContext(spec, max_events=2, max_hits=2 * n, max_peaks=cap)
    hits = H.DeviceHits(batch.layer, batch.phi, None, batch.offsets)
    pk, poff = ctx.peaks(ctx.vote(hits), 2, capacity=cap)
    _, cl, coff = ctx.peak_clusters(pk, poff, 2)
    fits = ctx.cluster_fit(hits, pk, poff, cl, coff)
    torch.cuda.synchronize()
    for e in range(2):
        ev = batch.event(e)
        opk = oracle.peaks(tab, oracle.vote_mask(tab, ev.layer, ev.phi))
        _, ocl = oracle.clusters(tab, opk)
        check_fit(H, H.fits_numpy(fits, coff, e), oracle.fit(tab, ev.layer, ev.phi, opk, ocl, None), what=f"event {e}")
