"""The candidate selection (an event's first rz_max_candidates peaks by
popcount, then cell) against a stable sort of the peaks: parts with and
without peaks, caps inside a popcount level, past the event's peaks and of
one, empty events, and peak lists cut at their capacity."""
import numpy as np
import pytest

import synth
from test_gpu_parity import H, small_spec  # noqa: F401
from test_rz_dense_gpu import noise_event

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,cap,kw,cut", [
    ([9000], 1000, dict(n_phi=512, n_qpt=200), None),              # 256 parts, some thousand peaks
    ([9000], 1, dict(n_phi=512, n_qpt=200), None),
    ([700, 0, 2500], 5000, dict(n_phi=128, n_qpt=40), None),       # a cap past some events' peaks
    ([600], 3, dict(n_phi=64, n_qpt=2), None),                     # fewer peaks than parts
    ([2500] * 6, 300, dict(n_phi=256, n_qpt=40, threshold=1), None),   # ten popcount levels
    ([2500] * 6, 300, dict(n_phi=256, n_qpt=40, threshold=1), 9000),   # the list ends inside an event
    ([300] * 511, 7, dict(n_phi=64, n_qpt=8), None),               # three parts per event
    ([300] * 512, 7, dict(n_phi=64, n_qpt=8), None),               # one workgroup per event
])
def test_selection_order(H, sizes, cap, kw, cut):  # noqa: F811
    import torch
    spec = small_spec(rz_max_candidates=cap, n_cot=4, **dict(dict(threshold=5), **kw))
    rng = np.random.default_rng(len(sizes) * cap)
    batch = synth.concat_events([noise_event(rng, n) for n in sizes])
    hits = H.DeviceHits.from_batch(batch)
    E = batch.n_events
    ctx = H.HoughContext(spec, max_events=E, max_hits=batch.n_hits)
    pk, poff = ctx.peaks(ctx.vote(hits), E, capacity=E * ctx.cells)
    limit = cut or E * ctx.cells
    rz, roff = ctx.rz_refine(hits, pk, poff, peak_capacity=limit, capacity=E * cap)
    torch.cuda.synchronize()
    offs = H.offsets_numpy(poff)
    assert offs[-1] > 20 and (not cut or offs[-1] > cut)
    for e in range(E):
        pc = H.peaks_numpy(pk, poff, e)["popcount"].astype(int)
        pc = pc[:max(0, limit - int(offs[e]))]
        want = np.argsort(-pc, kind="stable")[:cap]
        np.testing.assert_array_equal(H.rz_numpy(rz, roff, e)["peak"], want, err_msg=f"event {e}")
