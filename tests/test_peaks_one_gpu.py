"""The one-launch peak search (the default for n_phi 256 to 2048) against the
tile form on random accumulators, and against the oracle on small grids:
ragged strips, every number of rows per strip and of strips per workgroup, d0
planes, thresholds at and past the popcounts' range, capacity overflow, calls
of changing size on one context and replays of a captured graph (the
look-back's states carry over from launch to launch)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import H  # noqa: F401

pytestmark = pytest.mark.gpu


def make(H, n_phi, n_qpt, n_d0, threshold, E):
    spec = synth.grid_spec("c1_single_100trk")
    spec.update(n_qpt=n_qpt, n_phi=n_phi, n_d0=n_d0, threshold=threshold, d0_lo_mm=-50.0, d0_hi_mm=50.0)
    return spec, H.HoughContext(spec, max_events=E, max_hits=1)


def random_acc(ctx, E, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = ctx.new_acc(E)
    a.copy_(torch.randint(-32768, 32768, a.shape, generator=g, device="cuda", dtype=torch.int32).to(torch.int16) &
            torch.randint(-32768, 32768, a.shape, generator=g, device="cuda", dtype=torch.int32).to(torch.int16))
    if E > 2:
        a[1].zero_()                                   # an event of one flat plateau
    return a


def both(ctx, acc, E, cap):
    """(peaks, offsets) of the default form and of the tile form."""
    out = []
    for tuning in (dict(), dict(peak_algo=1)):
        ctx.set_tuning(**tuning)
        pk, off = ctx.new_peaks(cap).fill_(-1), ctx.new_offsets(E).fill_(-1)
        ctx.peaks(acc, E, capacity=cap, peaks=pk, offsets=off)
        out.append((pk, off))
    ctx.set_tuning()
    return out


def check(ctx, acc, E, cap=None):
    import torch
    cap = E * ctx.cells if cap is None else cap
    (pk, off), (pk1, off1) = both(ctx, acc, E, cap)
    torch.cuda.synchronize()
    assert torch.equal(off, off1)
    assert torch.equal(pk, pk1)
    return pk, off


@pytest.mark.parametrize("n_phi", [256, 512, 1024, 2048])
@pytest.mark.parametrize("n_qpt,n_d0,E", [(1, 1, 1), (3, 1, 4), (7, 3, 2), (33, 1, 1), (130, 2, 3), (515, 1, 9),
                                          (67, 5, 40), (100, 1, 300)])
def test_against_the_tile_form(H, n_phi, n_qpt, n_d0, E):  # noqa: F811
    E = max(1, E * 256 // n_phi) if E > 4 else E
    spec, ctx = make(H, n_phi, n_qpt, n_d0, 7, E)
    acc = random_acc(ctx, E, n_phi + n_qpt)
    pk, off = check(ctx, acc, E)
    assert 0 < int(off[-1]) < E * ctx.cells
    if ctx.cells <= 70000:                             # and the oracle
        tab = oracle.Tables(spec)
        for e in range(min(E, 2)):
            want = oracle.peaks(tab, H.acc_numpy(acc[e:e + 1])[0])
            np.testing.assert_array_equal(H.peaks_numpy(pk, off, e), want.astype(H.PEAK_DTYPE))


@pytest.mark.parametrize("threshold", [0, 16, 17, 100])
@pytest.mark.parametrize("n_phi,n_d0", [(256, 1), (512, 2), (2048, 1)])
def test_thresholds(H, n_phi, n_d0, threshold):  # noqa: F811
    _, ctx = make(H, n_phi, 9, n_d0, threshold, 2)
    acc = random_acc(ctx, 2, threshold)
    acc[0, 0, 3, :40] = -1                             # popcount 16
    check(ctx, acc, 2)


def test_capacity_overflow(H):  # noqa: F811
    _, ctx = make(H, 512, 40, 1, 6, 5)
    acc = random_acc(ctx, 5, 5)
    total = int(check(ctx, acc, 5)[1][-1])
    for cap in (0, 1, total // 2, total - 1, total):
        check(ctx, acc, 5, cap=cap)


def test_calls_of_changing_size_share_the_states(H):  # noqa: F811
    _, ctx = make(H, 256, 300, 1, 7, 400)
    accs = {E: random_acc(ctx, E, E) for E in (400, 3, 120, 1, 37)}
    for E in (400, 3, 3, 120, 1, 400, 1, 1, 37, 120, 400):
        check(ctx, accs[E], E)


def test_graph_replays_with_eager_calls_between(H):  # noqa: F811
    import torch
    spec = synth.grid_spec("c1_single_100trk")
    batch = synth.gen_batch("c1_single_100trk", 6)
    ctx = H.HoughContext(spec, max_events=6, max_hits=batch.n_hits)
    hits = H.DeviceHits.from_batch(batch)
    cap = 6 * ctx.cells
    want = ctx.peaks(ctx.vote(hits), 6)
    torch.cuda.synchronize()
    acc, pk, off = ctx.new_acc(6), ctx.new_peaks(cap), ctx.new_offsets(6)
    g = ctx.graph_capture(hits, acc, pk, cap, off, stream=torch.cuda.Stream())
    n = int(want[1][-1])
    other = random_acc(ctx, 2, 1)
    for _ in range(4):
        pk.fill_(-1)
        off.fill_(-1)
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(off, want[1]) and torch.equal(pk[:n], want[0][:n])
        check(ctx, other, 2)
