"""The rz form for cells of many members (chosen from 48 hits per cell on)
against the oracle, bit for bit: pass remainders in the cot and z0 bins,
layer counts, lists past their size, byte counts that pass 255, mid-pass
sweeps, an empty event and the wide multiply-high."""
import math

import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import H, check_event, run_gpu, small_spec  # noqa: F401

pytestmark = pytest.mark.gpu


def noise_event(rng, n, n_layers=10):
    return (rng.integers(0, n_layers, n).astype(np.uint8), rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32),
            rng.integers(-1_200_000, 1_200_000, n).astype(np.int32))


def check(H, spec, events):
    batch = synth.concat_events(events)
    assert batch.n_hits / batch.n_events / spec["n_phi"] >= 48
    res = run_gpu(H, spec, batch)
    tab = oracle.Tables(spec)
    for e in range(batch.n_events):
        check_event(H, tab, res, batch, e, rz=True)
    return res, batch


@pytest.mark.parametrize("sizes,kw", [
    ([2400, 0, 1600, 900], dict(n_phi=16, n_qpt=6)),                       # 56 to 150 members
    ([2400, 1600], dict(n_phi=16, n_qpt=6, n_cot=70, n_z0=253)),           # ragged passes and counter rows
    ([2400, 1600], dict(n_phi=16, n_qpt=6, n_cot=300, n_z0=10)),           # a second round of passes
    ([2400, 1600], dict(n_phi=16, n_qpt=6, n_cot=1, n_z0=1)),
    ([2400, 1600], dict(n_phi=16, n_qpt=6, cot_lo=1.2, cot_hi=-1.2)),      # Z decreasing
    ([4000, 3000], dict(n_phi=4, n_qpt=4, n_cot=64)),                      # passes past 255 votes
    ([4000, 3000], dict(n_phi=4, n_qpt=4, n_cot=65, n_z0=39)),             # as many out of range, in a row's last byte
    ([9000, 100], dict(n_phi=2, n_qpt=3, n_cot=33)),                       # more scanned hits than the list holds
    ([2400], dict(n_phi=16, n_qpt=6, z0_lo_um=-20_000_000, z0_hi_um=20_000_000)),   # 32-bit multiply-high
])
def test_dense_rz(H, sizes, kw):  # noqa: F811
    rng = np.random.default_rng(sum(sizes))
    check(H, small_spec(**kw), [noise_event(rng, n) for n in sizes])


@pytest.mark.parametrize("n_layers", [1, 3, 15])
def test_dense_rz_layer_counts(H, n_layers):  # noqa: F811
    spec = small_spec(n_phi=16, n_qpt=6)
    spec.update(n_layers=n_layers, layer_r_mm=list(np.linspace(60.0, 800.0, n_layers)), threshold=1)
    rng = np.random.default_rng(n_layers)
    check(H, spec, [noise_event(rng, n, n_layers) for n in (1700, 800)])


@pytest.mark.parametrize("copies", [24, 26])
def test_dense_rz_counts_around_255(H, copies):  # noqa: F811
    # identical bin-centre tracks: 10 members per copy in one (cot, z0) bin
    spec = small_spec(n_phi=16, n_qpt=41)
    K, N = spec["n_qpt"], spec["n_phi"]
    kap = spec["qpt_lo"] + (np.arange(K) + 0.5) * (spec["qpt_hi"] - spec["qpt_lo"]) / K
    layer, phi, z = synth.track_hits(kap[20], (7 + 0.5) / N * 2 * math.pi,
                                     cot=-1.2 + 160.5 * 2.4 / 256, z0=-200.0 + 140.5 * 400.0 / 256)
    nl, nphi, nz = noise_event(np.random.default_rng(3), 800)
    res, _ = check(H, spec, [(np.concatenate([layer] * copies + [nl]), np.concatenate([phi] * copies + [nphi]),
                              np.concatenate([z] * copies + [nz]))])
    assert H.rz_numpy(res["rz"], res["roff"], 0)["count"].max() >= 10 * copies


@pytest.mark.parametrize("sizes,kw", [
    ([900, 1000, 850], dict(n_phi=16, n_qpt=6)),                   # 48 to 64 members per cell
    ([900], dict(n_phi=16, n_qpt=5, n_cot=65, n_z0=39)),
    ([900], dict(n_phi=16, n_qpt=5, n_cot=64)),
])
def test_short_lists_around_the_choice(H, sizes, kw):  # noqa: F811
    """From 48 to 64 members per cell, candidate lists bounded by 16 per
    compute unit take the dense form, longer ones and those of one pass the
    other: the same records."""
    import torch
    spec = small_spec(threshold=4, **kw)
    rng = np.random.default_rng(sum(sizes))
    batch = synth.concat_events([noise_event(rng, n) for n in sizes])
    assert 48 <= batch.n_hits / batch.n_events / spec["n_phi"] < 64
    hits = H.DeviceHits.from_batch(batch)
    E = batch.n_events
    ctx = H.HoughContext(spec, max_events=E, max_hits=batch.n_hits)
    acc = ctx.vote(hits)
    pk, poff = ctx.peaks(acc, E)
    bound = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    res = [ctx.rz_refine(hits, pk, poff, capacity=cap) for cap in (bound, bound + 1)]
    torch.cuda.synchronize()
    tab = oracle.Tables(spec)
    for rz, roff in res:
        for e in range(E):
            check_event(H, tab, dict(acc=acc, pk=pk, poff=poff, rz=rz, roff=roff), batch, e, rz=True)


@pytest.mark.parametrize("kw", [dict(n_qpt=300), dict(n_qpt=300, rz_max_candidates=9000), dict(n_qpt=3)])
def test_shares_and_tickets(H, kw):  # noqa: F811
    """Lists divided evenly over the waves and lists past 32 per wave (one wave
    per compute unit), which go by tickets, give the same records; so do a few
    candidates over many waves."""
    import torch
    spec = small_spec(threshold=4, n_phi=256, n_cot=20, n_z0=32, **kw)
    rng = np.random.default_rng(4)
    batch = synth.concat_events([noise_event(rng, n) for n in (3000, 0, 2800)])
    hits = H.DeviceHits.from_batch(batch)
    ctx = H.HoughContext(spec, max_events=3, max_hits=batch.n_hits)
    pk, poff = ctx.peaks(ctx.vote(hits), 3)
    res = []
    for w in (1, 2, 16):
        ctx.set_tuning(rz_waves_per_cu=w, rz_counter_bits=4)
        res.append(ctx.rz_refine(hits, pk, poff))
    torch.cuda.synchronize()
    n = [int(H.offsets_numpy(roff)[-1]) for _, roff in res]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert n[0] == n[1] == n[2] and (n[0] > 32 * cus if spec["n_qpt"] == 300 else n[0] < 16 * cus)
    for e in range(3):
        a, b, c = (H.rz_numpy(rz, roff, e) for rz, roff in res)
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(a, c)
    if spec["n_qpt"] == 3:
        tab = oracle.Tables(spec)
        ev = batch.event(0)
        opk = oracle.peaks(tab, oracle.vote_mask(tab, ev.layer, ev.phi))
        np.testing.assert_array_equal(a_first := H.rz_numpy(*res[0], 0), oracle.rz(tab, ev.layer, ev.phi, ev.z, opk).astype(H.RZ_DTYPE))
        assert len(a_first)
