"""The row form of the vote and the bounds found layer by layer, against the
oracle: around the sizes of their choice, ragged row tiles, rows far apart in
offset, unreachable rows, small and odd layer counts, partial cell groups,
empty events and unaligned arrays."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import H, small_spec  # noqa: F401

pytestmark = pytest.mark.gpu


def event(rng, n, n_layers):
    layer = rng.integers(0, n_layers + 2, n).astype(np.uint8)          # two layers past the last
    phi = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    phi[::5] >>= np.uint32(7)                                           # some buckets hold many
    phi[1::11] = np.uint32(0xFFFFFFFF)
    return layer, phi, np.zeros(n, np.int32)


def layers(n):
    return dict(n_layers=n, layer_r_mm=list(np.linspace(60.0, 800.0, n)), threshold=max(1, n - 2))


@pytest.mark.parametrize("sizes,kw,shift", [
    ([700, 0, 1], dict(n_phi=64, n_qpt=5), 0),                  # a quarter of a cell group, ragged tile
    ([3000], dict(n_phi=256, n_qpt=1), 0),
    ([500, 4099], dict(n_phi=128, n_qpt=2), 2),                 # two rows far apart: J jumps inside a tile
    ([9000], dict(n_phi=512, n_qpt=3, n_d0=7, n_z0=0, n_cot=0, d0_lo_mm=-20.0, d0_hi_mm=20.0), 0),              # tiles across impact-parameter blocks
    ([6000], dict(n_phi=4096, n_qpt=9), 1),
    ([20000], dict(n_phi=8192, n_qpt=3), 0),
    ([5000] * 3, dict(n_phi=512, n_qpt=32, n_d0=16, n_z0=0, n_cot=0, d0_lo_mm=-120.0, d0_hi_mm=120.0), 0),   # unreachable rows
    ([2000] * 51, dict(n_phi=256, n_qpt=160), 0),               # 510 (event, layer) pairs, 4 rows per wave
    ([700] * 52, dict(n_phi=128, n_qpt=33), 0),                 # one more event: the forms before it
    ([4000], dict(n_phi=1024, n_qpt=4096), 0),                  # 2^22 cells, the most it is chosen for
    ([4000], dict(n_phi=1024, n_qpt=4097), 0),
    ([8192], dict(n_phi=256, n_qpt=37), 0),                     # the most hits a workgroup walks for its own table
    ([8193], dict(n_phi=256, n_qpt=37), 1),
    ([16300, 9, 0], dict(n_phi=128, n_qpt=33), 3),              # their mean is what counts
    ([8000, 8000, 8000, 8000, 769], dict(n_phi=64, n_qpt=9), 0),   # one hit too many in all
    ([600], dict(n_phi=256, n_qpt=37, **layers(11)), 0),        # more entries than a workgroup finds itself
    ([270000], dict(n_phi=256, n_qpt=37), 0),                   # a very large event: bounds in 64 parts
    ([20000, 0, 3], dict(n_phi=64, n_qpt=5), 1),                # no vector loads, one part each: by layer
    ([50000, 0, 3], dict(n_phi=64, n_qpt=5), 1),                # four parts, most of them empty
    ([90000, 7], dict(n_phi=256, n_qpt=9), 0),
    ([1500, 300], dict(n_phi=128, n_qpt=19, **layers(1)), 0),
    ([1500, 300], dict(n_phi=128, n_qpt=19, **layers(7)), 3),
    ([1500, 300], dict(n_phi=128, n_qpt=19, **layers(16)), 0),
])
def test_row_form_of_the_vote(H, sizes, kw, shift):  # noqa: F811
    import torch
    spec = small_spec(**kw)
    tab = oracle.Tables(spec)
    rng = np.random.default_rng(sum(sizes) + shift)
    batch = synth.concat_events([event(rng, n, spec["n_layers"]) for n in sizes])
    bufs = []
    for a, dt, view in ((batch.layer, torch.uint8, np.uint8), (batch.phi, torch.int32, np.int32)):
        t = torch.zeros(batch.n_hits + shift, dtype=dt, device="cuda")[shift:]
        t.copy_(torch.from_numpy(np.ascontiguousarray(a).view(view)))
        bufs.append(t)
    hits = H.DeviceHits(*bufs, None, batch.offsets)
    ctx = H.HoughContext(spec, max_events=len(sizes), max_hits=batch.n_hits)
    lead = 2 if shift else 0                                     # accumulator on 4 but not 8 bytes
    flat = torch.full((len(sizes) * tab.cells + lead + 8,), -1, dtype=torch.int16, device="cuda")
    acc = flat[lead:lead + len(sizes) * tab.cells].view(len(sizes), spec["n_d0"], spec["n_qpt"], spec["n_phi"])
    ctx.vote(hits, acc)
    torch.cuda.synchronize()
    got = H.acc_numpy(acc)
    for e in sorted({0, 1, len(sizes) // 2, len(sizes) - 1} & set(range(len(sizes)))):
        ev = batch.event(e)
        np.testing.assert_array_equal(got[e], oracle.vote_mask(tab, ev.layer, ev.phi), err_msg=f"event {e}")
    assert (flat[:lead] == -1).all() and (flat[-8:] == -1).all()
