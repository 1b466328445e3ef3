"""Assembling events from a pool, against numpy: lengths around a thread's
batch, empty events, repeated sources, no z, and a destination that is too
small."""
import numpy as np
import pytest

from test_gpu_parity import H  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,with_z,short", [
    ([0, 1, 70_001, 262_144, 262_145, 3], True, 0),      # 256 blocks of 256, four hits per thread
    ([300_007], False, 0),
    ([100, 0, 5000, 65_537] * 17, True, 0),              # 68 events: 64 blocks each
    ([5000, 20_000], True, 7_001),
])
def test_gather_events(H, lens, with_z, short):  # noqa: F811
    import torch
    rng = np.random.default_rng(len(lens))
    n_src = 400_000
    layer = rng.integers(0, 256, n_src).astype(np.uint8)
    phi = rng.integers(0, 1 << 32, n_src, dtype=np.uint64).astype(np.uint32)
    z = rng.integers(-(1 << 31), 1 << 31, n_src).astype(np.int32) if with_z else None
    pool = H.DeviceHits(layer, phi, z, np.array([0, n_src], np.uint64))
    lens = np.array(lens, np.int64)
    src = rng.integers(0, n_src - lens + 1)
    dst = np.concatenate([[0], np.cumsum(lens)[:-1]])
    total = int(lens.sum()) - short
    out_l = torch.zeros(total + 1, dtype=torch.uint8, device="cuda")
    out_p = torch.zeros(total + 1, dtype=torch.int32, device="cuda")
    out_z = torch.zeros(total + 1, dtype=torch.int32, device="cuda") if with_z else None
    dev = [torch.from_numpy(a.astype(np.int64)).cuda() for a in (src, lens, dst)]
    H.gather_events(pool, *dev, len(lens), out_l[:total], out_p[:total], out_z[:total] if with_z else None)
    torch.cuda.synchronize()
    idx = np.concatenate([np.arange(s, s + n) for s, n in zip(src, lens)])[:total]
    np.testing.assert_array_equal(out_l.cpu().numpy(), np.append(layer[idx], 0))
    np.testing.assert_array_equal(out_p.cpu().numpy().view(np.uint32), np.append(phi[idx], 0))
    if with_z:
        np.testing.assert_array_equal(out_z.cpu().numpy(), np.append(z[idx], 0))
