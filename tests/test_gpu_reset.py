"""Reset clears only what a volume has used: after any use, an overflow among
them, the volume then behaves as a new one, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu

S, MU = 0.01, 0.04


@pytest.fixture(scope="module")
def keyframes():
    assert torch.cuda.is_available(), "GPU tests need a device"
    wl = synth.workload(3)
    z, rgb = synth.frames(wl, range(20), device="cuda")
    z, rgb = torch.from_numpy(z).cuda(), torch.from_numpy(rgb).cuda()
    kfs = [scsurf.kf_fuse(z[5 * k:5 * k + 5], rgb[5 * k:5 * k + 5], wl.R[5 * k:5 * k + 5], wl.t[5 * k:5 * k + 5],
                          wl.intr) for k in range(4)]
    return wl, kfs, wl.R[0:20:5], wl.t[0:20:5]


@pytest.mark.parametrize("color", ["rgba8", "f32"])
@pytest.mark.parametrize("used", ["untouched", "plain", "batched", "pool full", "hash full", "twice"])
def test_reset_volume_is_as_new(keyframes, color, used):
    print(f"[gpu] reset after: {used}, {color}", flush=True)
    wl, kfs, R, t = keyframes
    mode = scsurf.COLOR_RGBA8
    if color == "f32":
        mode = scsurf.COLOR_F32
        kfs = [scsurf.Keyframe(k.depth, k.weight, (k.color[..., :3].float() / 255.0).contiguous()) for k in kfs]
    buckets = 1 << 10 if used == "hash full" else 1 << 16
    pool = 512 if used == "pool full" else 1 << 15
    vol, new = (scsurf.Volume(S, MU, buckets, pool, mode) for _ in range(2))
    for _ in range(2 if used == "twice" else 1):
        if used != "untouched":
            if used == "plain":
                vol.integrate(kfs[3], wl.intr, R[3], t[3])
            else:
                vol.integrate_batch(kfs, wl.intr, R, t)
            _, err = vol.query()
            want = {"pool full": scsurf.SC_EPOOLFULL, "hash full": scsurf.SC_EHASHFULL}.get(used, scsurf.SC_OK)
            assert err == want
        vol.reset()
        assert vol.query() == (0, scsurf.SC_OK)
    # part of one keyframe, so that the overflowing volumes hold it too
    part = kfs[0]
    if used in ("pool full", "hash full"):
        keep = torch.zeros_like(part.weight)
        keep[100:120, 100:120] = 1.0
        part = scsurf.Keyframe(part.depth, part.weight * keep, part.color)
    for v in (vol, new):
        v.integrate(part, wl.intr, R[0], t[0])
        v.reintegrate_batch([part], wl.intr, (R[:1], t[:1]), (R[1:2], t[1:2]), 1)
        assert v.check_error() > 0
    a, b = vol.export_sorted(), new.export_sorted()
    for k in ("blocks", "D", "W", "C"):
        np.testing.assert_array_equal(a[k], b[k])
