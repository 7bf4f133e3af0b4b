"""The host store without pinned memory for all of it: records in pageable
memory pass through the staging buffer (256 at once).  A field sent out and
brought back, and updates in a pool smaller than the field, equal the resident
volume bit for bit."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu


def _same(a, b):
    for k in a:
        np.testing.assert_array_equal(b[k], a[k], err_msg=k)


@pytest.mark.parametrize("n,mode,pinned", [(1, scsurf.COLOR_RGBA8, 0), (256, scsurf.COLOR_F32, 0),
                                           (257, scsurf.COLOR_RGBA8, 0), (2600, scsurf.COLOR_RGBA8, 0),
                                           (2600, scsurf.COLOR_RGBA8, 9 << 20)])
def test_field_survives_the_pageable_store(n, mode, pinned):
    print(f"[gpu] pageable host store, {n} blocks, colour mode {mode}, pinned {pinned}", flush=True)
    rng = np.random.default_rng(n)
    f = {"blocks": np.stack(np.unravel_index(rng.permutation(32 ** 3)[:n], (32, 32, 32)), 1).astype(np.int32) - 16,
         "D": rng.normal(0, 0.02, (n, 512)).astype(np.float32),
         "W": rng.integers(1, 900, (n, 512)).astype(np.float32),
         "C": rng.integers(0, 256, (n, 512, 4), dtype=np.uint8) if mode == scsurf.COLOR_RGBA8
         else rng.uniform(0, 1, (n, 3, 512)).astype(np.float32)}
    vol = scsurf.Volume(0.01, 0.04, 1 << 13, n, color_mode=mode)
    with pytest.raises(scsurf.ScError):
        vol.stream_pinned_limit(0)
    for turn in range(2):
        vol.import_field({k: torch.from_numpy(v).cuda() for k, v in f.items()})
        ref = vol.export_sorted()
        vol.stream_enable(True)
        vol.stream_pinned_limit(pinned)
        for radius in (1.4, 0.9, 0.4, 0.0):
            vol.stream_out((0.3, -0.2, 9.0 if radius == 0.0 else 0.1), radius)
            _same(ref, vol.export_sorted(with_host=True))
            if radius == 0.9:
                vol.stream_in_all()
                _same(ref, vol.export_sorted())
        assert vol.stream_stats()[:2] == (0, n)
        if turn == 0:
            vol.reset()
            vol.stream_enable(False)
    vol.stream_in_all()
    assert vol.check_error() == n
    _same(ref, vol.export_sorted())
    vol.close()


@pytest.mark.parametrize("batched", [False, True])
def test_updates_in_a_small_pool(batched):
    print(f"[gpu] pageable host store, updates, batched {batched}", flush=True)
    wl = synth.workload(3)
    groups = synth.keyframe_groups(wl)[:8]
    kfs = []
    for g in groups:
        z, rgb = synth.frames(wl, g, device="cuda")
        kfs.append(scsurf.kf_fuse(torch.as_tensor(z).cuda(), torch.as_tensor(rgb).cuda(), wl.R[g], wl.t[g], wl.intr))
    first = np.array([g[0] for g in groups])
    A = (wl.R[first], wl.t[first])
    B = synth.perturb_all(A[0], A[1], 0.02, 1.0, 2)
    out = []
    for pool in (1 << 15, None):
        vol = scsurf.Volume(0.01, 0.04, 1 << 16, pool or int(0.75 * out[0]["blocks"].shape[0]), max_batch_ops=1)
        if not pool:
            vol.stream_enable(True)
            vol.stream_pinned_limit(0)
        for k, kf in enumerate(kfs):
            vol.integrate(kf, wl.intr, A[0][k], A[1][k])
        update = vol.reintegrate_batch if batched else vol.reintegrate_plain
        update(kfs, wl.intr, A, B, len(kfs), scsurf.SEL_ALL_ORDERED)
        vol.check_error()
        if not pool:
            stats = vol.stream_stats()
            assert stats[2] > 256 and stats[3] > 256  # more than the staging buffer holds, both ways
        out.append(vol.export_sorted(with_host=not pool))
        vol.close()
    _same(*out)
