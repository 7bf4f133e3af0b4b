"""The one-keyframe update's touched-block records, taken by a batched
de-integration: a record of a few blocks, of thousands, and one that outgrows
what a wavefront holds (2.5 mm voxels: about 10^5 candidates), each against
the plain path, bit for bit; packed keyframes and unpacked ones."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("voxel,rows", [(0.02, 4), (0.01, 480), (0.0025, 480)])
def test_plain_integration_then_batched_update(voxel, rows, packed):
    print(f"[gpu] plain records: voxel {voxel}, {rows} rows, packed {packed}", flush=True)
    wl = synth.workload(2)
    z, rgb = synth.frames(wl, [0], device="cuda")
    kf = scsurf.kf_fuse(torch.from_numpy(z).cuda(), torch.from_numpy(rgb).cuda(), wl.R[:1], wl.t[:1], wl.intr)
    kf.weight[rows:] = 0.0
    if packed:
        kf = scsurf.keyframe_pack(kf)
    Rn, tn = synth.perturb_fixed(wl.R[:1], wl.t[:1], 0.02, 1.0, 5)
    vols = [scsurf.Volume(voxel, 4 * voxel, 1 << 20, 1 << 18) for _ in range(2)]
    for v in vols:
        v.integrate(kf, wl.intr, wl.R[0], wl.t[0])
    vols[0].reintegrate_batch([kf], wl.intr, (wl.R[:1], wl.t[:1]), (Rn, tn), 1)
    vols[1].deintegrate(kf, wl.intr, wl.R[0], wl.t[0])
    vols[1].integrate(kf, wl.intr, Rn[0], tn[0])
    n = [v.check_error() for v in vols]
    assert n[0] == n[1] and (voxel > 0.0025 or n[0] > 65536)
    a, b = (v.export_sorted() for v in vols)
    assert (a["W"] > 0).any()
    for k in ("blocks", "D", "W", "C"):
        np.testing.assert_array_equal(a[k], b[k])
