"""The warp by source tiles at an odd size (650 keyframe tiles), and groups on
either side of the line between it and the warp by displacements, against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1709_03763_amd import scsurf, synth
from test_gpu_fuse_groups import _check, test_warp_displacements as displaced

pytestmark = pytest.mark.gpu


def test_displaced_frames_by_source_tiles():
    displaced(409, 387, False)


@pytest.mark.parametrize("W,H,n", [(640, 480, 12), (640, 480, 13), (400, 383, 24), (400, 384, 25), (416, 384, 24)])
def test_either_side_of_the_line(W, H, n):
    print(f"[gpu] warp rule {W}x{H}, {n} frames", flush=True)
    wl = synth.workload(2)
    idx = np.arange(n) * 4
    z, rgb = synth.frames(wl, idx)
    z, rgb = np.ascontiguousarray(z[:, :H, :W]), np.ascontiguousarray(rgb[:, :H, :W])
    i = wl.intr
    intr = synth.Intrinsics(W, H, i.fx, i.fy, i.cx, i.cy)
    kf = scsurf.kf_fuse(torch.from_numpy(z).cuda(), torch.from_numpy(rgb).cuda(), wl.R[idx], wl.t[idx], intr)
    _check(kf, oracle.kf_fuse(z, rgb, intr, wl.R[idx], wl.t[idx]))
