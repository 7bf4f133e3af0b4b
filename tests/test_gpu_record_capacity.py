"""Touched-block records up to their capacity (16,384 blocks, however the
appends are spread): a de-integration takes the record as its candidates,
which shows in the candidate count; above the capacity it generates them.
Written by the one-keyframe update and by the batched one; each against the
one-keyframe path bit for bit."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu

CAPACITY = 16384
VOXEL = 0.005


@pytest.fixture(scope="module")
def view():
    wl = synth.workload(2)
    z, rgb = synth.frames(wl, [0], device="cuda")
    kf = scsurf.kf_fuse(torch.from_numpy(z).cuda(), torch.from_numpy(rgb).cuda(), wl.R[:1], wl.t[:1], wl.intr)
    vol = scsurf.Volume(VOXEL, 4 * VOXEL, 1 << 18, 1 << 16)

    def rows(n):
        return scsurf.Keyframe(kf.depth, torch.cat([kf.weight[:n], torch.zeros_like(kf.weight[n:])]), kf.color)

    def touched(n):
        vol.reset()
        vol.integrate(rows(n), wl.intr, wl.R[0], wl.t[0])
        return vol.check_error()

    def most(limit):  # the rows that touch at most `limit` blocks
        lo, hi = 0, wl.intr.height
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if touched(mid) <= limit else (lo, mid)
        return lo

    yield wl, rows, touched, most
    vol.close()


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("writer", ["plain", "batch"])
@pytest.mark.parametrize("limit,used", [(12000, True), (CAPACITY, True), (CAPACITY + 500, False)])
def test_record_of_many_blocks(view, limit, used, writer, packed):
    print(f"[gpu] record of {limit} blocks, {writer}, packed {packed}", flush=True)
    wl, rows, touched, most = view
    n_rows = most(limit)
    n = touched(n_rows)
    assert limit - 200 < n <= limit
    kf = rows(n_rows)
    if packed:
        kf = scsurf.keyframe_pack(kf)
    A = (wl.R[:1], wl.t[:1])
    B = (wl.R[:1], wl.t[:1] + 8 * VOXEL * np.array([500.0, 0.0, 0.0]))  # whole blocks away: the same blocks, moved
    vol = scsurf.Volume(VOXEL, 4 * VOXEL, 1 << 18, 1 << 16)
    proposed = []
    for T in (A, B):
        vol.reset()
        vol.integrate_batch([kf], wl.intr, *T)
        vol.check_error()
        proposed.append(vol.stats()[0])
    vol.reset()
    if writer == "plain":
        vol.integrate(kf, wl.intr, A[0][0], A[1][0])
    else:
        vol.integrate_batch([kf], wl.intr, *A)
    before = vol.stats()[0]
    vol.reintegrate_batch([kf], wl.intr, A, B, 1, scsurf.SEL_ALL_ORDERED)
    vol.check_error()
    assert proposed[0] > n
    assert vol.stats()[0] - before == (n if used else proposed[0]) + proposed[1]
    got = vol.export_sorted()
    vol.reset()
    vol.integrate(kf, wl.intr, A[0][0], A[1][0])
    vol.deintegrate(kf, wl.intr, A[0][0], A[1][0])
    vol.integrate(kf, wl.intr, B[0][0], B[1][0])
    vol.check_error()
    exp = vol.export_sorted()
    vol.close()
    for k in exp:
        np.testing.assert_array_equal(got[k], exp[k], err_msg=k)
