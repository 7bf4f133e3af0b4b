"""Triangles of a block are listed a window at a time: a checkerboard field,
whose blocks hold far more than one window, and ragged neighbourhoods (one
block to a 2x2x2 group with each corner block missing in turn), against the
oracle's triangles in the library's order."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mesh as M
from paper_1709_03763_amd import scsurf

pytestmark = pytest.mark.gpu

S = 0.01


def _mesh(blocks, D, W):
    vol = scsurf.Volume(S, 4 * S, 1 << 10, 1 << 8)
    vol.import_field({"blocks": torch.from_numpy(blocks).cuda(), "D": torch.from_numpy(D).cuda(),
                      "W": torch.from_numpy(W).cuda()})
    xyz, keys = vol.mesh()
    # fewer rows than triangles: the first ones; one output alone
    part = torch.full((max(len(xyz) - 5, 1), 3, 3), -7.0, device="cuda")
    n = ctypes.c_int64()
    scsurf.check(scsurf.lib().sc_volume_mesh(vol.handle, scsurf.stream_handle(), part.data_ptr(), None,
                                             len(part) - 1, ctypes.byref(n)), "sc_volume_mesh")
    assert n.value == len(xyz)
    assert torch.equal(part[:-1], xyz[:len(part) - 1]) and (part[-1] == -7.0).all()
    f = {"blocks": blocks.astype(np.int64), "D": D.astype(np.float64), "W": W.astype(np.float64)}
    return xyz.cpu().numpy(), keys.cpu().numpy(), M.marching_cubes(f, S)


def _sorted(tri, keys):
    """Each triangle from its smallest key on, the triangles in key order."""
    code = (keys.astype(np.int64) + (1 << 10)) @ np.array([1 << 36, 1 << 24, 1 << 12, 1], np.int64)
    at = (np.argmin(code, 1)[:, None] + np.arange(3)) % 3
    code, tri = np.take_along_axis(code, at, 1), np.take_along_axis(tri, at[..., None], 1)
    o = np.lexsort(code.T[::-1])
    return tri[o], code[o]


@pytest.mark.parametrize("missing", [-2, -1] + list(range(8)))
def test_checkerboard_and_ragged_neighbourhoods(missing):
    print(f"[gpu] mesh windows, missing {missing}", flush=True)
    rng = np.random.default_rng(missing + 20)
    n = [(x, y, z) for z in (0, 1) for y in (0, 1) for x in (0, 1)]
    blocks = np.array([b for i, b in enumerate(n) if i != missing] if missing > -2 else [(0, 0, 0)], np.int32) - 1
    x, y, z = np.meshgrid(*[np.arange(8)] * 3, indexing="ij")
    sign = np.where((x + y + z).transpose(2, 1, 0).reshape(-1) % 2, -1.0, 1.0)
    D = (sign * rng.uniform(0.001, 0.03, (len(blocks), 512))).astype(np.float32)
    W = np.where(rng.random((len(blocks), 512)) < (0.0 if missing < 0 else 0.02), 0.0, 1.0).astype(np.float32)
    xyz, keys, (tri, ref_keys) = _mesh(blocks, D, W)
    assert len(xyz) == len(tri) and (missing >= 0 or len(xyz) > 1024)
    a, b = _sorted(xyz, keys), _sorted(np.asarray(tri), np.asarray(ref_keys).reshape(len(tri), 3, 4))
    np.testing.assert_array_equal(a[1], b[1])
    np.testing.assert_array_equal(a[0], b[0].astype(np.float32))
