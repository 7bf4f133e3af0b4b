"""The distance search leaves cells out by their boxes: against every pair, in
the same FP32 operations, on points at and beside cell borders, at large
coordinates (up to the clamped cells), and on infinite and NaN coordinates."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import surface

pytestmark = pytest.mark.gpu


def _all_pairs(ref, q, radius):
    e = [q[:, None, r] - ref[None, :, r] for r in range(3)]
    d2 = (e[0] * e[0] + e[1] * e[1]) + e[2] * e[2]
    d2 = torch.where(torch.isnan(d2), torch.full_like(d2, float("inf")), d2).amin(1)
    return torch.clamp(torch.sqrt(d2), max=float(np.float32(radius)))


@pytest.mark.parametrize("radius", [0.05, 1.0e-3, 3.0e-23, 7.0])
@pytest.mark.parametrize("where", ["inside", "borders", "far", "clamped", "odd"])
def test_pruned_search_equals_all_pairs(radius, where):
    print(f"[gpu] distances: radius {radius}, {where}", flush=True)
    rng = np.random.default_rng(11)
    edge = float(np.float32(radius)) * (1.0 + 1.0 / 64.0)
    cells = {"inside": 6, "borders": 4, "far": 5, "clamped": 3, "odd": 4}[where]
    p = rng.uniform(-cells, cells, (3000, 3))
    if where == "borders":
        # integers of the cell coordinate, a few steps of FP32 to either side
        p = np.rint(p) * (1.0 + rng.integers(-3, 4, p.shape) * 2.0 ** -23)
    if where == "far":
        p[:, 0] += 90000.0
        p[:, 1] -= 300000.0
    if where == "clamped":
        p[:, 0] += 1.0e6
        p[:, 2] -= 1.0e6
    p = (p * edge).astype(np.float32)
    if where == "odd":
        p[::97, 0], p[5::101, 1], p[7::103, 2] = np.nan, np.inf, -np.inf
    ref, q = torch.from_numpy(p[:1700]).cuda(), torch.from_numpy(p[1700:]).cuda()
    d, total = surface.nn_distance(ref, q, radius)
    want = _all_pairs(ref, q, radius)
    # one FP32 step of the square root
    torch.testing.assert_close(d, want, rtol=2.0 ** -23, atol=0.0)
    assert abs(total - float(d.double().sum())) <= 1e-12 * float(d.double().sum())
