"""The differentiable forward on a streamed volume whose pool takes the prior
and the keyframes one by one, but not the prior and all keyframes' candidate
blocks at once: every block stays on the device, and the backward runs."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import autograd as sca
from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu

S, MU = 0.01, 0.04


def test_forward_and_backward_in_a_small_streamed_pool():
    W, H = 60, 44
    rng = np.random.default_rng(5)
    intr = synth.Intrinsics(W, H, 55.0, 55.0, 0.5 * (W - 1), 0.5 * (H - 1))
    depth = torch.from_numpy((1.0 + 0.002 * rng.standard_normal((2, H, W))).astype(np.float32)).cuda()
    weight = torch.from_numpy((rng.integers(0, 2048, (2, H, W)) / 1024.0).astype(np.float32)).cuda()
    color = torch.from_numpy(rng.uniform(0, 1, (2, H, W, 3)).astype(np.float32)).cuda()
    R, t = np.stack([np.eye(3)] * 2), np.array([[0.0, 0.0, 0.0], [9.0, 0.0, 0.0]])
    kfs = [scsurf.Keyframe(depth[k], weight[k], color[k]) for k in range(2)]
    big = scsurf.Volume(S, MU, 1 << 16, 1 << 14, color_mode=scsurf.COLOR_F32)
    proposed, touched = [], []
    for k in range(2):
        big.reset()
        big.integrate_batch(kfs[k:k + 1], intr, R[k:k + 1], t[k:k + 1])
        touched.append(big.check_error())
        proposed.append(big.stats()[0])
    n0 = 40
    blocks = torch.zeros((n0, 3), dtype=torch.int32, device="cuda")
    blocks[:, 0], blocks[:, 1] = torch.arange(n0, device="cuda"), 500
    prior = {"blocks": blocks, "D": torch.rand((n0, 512), device="cuda") * MU, "W": torch.ones((n0, 512), device="cuda"),
             "C": torch.rand((n0, 3, 512), device="cuda")}
    pool = n0 + max(proposed[0], touched[0] + proposed[1])
    assert n0 + sum(proposed) > pool
    out = []
    for vol in (big, scsurf.Volume(S, MU, 1 << 16, pool, color_mode=scsurf.COLOR_F32)):
        streamed = vol is not big
        print(f"[gpu] differentiable forward, prior, streamed {streamed}", flush=True)
        vol.stream_enable(streamed)
        d, c, xi = (x.clone().requires_grad_() for x in (depth, color, torch.zeros((2, 6), device="cuda")))
        p = dict(prior, D=prior["D"].clone().requires_grad_())
        D, C, Wv = sca.integrate(d, c, weight, xi, vol, intr, R, t, p)
        assert D.shape[0] == n0 + sum(touched)
        field = vol.export_sorted()
        (D.sum() + C.sum()).backward()
        out.append((field, [g.grad.cpu().numpy() for g in (d, c, xi)], p["D"].grad.cpu().numpy()))
        vol.close()
    for k in out[0][0]:
        np.testing.assert_array_equal(out[1][0][k], out[0][0][k], err_msg=k)
    np.testing.assert_array_equal(out[1][2], out[0][2])
    # sums of the same terms in another order
    for a, b in zip(*(o[1] for o in out)):
        np.testing.assert_allclose(a, b, rtol=1e-5, atol=1e-5 * np.abs(b).max())
