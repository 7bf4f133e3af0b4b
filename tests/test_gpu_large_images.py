"""Keyframes of more than 2^24 pixels, observed in the corner where the pixel
indices are largest: the one-keyframe and the batched update and the adjoint
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import compare_fields
from oracle import adjoint as oadj
from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu

S, MU = 0.01, 0.04
SIZES = [(5000, 4000), (16384, 1025)]


def _corner(W, H, rgba, seed):
    """Two keyframes whose last 24 x 31 pixels are observed, and their poses."""
    rng = np.random.default_rng(seed)
    intr = synth.Intrinsics(W, H, 250.0, 250.0, W - 16.0, H - 12.0)
    kfs = []
    for _ in range(2):
        z, w = np.zeros((H, W), np.float32), np.zeros((H, W), np.float32)
        z[-24:, -31:] = 0.9 + rng.normal(0, 0.002, (24, 31))
        w[-24:, -31:] = rng.integers(1, 2048, (24, 31)) / 1024.0
        c = np.zeros((H, W, 4 if rgba else 3), np.uint8 if rgba else np.float32)
        c[-24:, -31:] = rng.integers(0, 256, (24, 31, c.shape[2])) if rgba else rng.uniform(0, 1, (24, 31, 3))
        kfs.append({"depth": z, "weight": w, "color": c})
    return intr, kfs, np.stack([np.eye(3)] * 2), rng.normal(0, 0.01, (2, 3))


def _cuda(kf):
    return scsurf.Keyframe(*(torch.from_numpy(kf[k]).cuda() for k in ("depth", "weight", "color")))


@pytest.mark.parametrize("kind", ["f32", "rgba", "packed"])
@pytest.mark.parametrize("W,H", SIZES)
def test_updates_match_oracle(W, H, kind):
    print(f"[gpu] large images {W}x{H} {kind}", flush=True)
    rgba = kind != "f32"
    intr, kfs, R, t = _corner(W, H, rgba, 3)
    tn = t + np.array([0.013, -0.008, 0.004])
    ref = oracle.Volume(S, MU, color_f32=not rgba)
    for k in range(2):
        ref.integrate(kfs[k], intr, R[k], t[k])
    first = ref.export()
    assert len(first["blocks"]) > 2
    for k in range(2):
        ref.deintegrate(kfs[k], intr, R[k], t[k])
    for k in range(2):
        ref.integrate(kfs[k], intr, R[k], tn[k])
    second = ref.export()
    dk = [_cuda(k) for k in kfs]
    if kind == "packed":
        dk = [scsurf.keyframe_pack(k) for k in dk]
    for batched in (False, True):
        vol = scsurf.Volume(S, MU, 1 << 14, 1 << 10, scsurf.COLOR_RGBA8 if rgba else scsurf.COLOR_F32)
        if batched:
            vol.integrate_batch(dk, intr, R, t)
        else:
            for k in range(2):
                vol.integrate(dk[k], intr, R[k], t[k])
        vol.check_error()
        compare_fields(vol.export_sorted(), first, exact_color=rgba)
        update = vol.reintegrate_batch if batched else vol.reintegrate_plain
        update(dk, intr, (R, t), (R, tn), 2, scsurf.SEL_ALL_ORDERED)
        vol.check_error()
        compare_fields(vol.export_sorted(), second, exact_color=rgba)
        vol.close()


@pytest.mark.parametrize("W,H", SIZES)
def test_pixel_gradients_match_oracle(W, H):
    print(f"[gpu] large images {W}x{H} adjoint", flush=True)
    intr, kfs, R, t = _corner(W, H, False, 4)
    dk = [_cuda(k) for k in kfs]
    vol = scsurf.Volume(S, MU, 1 << 14, 1 << 10, scsurf.COLOR_F32)
    vol.integrate_batch(dk, intr, R, t)
    nb = vol.check_error()
    f = vol.export()
    blocks = f["blocks"].cpu().numpy().astype(np.int64)
    i = np.arange(512)
    vox = (8 * blocks[:, None, :] + np.stack([i & 7, (i >> 3) & 7, i >> 6], 1)[None]).reshape(-1, 3)
    fz = oadj.FrozenIntegration(S, MU, kfs, intr, R, t)
    rows = {tuple(x): j for j, x in enumerate(vox)}
    at = np.array([rows[tuple(x)] for x in fz.vox])
    # upstream gradients of one sign: a sum of m rounded terms is then within (m + 3) 2^-24 of itself
    rng = np.random.default_rng(7)
    gD = rng.uniform(0.1, 1.0, (nb, 512)).astype(np.float32)
    gC = rng.uniform(0.1, 1.0, (nb, 3, 512)).astype(np.float32)
    g_depth, g_color, g_xi = (torch.zeros(s, device="cuda") for s in ((2, H, W), (2, H, W, 3), (2, 6)))
    vol.integrate_backward(dk, intr, R, t, torch.from_numpy(gD).cuda(), torch.from_numpy(gC).cuda(), g_depth, g_color,
                           g_xi)
    Wv = f["W"].cpu().numpy().reshape(-1)[at].astype(np.float64)
    ref = fz.grad(gD.reshape(-1)[at].astype(np.float64),
                  gC.transpose(0, 2, 1).reshape(-1, 3)[at].astype(np.float64), R, t, Wv)
    tol = (max(np.bincount(p - p.min()).max() for p in fz.pix) + 3) * 2.0 ** -24
    for g, name in ((g_depth, "depth"), (g_color, "color")):
        g = g.cpu().numpy()
        np.testing.assert_allclose(g[:, -24:, -31:], ref[name][:, -24:, -31:], rtol=tol, atol=0)
        assert (g[:, -24:, -31:] != 0).any()
        g[:, -24:, -31:] = 0
        assert not g.any()  # no other pixel
    vol.close()
