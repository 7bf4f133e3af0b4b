"""A fusion under stream capture whose images the workspace already fits: it
allocates nothing, whatever earlier calls were.  The captured graph is
replayed with other work between and equals the eager fusion."""
import pytest
import torch

from paper_1709_03763_amd import scsurf, synth

pytestmark = pytest.mark.gpu


def test_fusion_of_many_frames_captured_after_colour_prep():
    # larger than any fusion of the other tests, which share the workspace
    n, W, H = 30, 1400, 1000
    print(f"[gpu] fusion of {n} frames {W}x{H} captured", flush=True)
    g = torch.Generator().manual_seed(3)
    rgb = torch.randint(0, 256, (n, H, W, 3), generator=g, dtype=torch.uint8).cuda()
    u, v = torch.arange(W, device="cuda"), torch.arange(H, device="cuda")[:, None]
    depth = (1.5 + 0.1 * torch.sin(0.01 * u) + 0.05 * torch.cos(0.02 * v)).expand(n, H, W).contiguous()
    intr = synth.Intrinsics(W, H, 1200.0, 1200.0, 0.5 * (W - 1), 0.5 * (H - 1))
    R = torch.eye(3).expand(n, 3, 3).numpy().astype("float64")
    t = torch.zeros((n, 3)).numpy().astype("float64")
    t[:, 0] = [0.002 * i for i in range(n)]
    out = scsurf.Keyframe(torch.zeros((H, W), device="cuda"), torch.zeros((H, W), device="cuda"),
                          torch.zeros((H, W, 4), dtype=torch.uint8, device="cuda"))
    scsurf.color_prep(rgb)  # the workspace for these images
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        scsurf.kf_fuse(depth, rgb, R, t, intr, out=out)
    ref = scsurf.kf_fuse(depth, rgb, R, t, intr)
    assert (ref.weight > 0).float().mean().item() > 0.5
    for _ in range(3):
        for x in (out.depth, out.weight, out.color):
            x.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        for a in ("depth", "weight", "color"):
            assert torch.equal(getattr(out, a), getattr(ref, a)), a
