"""The export reads the number of blocks on the device: rows up to the capacity
given, the rest untouched, the whole number returned, for fewer and for more
blocks than the launch has workgroups."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,mode", [(1, scsurf.COLOR_RGBA8), (37, scsurf.COLOR_F32), (16500, scsurf.COLOR_RGBA8)])
def test_export_up_to_a_capacity(n, mode):
    print(f"[gpu] export of {n} blocks, colour mode {mode}", flush=True)
    rng = np.random.default_rng(n)
    blocks = np.stack(np.unravel_index(rng.permutation(32 ** 3)[:n], (32, 32, 32)), 1).astype(np.int32)
    rgba = mode == scsurf.COLOR_RGBA8
    f = {"blocks": torch.from_numpy(blocks).cuda(), "D": torch.randn((n, 512), device="cuda"),
         "W": torch.randint(1, 900, (n, 512), device="cuda").float(),
         "C": torch.randint(0, 256, (n, 512, 4), device="cuda", dtype=torch.uint8) if rgba
         else torch.rand((n, 3, 512), device="cuda")}
    vol = scsurf.Volume(0.01, 0.04, 1 << 16, 1 << 15, color_mode=mode)
    L = scsurf.lib()
    out = ctypes.c_int64(-1)
    scsurf.check(L.sc_volume_export(vol.handle, scsurf.stream_handle(), None, None, None, None, 5, ctypes.byref(out)),
                 "empty")
    assert out.value == 0
    vol.import_field(f)
    whole = vol.export()
    order = lambda b: np.lexsort(b.cpu().numpy().T)  # noqa: E731
    o, e = order(whole["blocks"]), order(f["blocks"])
    for k in f:
        assert torch.equal(whole[k][o], f[k][e]), k
    for cap in sorted({0, 1, n - 1, n, n + 5}):
        rows = max(cap, 1) + 1
        buf = {k: torch.full((rows,) + v.shape[1:], 7, dtype=v.dtype, device="cuda") for k, v in whole.items()}
        scsurf.check(L.sc_volume_export(vol.handle, scsurf.stream_handle(), buf["blocks"].data_ptr(),
                                        buf["D"].data_ptr(), buf["W"].data_ptr(), buf["C"].data_ptr(), cap,
                                        ctypes.byref(out)), "export")
        assert out.value == n
        m = min(cap, n)
        for k in buf:
            assert torch.equal(buf[k][:m], whole[k][:m]) and (buf[k][m:] == 7).all(), (cap, k)
    only = torch.full((n, 512), 7.0, device="cuda")
    scsurf.check(L.sc_volume_export(vol.handle, scsurf.stream_handle(), None, None, only.data_ptr(), None, n, None), "W")
    assert torch.equal(only, whole["W"])
    vol.close()
