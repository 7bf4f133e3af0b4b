"""The host store of streamed-out blocks: a field of random blocks sent out by
spheres and brought back stays the same bit for bit, with the counts that the
sphere test gives, over the store's chunks (1,024 records and more), its reuse
after a reset and calls on other streams."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf

pytestmark = pytest.mark.gpu

S = 0.01


@pytest.mark.parametrize("n,mode", [(1, scsurf.COLOR_RGBA8), (1024, scsurf.COLOR_RGBA8), (1025, scsurf.COLOR_F32),
                                    (3600, scsurf.COLOR_RGBA8)])
def test_field_survives_the_store(n, mode):
    print(f"[gpu] host store, {n} blocks, colour mode {mode}", flush=True)
    rng = np.random.default_rng(n)
    blocks = np.stack(np.unravel_index(rng.permutation(32 ** 3)[:n], (32, 32, 32)), 1).astype(np.int32) - 16
    f = {"blocks": blocks, "D": rng.normal(0, 0.02, (n, 512)).astype(np.float32),
         "W": rng.integers(1, 900, (n, 512)).astype(np.float32),
         "C": rng.integers(0, 256, (n, 512, 4), dtype=np.uint8) if mode == scsurf.COLOR_RGBA8
         else rng.uniform(0, 1, (n, 3, 512)).astype(np.float32)}
    vol = scsurf.Volume(S, 0.04, 1 << 13, n, color_mode=mode)  # the pool is full when every block is in it
    side = torch.cuda.Stream()
    for turn in range(3):
        vol.import_field({k: torch.from_numpy(v).cuda() for k, v in f.items()})
        ref = vol.export_sorted()
        vol.stream_enable(True)
        out = 0
        for center, radius in (((0.3, -0.2, 0.1), 1.2), ((-0.4, 0.3, 0.0), 0.9), ((0.0, 0.0, 0.0), 0.4),
                               ((9.0, 9.0, 9.0), 1.0)):
            at = vol.export()["blocks"].cpu().numpy().astype(np.float64)
            d = ((np.float64(np.float32(S)) * (8 * at + 3.5) - np.array(center)) ** 2).sum(1)
            gone = int((d > radius * radius).sum())
            side.wait_stream(torch.cuda.current_stream())
            vol.stream_out(center, radius, stream=side if turn == 1 else None)
            torch.cuda.current_stream().wait_stream(side)
            out += gone
            assert vol.stream_stats()[:2] == (n - out, out)
            got = vol.export_sorted(with_host=True)
            for k in ref:
                np.testing.assert_array_equal(got[k], ref[k], err_msg=k)
            if radius == 0.9:
                vol.stream_in_all()
                assert vol.stream_stats()[:2] == (n, 0)
                for k, v in vol.export_sorted().items():
                    np.testing.assert_array_equal(v, ref[k], err_msg=k)
                out = 0
        assert out == n  # the last sphere holds nothing
        if turn < 2:
            vol.reset()
        else:
            vol.stream_in_all()
            assert vol.check_error() == n
            for k, v in vol.export_sorted().items():
                np.testing.assert_array_equal(v, ref[k], err_msg=k)
        assert vol.stream_stats()[1] == 0
        vol.stream_enable(False)
    vol.close()
