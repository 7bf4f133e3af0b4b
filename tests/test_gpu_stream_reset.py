"""A reset of a streamed volume whose host store is larger than what a reset
keeps (256 MiB): only enqueued, also under stream capture, and the store
serves further turns, with the surplus given back between them."""
import numpy as np
import pytest
import torch

from paper_1709_03763_amd import scsurf

pytestmark = pytest.mark.gpu


def test_reset_of_a_large_store():
    n = 36000  # 295 MB of RGBA8 blocks
    g = torch.Generator(device="cuda").manual_seed(2)
    at = torch.randperm(48 ** 3, generator=g, device="cuda")[:n]
    blocks = torch.stack([at // 2304, at // 48 % 48, at % 48], 1).int() - 24
    f = {"blocks": blocks, "D": torch.rand((n, 512), generator=g, device="cuda"),
         "W": torch.randint(1, 900, (n, 512), generator=g, device="cuda").float(),
         "C": torch.randint(0, 256, (n, 512, 4), generator=g, device="cuda", dtype=torch.uint8)}
    vol = scsurf.Volume(0.01, 0.04, 1 << 17, n)
    for turn in range(3):
        print(f"[gpu] large host store, turn {turn}", flush=True)
        vol.import_field(f)
        vol.stream_enable(True)
        vol.stream_out((99.0, 0.0, 0.0), 1.0)
        assert vol.stream_stats()[:2] == (0, n)
        if turn < 2:
            if turn == 0:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph):
                    vol.reset()
                graph.replay()
            else:
                vol.reset()
            assert vol.stream_stats()[:2] == (0, 0)
            assert vol.query() == (0, scsurf.SC_OK)
        else:
            vol.stream_in_all()
            assert vol.check_error() == n
            e = vol.export()
            order = [torch.argsort((b[:, 0] * 48 + b[:, 1]) * 48 + b[:, 2]) for b in (e["blocks"], f["blocks"])]
            for k in f:
                assert torch.equal(e[k][order[0]], f[k][order[1]]), k
    vol.close()
