"""Tile binning over the sizes its tables change at: pairs placed in their tile
lists directly with one, two or four tiles per thread (up to 1,024 tiles, at
most 255 rows and columns of them), views of more than one slice of chunks in
the scan, both chunk sizes of the emission; and the grids just outside, which
sort the pairs.  RXGS_PAIR_SORT=1 sorts them on every grid: pairs, ranges and
outputs are the same, bit for bit."""
import math

import numpy as np
import pytest

from paper_2605_24290_amd import scenes as S

from .parity import gpu, needs_gpu, renderer_for

pytestmark = [gpu, needs_gpu]


@pytest.mark.parametrize("H,W,K,N", [
    (128, 512, 3000, 3),       # 256 tiles: one per thread, all threads
    (129, 450, 3000, 3),       # 261: two per thread
    (256, 512, 20_000, 2),     # 512: two per thread, all threads; two slices of chunks
    (250, 516, 3000, 3),       # 528: four per thread
    (256, 1024, 17_000, 1),    # 1,024: the largest; two slices
    (360, 720, 3000, 2),       # 1,035: sorted
    (16, 4080, 3000, 2),       # 255 columns
    (16, 4082, 3000, 2),       # 256 columns: sorted
    (20, 40, 70_000, 16),      # 6 tiles; chunks of 1,024 entries, two slices
    (180, 360, 70_000, 16),    # 276 tiles; the same
])
def test_binning_equals_pair_sort(H, W, K, N, monkeypatch):
    import torch
    from paper_2605_24290_amd import rxgs
    wl = S.make_workload("c1", K=K, N=N, grid=S.Grid(H, W, -H * math.pi / W, 2 * math.pi / W), seed=H + W)
    out = []
    for env in ("0", "1"):
        monkeypatch.setenv("RXGS_PAIR_SORT", env)
        r = renderer_for(wl)
        saved = rxgs.Saved(r)
        C, P, _ = r.render(wl.rx, tx=wl.tx, mode="rx", saved=saved)
        torch.cuda.synchronize()
        info = saved.info()
        assert info["tiles"] == ((H + 15) // 16) * ((W + 15) // 16)
        pairs = saved.export(rxgs.EXPORT_PAIRS, np.int32, (info["D"],))
        ranges = saved.export(rxgs.EXPORT_RANGES, np.uint32, (info["V"] * info["tiles"], 2))
        out.append((C.cpu().numpy(), P.cpu().numpy(), pairs, ranges))
        saved.close()
        r.close()
    assert out[0][2].size > 100
    for a, b in zip(*out):
        assert np.array_equal(a, b)
