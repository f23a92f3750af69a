"""Renders near the scratch array's limit (rxgs_render_noalloc): sizes that fill
RXGS_NOALLOC_SCRATCH_BYTES with 52-byte projection terms per Gaussian and no
sums per slice of chunks stay accepted with the wider layout, on grids on both
sides of 255 tiles, and equal rxgs_render bit for bit."""
import math

import pytest

from paper_2605_24290_amd import scenes as S

from .parity import gpu, needs_gpu
from .test_zz_no_alloc import _call_noalloc, _reference

pytestmark = [gpu, needs_gpu]

UPPER1 = S.Grid(90, 360, 0.0, math.pi / 180)
FULL1 = S.Grid(180, 360, -math.pi / 2, math.pi / 180)
UPPER5 = S.Grid(18, 72, 0.0, math.pi / 36)


@pytest.mark.parametrize("grid, K, N, mode", [
    (UPPER1, 433_500, 1, "rx"), (UPPER1, 1_000, 102, "rx"), (UPPER1, 20_000, 374, "tx"),
    (FULL1, 260_500, 1, "rx"), (FULL1, 1_000, 63, "rx"), (FULL1, 20_000, 346, "tx"),
    (UPPER5, 462_000, 1, "rx"), (UPPER5, 1_000, 170, "rx"), (UPPER5, 20_000, 391, "tx")])
def test_noalloc_near_the_scratch_limit(grid, K, N, mode, monkeypatch):
    import torch
    from paper_2605_24290_amd import rxgs
    monkeypatch.delenv("RXGS_PAIR_SORT", raising=False)   # (the sort's other copies take more)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    box = torch.tensor([10.0, 10.0, 3.0], device="cuda")

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    q = normal(K, 4)   # (the order of the draws fixes the scene, and with it the pairs)
    means = torch.rand((K, 3), generator=g, device="cuda") * box
    scene = [means, -1.5 + 0.3 * normal(K, 3), q / q.norm(dim=1, keepdim=True), normal(K)]
    r = rxgs.Renderer(grid)
    r.upload_scene(*scene, radiance=normal(K, 2))
    g.manual_seed(6)
    rx = (torch.rand((N, 3), generator=g, device="cuda") * box).cpu().numpy()
    tx = None if mode == "rx" else rx[:1]
    st, *got = _call_noalloc(r, rx, tx, mode)
    assert st == 0, rxgs.lib().rxgs_last_error(r._ctx)
    for a, b in zip(got, _reference(r, rx, tx, mode)):
        assert torch.equal(a, b)
    r.close()
