"""The MLP and feature gradients at Gaussian counts around the chunks of 128 of
the first layer's contraction (odd counts, one Gaussian, one past a chunk), and
with position blocks marked before they are cleared (RXGS_ZERO_VISIBLE_MIN=0)
for several receivers per view.  Against the oracle's reverse mode under the
suite's rule for gradients."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_24290_amd import scenes as S

from .parity import gpu, needs_gpu
from .test_gpu_backward import FIELDS_MLP, _compare, _gpu_grads

pytestmark = [gpu, needs_gpu]

GRID = S.Grid(45, 90, -math.pi / 2, math.pi / 45)


@pytest.mark.parametrize("K", [3, 127, 129, 257])
@pytest.mark.parametrize("mode", ["tx", "rx"])
def test_gaussian_counts(K, mode, monkeypatch):
    monkeypatch.setenv("RXGS_ZERO_VISIBLE_MIN", "0")
    wl = S.make_workload("c1", K=K, N=5, grid=GRID, seed=K)
    dC = np.random.default_rng(K).normal(size=(5, 2, GRID.H, GRID.W)).astype(np.float32)
    gg, _ = _gpu_grads(wl, mode, dC=dC)
    cen, rv = O.views_for(mode, wl.tx, wl.rx)
    go = O.backward(wl.scene, wl.grid, cen, wl.rx, rv, dC, None, mlp=wl.mlp)
    _compare(gg, go, FIELDS_MLP)
