"""The conditioned radiance at the channel counts its kernels change at: one to
four channels (a lane per position and channel, the basis walked by each), five
and more (basis values through LDS, several positions per lane; the local MLP's
last layer in blocks of 8 channels) with full and part-filled channel groups,
and more components than the LDS table takes.  Against the FP64 oracle under
the rule of the other conditioned-radiance tests (2e-5 of a row's largest
value: sums of at most 100 FP32 terms)."""
import numpy as np
import pytest

from oracle import oracle as O

from .parity import gpu, needs_gpu
from .test_gpu_rxcond import _check_radiance, _gpu_radiance, _setup, _views

pytestmark = [gpu, needs_gpu]


@pytest.mark.parametrize("mode,kind,lmax,C", [
    ("tx", O.BASIS_FLE, 2, 4),
    ("rx", O.BASIS_FLE, 4, 5),
    ("tx", O.BASIS_SH, 0, 8),
    ("rx", O.BASIS_FLE, 4, 9),
    ("rx", O.BASIS_SH, 3, 16),
    ("tx", O.BASIS_FLE, 4, 17),
    ("tx", O.BASIS_FLE, 6, 32),    # 49 components: the LDS table's largest
    ("rx", O.BASIS_SH, 7, 6),      # 64: past it
])
def test_channel_layouts(mode, kind, lmax, C):
    import torch
    from paper_2605_24290_amd import rxgs
    N = 3
    r, wl, m = _setup(333, N, kind, lmax, C, seed=40 + C)   # (a part-filled last item)
    saved = rxgs.Saved(r)
    r.render_rxcond(wl.rx, tx=wl.tx, mode=mode, saved=saved)
    torch.cuda.synchronize()
    rad, order, nvis = _gpu_radiance(r, saved, N, C)
    cen, rv = _views(mode, wl)
    ora = O.rxcond_radiance(m, wl.scene, cen, wl.rx, rv, occ=O.occupancy(wl.scene, m.G))
    _check_radiance(rad, order, nvis, ora, rv, C)
    saved.close()
    r.close()
