"""The multi-receiver blend (chunks of up to 16 or 32 rows on the matrix
cores) at the edges of its chunks: views of 2 to 33 receivers, a view of one
receiver beside others, partial last groups of four entries, a radiance
prefix with records, and the 32-row chunks of very large launches.  Spectra
against the FP64 oracle under the suite's rule (1e-4 of a receiver's largest
value; the sums are FP32 as before); a receiver's spectrum does not depend on
the chunk it falls in, so other batchings of the same receivers give the same
bits."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_24290_amd import scenes as S

from .parity import compare_spectra, gpu, needs_gpu, renderer_for

pytestmark = [gpu, needs_gpu]

GRID = S.Grid(45, 90, -math.pi / 2, math.pi / 45)


@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("sizes,K", [((2,), 5), ((3, 1, 17), 301), ((16, 0, 33), 700), ((15, 32), 1203)])
def test_rows_per_view(sizes, K, saved):
    import torch
    from paper_2605_24290_amd import rxgs
    wl = S.make_workload("c1", K=K, N=sum(sizes), Q=len(sizes), grid=GRID, seed=91 + K)
    off = [0] + [int(x) for x in np.cumsum(sizes)]
    r = renderer_for(wl)
    st = rxgs.Saved(r) if saved else None
    C, P, _ = r.render(wl.rx, tx=wl.tx, rx_off=off, mode="tx", saved=st)
    torch.cuda.synchronize()
    cen, rv = O.views_for("tx", wl.tx, wl.rx, off)
    ora = O.render(wl.scene, wl.grid, cen, wl.rx, rv, mlp=wl.mlp)
    compare_spectra(C.cpu().numpy(), ora)
    assert (np.abs(P.cpu().numpy() - ora["power"]) <= 1e-4 * np.abs(ora["power"])).all()
    if saved:
        # the radiance export: one row per receiver, whatever the device layout
        info = st.info()
        rad = st.export(rxgs.EXPORT_RADIANCE, np.float32, (info["N"], info["K_pad"], 2))
        order = st.export(rxgs.EXPORT_ORDER, np.int32, (info["V"], info["K_pad"]))
        nvis = st.export(rxgs.EXPORT_NVIS, np.int32, (info["V"],))
        want = O.radiance(wl.scene, wl.rx, wl.mlp)
        for v in range(len(sizes)):
            for j in range(off[v], off[v + 1]):
                ref = want[j][order[v, :nvis[v]]]
                assert np.abs(rad[j, :nvis[v]] - ref).max(initial=0) <= 2e-5 * max(np.abs(want[j]).max(), 1e-30)
        st.close()
    r.close()


def test_rows_batching_bits():
    """64 receivers of one transmitter in a thick scene (prefix and records):
    together, in batches of 16, and in ragged batches."""
    import torch
    wl = S.make_workload("c1", K=20_000, N=64)
    r = renderer_for(wl)
    C = r.render(wl.rx, tx=wl.tx, mode="tx")[0].clone()
    for cuts in (range(0, 65, 16), (0, 2, 5, 22, 64)):
        cuts = list(cuts)
        for a, b in zip(cuts[:-1], cuts[1:]):
            part = r.render(wl.rx[a:b], tx=wl.tx, mode="tx")[0]
            assert torch.equal(part, C[a:b]), (a, b)
    r.close()


def test_wide_chunks_bits():
    """979 receivers on 270 tiles: chunks of 32 rows, against batches that
    take chunks of 16 (of at least two receivers: a launch of one row per view
    evaluates the exponent in another form)."""
    import torch
    grid = S.Grid(90, 720, 0.0, math.pi / 180)
    wl = S.make_workload("c1", K=400, N=979, grid=grid)
    r = renderer_for(wl)
    C, P, _ = r.render(wl.rx, tx=wl.tx, mode="tx")
    C, P = C.clone(), P.clone()
    for a in range(0, 979, 162):
        b = min(a + 162, 979)
        Cp, Pp, _ = r.render(wl.rx[a:b], tx=wl.tx, mode="tx")
        assert torch.equal(Cp, C[a:b]) and torch.equal(Pp, P[a:b]), a
    r.close()


@pytest.mark.parametrize("H,W,K,N,faint", [
    (18, 72, 9000, 21, True),     # lists of several staged batches, never saturated, past the prefix
    (18, 72, 9000, 21, False),
    (45, 90, 3000, 16, True),     # full sphere: entries around the azimuth circle; ragged tiles
    (5, 6, 700, 2, True),         # one tile, most of it outside the grid
    (90, 360, 513, 33, False),    # one entry past a batch at most
])
def test_few_workgroups_bits(H, W, K, N, faint):
    """Launches of few workgroups (eight waves per tile) against saving renders of
    the same receivers, which take four: spectra and powers bit for bit."""
    import torch
    from paper_2605_24290_amd import rxgs
    el0 = 0.0 if H * 4 == W else -math.pi / 2
    wl = S.make_workload("c1", K=K, N=N, grid=S.Grid(H, W, el0, (math.pi / 2 if el0 == 0.0 else math.pi) / H), seed=K + N)
    if faint:
        wl.scene.logits[:] -= 4.0
    r = renderer_for(wl)
    C, P, _ = r.render(wl.rx, tx=wl.tx, mode="tx")
    C, P = C.clone(), P.clone()
    st = rxgs.Saved(r)
    Cs, Ps, _ = r.render(wl.rx, tx=wl.tx, mode="tx", saved=st)
    torch.cuda.synchronize()
    assert float(C.abs().max()) > 0
    assert torch.equal(C, Cs) and torch.equal(P, Ps)
    st.close()
    r.close()
