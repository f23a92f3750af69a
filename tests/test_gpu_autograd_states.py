"""Forward states kept between the autograd function's steps: the same
gradients as with fresh states (one and several renders per graph, a changing
scene size, a second stream), a bounded number of them, and their memory given
back when an allocation fails and on close."""
import math

import numpy as np
import pytest

from paper_2605_24290_amd import scenes as S

from .parity import gpu, needs_gpu

pytestmark = [gpu, needs_gpu]

GRID = S.Grid(18, 36, -math.pi / 2, math.pi / 18)


def _leaves(wl):
    import torch
    sc = wl.scene
    ts = [sc.means, sc.log_scales, sc.quats, sc.logits, sc.features, S.flat_mlp(wl.mlp)]
    return [torch.tensor(t, device="cuda", requires_grad=True) for t in ts]


def _step(r, wl, leaves, cuts=((0, None),)):
    """Gradients of a loss over the receivers, in len(cuts) renders of one graph."""
    import torch
    from paper_2605_24290_amd.autograd import rx_render
    tx, rx = torch.as_tensor(wl.tx, device="cuda"), torch.as_tensor(wl.rx, device="cuda")
    loss = 0.0
    for a, b in cuts:
        C, P = rx_render(r, *leaves, rx[a:b], tx=tx)
        loss = loss + (C - 0.1).square().sum() + 0.2 * P.sum()
    return torch.autograd.grad(loss, leaves)


def _close(a, b):
    # two runs of the atomic backward: FP32 sums of at most some thousand terms in another order
    for x, y in zip(a, b):
        assert float((x - y).abs().max()) <= 1e-5 * max(float(y.abs().max()), 1e-30)


def test_reused_states_same_gradients():
    import torch
    from paper_2605_24290_amd import rxgs
    r = rxgs.Renderer(GRID)
    cuts = ((0, 2), (2, 3), (3, 7))
    for K in (300, 900, 120):
        wl = S.make_workload("c1", K=K, N=7, grid=GRID)
        leaves = _leaves(wl)
        fresh = rxgs.Renderer(GRID)
        want, want3 = _step(fresh, wl, leaves), _step(fresh, wl, leaves, cuts)
        fresh.close()
        for _ in range(3):
            _close(_step(r, wl, leaves), want)
            _close(_step(r, wl, leaves, cuts), want3)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            other = _step(r, wl, leaves)
        mine = _step(r, wl, leaves)
        torch.cuda.synchronize()
        _close(other, want)
        _close(mine, want)
    assert len(r._idle) == 3
    assert r.release_idle_states() == 3 and r.release_idle_states() == 0
    _step(r, wl, leaves, tuple((i, i + 1) for i in range(7)))
    assert len(r._idle) == rxgs.Renderer.IDLE_MAX
    r.close()
    assert not r._idle


def test_second_backward_still_refused():
    import torch
    from paper_2605_24290_amd import rxgs
    from paper_2605_24290_amd.autograd import rx_render
    wl = S.make_workload("c1", K=100, N=2, grid=GRID)
    leaves = _leaves(wl)
    r = rxgs.Renderer(GRID)
    C, _ = rx_render(r, *leaves, torch.as_tensor(wl.rx, device="cuda"), tx=torch.as_tensor(wl.tx, device="cuda"))
    C.sum().backward(retain_graph=True)
    with pytest.raises(rxgs.RxgsError):
        C.sum().backward()
    r.close()


def test_given_back_when_memory_runs_out():
    import torch
    from paper_2605_24290_amd import rxgs
    al = rxgs.TorchAllocator()
    r = rxgs.Renderer(GRID, allocator=al)
    wl = S.make_workload("c1", K=500, N=4, grid=GRID)
    leaves = _leaves(wl)
    _step(r, wl, leaves)
    torch.cuda.synchronize()
    assert len(r._idle) == 1
    held = al.live_bytes
    # the next allocation fails (both its sizes are asked for): the kept state
    # goes back and the render succeeds
    big = S.make_workload("c1", K=500, N=64, grid=GRID)
    want = rxgs.Renderer(GRID)
    want.upload_scene(*[t.detach() for t in leaves[:4]], features=leaves[4].detach())
    want.upload_mlp(leaves[5].detach())
    ref = want.render(big.rx, tx=big.tx)[0]
    al.fail_next = 2
    got = r.render(big.rx, tx=big.tx)[0]
    assert al.n_failed == 2 and not r._idle
    assert torch.equal(got, ref)
    # without kept states an allocation failure is reported as before
    r2 = rxgs.Renderer(GRID, allocator=al)
    r2.upload_scene(*[t.detach() for t in leaves[:4]], features=leaves[4].detach())
    r2.upload_mlp(leaves[5].detach())
    al.fail_next = 2
    with pytest.raises(rxgs.RxgsError) as e:
        r2.render(big.rx, tx=big.tx)
    assert e.value.status == 2
    for x in (r, r2, want):
        x.close()
    assert held > 0 and al.live_bytes == 0
