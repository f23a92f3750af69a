"""Performance cases of the multi-receiver Gaussian rasterizer.

Each case is one call (or one training step) through the package's public
entry points, as a program that uses it makes it: renders of receiver batches
in both view modes, training steps with gradients of every parameter, the
conditioned radiance, and coverage maps.  Sizes follow the package's own
presets (paper_2605_24290_amd/scenes.py) and its benchmark's workloads; the
inputs are drawn on the GPU from the seed alone, with the presets'
distributions.

``exact`` evaluates the same outputs in 64 bits with plain torch: every pixel
walks its view's Gaussians in (32-bit depth key, index) order, without tiles,
lists or sorts of pairs.
"""
import math
import random

import torch

from paper_2605_24290_amd import autograd, rxgs, scenes

DEVICE = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")

# (rows, columns, full sphere): the 1-degree upper hemisphere of the spatial
# spectra, 2 degrees and 1 degree over the full sphere, and the 5-degree grid
# of the channel-state workload
GRIDS = {"upper1": (90, 360, False), "full2": (90, 180, True), "full1": (180, 360, True),
         "upper5": (18, 72, False)}
# scene boxes (m) with the log-scale mean and deviation of their Gaussians
ROOMS = {"hall": ((10.0, 10.0, 3.0), -1.5, 0.3), "room": ((8.0, 6.0, 3.0), -1.5, 0.3),
         "floor": ((40.0, 40.0, 4.0), -1.0, 0.5)}


def listed():
    return [
        # one receiver at a time, as the per-receiver loop and an interactive
        # query call it: launches and the wait for the counts set its time
        dict(name="render_one_rx", op="render", K=32_000, N=1, Q=1, mode="rx", grid="upper1", room="room",
             radiance="mlp"),
        # the smallest training step, through the autograd function: a scene
        # of direct radiance while a model is brought up
        dict(name="train_small_direct", op="autograd", K=1_024, N=4, Q=1, mode="tx", grid="full2", room="hall",
             radiance="direct"),
        # the benchmark's render: 64 receivers, each its own view
        dict(name="render_rx_64", op="render", K=50_000, N=64, Q=1, mode="rx", grid="upper1", room="hall",
             radiance="mlp"),
        # the same receivers sharing one transmitter's view
        dict(name="render_tx_64", op="render", K=50_000, N=64, Q=1, mode="tx", grid="upper1", room="hall",
             radiance="mlp"),
        # a full-sphere grid at 1 degree, with an odd receiver count
        dict(name="render_rx_sphere", op="render", K=50_000, N=17, Q=1, mode="rx", grid="full1", room="hall",
             radiance="mlp"),
        # a batch of a serving loop: 16 transmitters of uneven receiver sets
        # over the resident 200k-Gaussian scene
        dict(name="render_tx_batch", op="render", K=200_000, N=701, Q=16, mode="tx", grid="upper1", room="hall",
             radiance="mlp"),
        # training steps on 100k Gaussians and 32 receivers, in both modes
        dict(name="train_rx_32", op="train", K=100_000, N=32, Q=1, mode="rx", grid="upper1", room="hall",
             radiance="mlp"),
        dict(name="train_tx_32", op="autograd", K=100_000, N=32, Q=1, mode="tx", grid="upper1", room="hall",
             radiance="mlp"),
        # the conditioned radiance at its inference size: 21 receivers, 100
        # components; and 26 channels per receiver, each its own view
        dict(name="cond_fle_tx", op="rxcond", K=32_000, N=21, Q=1, mode="tx", grid="upper1", room="room",
             basis="fle", lmax=9, channels=1),
        dict(name="cond_channels_rx", op="rxcond", K=32_000, N=21, Q=1, mode="rx", grid="upper5", room="room",
             basis="fle", lmax=4, channels=26),
        # the largest scene: a coverage map of 4,096 receivers, and a training
        # step over a batch of views
        dict(name="coverage_4096", op="coverage", K=1_000_000, N=4_096, Q=1, mode="tx", grid="upper1", room="floor",
             radiance="mlp"),
        dict(name="train_rx_floor", op="train", K=1_000_000, N=128, Q=1, mode="rx", grid="upper1", room="floor",
             radiance="mlp"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(["render", "render", "render", "train", "train", "autograd", "rxcond", "coverage"])
    c = dict(op=op, K=0, N=0, Q=1, mode=rng.choice(["rx", "tx"]), grid="upper1", room="hall", radiance="mlp")
    if op == "render":
        c.update(K=_log_int(rng, 1_000, 250_000), N=_log_int(rng, 1, 128),
                 grid=rng.choice(["upper1", "upper1", "full2", "full1"]),
                 radiance=rng.choice(["mlp", "mlp", "mlp", "direct"]), room=rng.choice(["hall", "room"]))
        if c["mode"] == "tx":
            c.update(Q=rng.randint(1, 16), N=_log_int(rng, 16, 800))
    elif op in ("train", "autograd"):
        c.update(K=_log_int(rng, 1_000, 150_000), N=_log_int(rng, 1, 48), grid=rng.choice(["upper1", "upper1", "full2"]),
                 radiance=rng.choice(["mlp", "mlp", "mlp", "direct"]))
    elif op == "rxcond":
        del c["radiance"]
        c.update(K=_log_int(rng, 2_000, 40_000), N=_log_int(rng, 1, 24), room="room",
                 basis=rng.choice(["fle", "sh"]), lmax=rng.randint(2, 9), channels=1)
        if rng.random() < 0.4:
            c.update(grid="upper5", lmax=rng.randint(1, 4), channels=rng.randint(2, 26))
    else:
        c.update(K=_log_int(rng, 100_000, 1_000_000), N=_log_int(rng, 300, 4_096), mode="tx", room="floor")
    return c


# ---------------------------------------------------------------------------
# inputs

def _grid(case):
    H, W, full = GRIDS[case["grid"]]
    return scenes.Grid(H, W, -math.pi / 2 if full else 0.0, (math.pi if full else math.pi / 2) / H)


def _inputs(case, seed):
    """Seeded inputs on the device, drawn with the presets' distributions."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed * 7919 + 8371)
    (bx, by, bz), mu, sd = ROOMS[case["room"]]
    K, N, Q = case["K"], case["N"], case["Q"]
    box = torch.tensor([bx, by, bz], device=DEVICE)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEVICE)

    def uniform(*shape):
        return torch.rand(shape, generator=g, device=DEVICE)

    p = dict(means=uniform(K, 3) * box, log_scales=mu + sd * normal(K, 3))
    q = normal(K, 4)
    p["quats"] = q / q.norm(dim=1, keepdim=True)
    p["logits"] = normal(K)
    if case.get("radiance") == "mlp":
        p["features"] = normal(K, scenes.FEAT_DIM)
        parts = []
        for shape in scenes.MLP_SHAPES:
            bound = math.sqrt(6.0 / (shape[0] + shape[1])) if len(shape) == 2 else 0.0
            parts.append(((2.0 * uniform(*shape) - 1.0) * bound).reshape(-1))
        p["mlp"] = torch.cat(parts)
    elif case.get("radiance") == "direct":
        a, ph = torch.exp(0.5 * normal(K)), 2.0 * math.pi * uniform(K)
        p["radiance"] = torch.stack([a * torch.cos(ph), a * torch.sin(ph)], dim=1)
    tx, rx = uniform(Q, 3) * box, uniform(N, 3) * box
    off = None
    if case["mode"] == "tx":
        # receivers per transmitter: log-uniform from 1 to 256, scaled to N in all
        w = torch.exp(torch.rand(Q, generator=g, device=DEVICE).double() * math.log(257.0)).cpu()
        cum = torch.cumsum(w, 0) / w.sum()
        q0 = min(Q, N)
        off = [0] + [int(min(i + 1, q0) + round(float(c) * (N - q0))) for i, c in enumerate(cum)]
    else:
        tx = None
    return p, tx, rx, off, g


def _cond_model(case, g):
    """The conditioning model's arrays (coefficients, flat parameters)."""
    L, C = (case["lmax"] + 1) ** 2, case["channels"]
    co = 0.3 * torch.randn((case["K"], L, C, 2), generator=g, device=DEVICE)
    parts = []
    for i, shape in enumerate(scenes.rxcond_shapes(case["lmax"], C, 6, 64)):
        if i == 0:      # frequencies 2^f along each axis
            w = torch.zeros(shape, device=DEVICE)
            for a in range(3):
                for f in range(6):
                    w[6 * a + f, a] = 2.0 ** f
        elif i == 1:    # component embeddings
            w = torch.randn(shape, generator=g, device=DEVICE)
        elif len(shape) == 2:
            w = (2.0 * torch.rand(shape, generator=g, device=DEVICE) - 1.0) * math.sqrt(6.0 / sum(shape))
        else:
            w = torch.zeros(shape, device=DEVICE)
        parts.append(w.reshape(-1))
    kind = scenes.BASIS_FLE if case["basis"] == "fle" else scenes.BASIS_SH
    return scenes.RxCondModel(kind, case["lmax"], C, 6, 64, co, torch.cat(parts))


def _targets(case, g):
    grid = _grid(case)
    return 0.5 * torch.randn((case["N"], 2, grid.H, grid.W), generator=g, device=DEVICE)


SCENE = ("means", "log_scales", "quats", "logits")


def _radiance_of(p):
    return p["features"] if "features" in p else p["radiance"]


def prepare(case, seed):
    p, tx, rx, off, g = _inputs(case, seed)
    r = rxgs.Renderer(_grid(case))
    s = dict(op=case["op"], r=r, p=p, tx=tx, rx=rx, off=off, mode=case["mode"])
    if case["op"] == "rxcond":
        r.upload_scene(*[p[k] for k in SCENE])
        r.upload_rxcond(_cond_model(case, g))
    elif case["op"] in ("render", "coverage"):
        r.upload_scene(*[p[k] for k in SCENE], radiance=p.get("radiance"), features=p.get("features"))
        if "mlp" in p:
            r.upload_mlp(p["mlp"])
        if case["op"] == "coverage":
            grid = _grid(case)
            s["out"] = (torch.empty((case["N"], 2, grid.H, grid.W), device=DEVICE),
                        torch.empty((case["N"],), device=DEVICE))
    else:
        s["Y"] = _targets(case, g)
        if case["op"] == "train":
            s["saved"] = rxgs.Saved(r)
        else:
            s["leaves"] = [p[k].requires_grad_(True) for k in p]
            s["update"] = [torch.zeros_like(x) for x in s["leaves"]]
    return s


POWER_WEIGHT = 0.1   # of the received power in the autograd step's loss


def run(s):
    r, p = s["r"], s["p"]
    if s["op"] == "render":
        return r.render(s["rx"], tx=s["tx"], rx_off=s["off"], mode=s["mode"])[:2]
    if s["op"] == "rxcond":
        return r.render_rxcond(s["rx"], tx=s["tx"], rx_off=s["off"], mode=s["mode"])[:2]
    if s["op"] == "coverage":
        return r.render_chunked(s["rx"], tx=s["tx"], rx_off=s["off"], mode=s["mode"], out=s["out"])[:2]
    if s["op"] == "train":
        # a step on this step's parameters: scene in, render, L2 loss, gradients out
        r.upload_scene(*[p[k] for k in SCENE], radiance=p.get("radiance"), features=p.get("features"))
        if "mlp" in p:
            r.upload_mlp(p["mlp"])
        C, P, _ = r.render(s["rx"], tx=s["tx"], rx_off=s["off"], mode=s["mode"], saved=s["saved"])
        g = r.backward(s["saved"], C, 2.0 * (C - s["Y"]))
        return [C, P] + [g[k] for k in p]
    C, P = autograd.rx_render(r, *[p[k] for k in SCENE], _radiance_of(p), p.get("mlp"), s["rx"], tx=s["tx"],
                              mode=s["mode"], rx_off=s["off"])
    loss = (C - s["Y"]).square().sum() + POWER_WEIGHT * P.sum()
    grads = torch.autograd.grad(loss, s["leaves"])
    with torch.no_grad():
        # the optimizer's in-place update, of size zero so that every pass
        # computes the same outputs; the next step's parameters are new to the
        # renderer all the same, as in training
        torch._foreach_add_(s["leaves"], s["update"])
    return [C.detach(), P.detach(), *grads]


# In these scenes a pixel composites about this many Gaussians before its
# transmittance falls below the threshold, and a view's pixels together about
# so many different ones.
PER_PIXEL = 54
PER_VIEW = 500


def work(case):
    H, W, _ = GRIDS[case["grid"]]
    K, N, px = case["K"], case["N"], H * W
    V = case["Q"] if case["mode"] == "tx" else N
    ch = case.get("channels", 1)
    if case["op"] == "rxcond":
        L = (case["lmax"] + 1) ** 2
        radiance_in, per_pair = K * L * ch * 2, 2 * 64 * (6 + 64 + 4 * ch) + 18 * L * ch
    elif case["radiance"] == "mlp":
        radiance_in, per_pair = K * scenes.FEAT_DIM + scenes.MLP_NPARAM, 2 * 64 * (64 + 2)
    else:
        radiance_in, per_pair = K * 2, 0
    depth = min(PER_PIXEL, K // 16 + 1)
    shown = min(PER_VIEW, K)
    out = N * ch * (2 * px + 1)
    nbytes = 4 * (11 * K + radiance_in + 3 * N + out)
    # depth of every (view, Gaussian), weights of the composited pairs, one
    # complex multiply-add per output row, radiance of the composited Gaussians
    flops = 20 * V * K + depth * px * (32 * V + 4 * N * ch) + N * shown * per_pair
    if case["op"] in ("train", "autograd"):
        nbytes += 4 * (11 * K + radiance_in) + 4 * N * 2 * px
        flops += 2 * (flops - 20 * V * K)
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------------------------------
# the outputs in 64 bits

ALPHA_MIN, W_MAX, T_EPS, DILATE = 1.0 / 255.0, 0.99, 1e-4, 0.3
NEAR2 = 0.04                # squared distance (m^2) below which a Gaussian is culled
CELLS = 1 << 23             # (pixel, Gaussian) cells of one dense block
EXACT_MOST = 64_000_000     # (view, Gaussian) pairs above which it takes too long


def _depth_order(means, c):
    """Gaussians of a view, nearest first: by the 32-bit squared distance
    (each operation rounded), ties by index; near ones left out."""
    d = means - c
    key = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
    key, order = torch.sort(key, stable=True)
    return order[key >= torch.tensor(NEAR2, dtype=torch.float32, device=key.device)]


def _project(p, idx, c, grid):
    """Pixel position, inverse projected covariance and opacity of Gaussians idx."""
    m, ls, q, lg = (p[k][idx] for k in SCENE)
    d = m - c
    dx, dy, dz = d.unbind(1)
    h = torch.sqrt(dx * dx + dy * dy).clamp(min=1e-6)
    az = torch.atan2(dy, dx)
    u = torch.where(az < 0, az + 2 * math.pi, az) / grid.del_az - 0.5
    v = (torch.atan2(dz, h) - grid.el0) / grid.del_el - 0.5
    rho2 = h * h + dz * dz
    zero = torch.zeros_like(dx)
    ju = torch.stack([-dy / (h * h), dx / (h * h), zero], 1) / grid.del_az
    jv = torch.stack([-dx * dz / (rho2 * h), -dy * dz / (rho2 * h), h / rho2], 1) / grid.del_el
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    s2 = torch.exp(2 * ls)
    ru, rv = (R * ju[:, :, None]).sum(1), (R * jv[:, :, None]).sum(1)     # R^T j
    A = (ru * ru * s2).sum(1) + DILATE
    B = (ru * rv * s2).sum(1)
    D = (rv * rv * s2).sum(1) + DILATE
    det = A * D - B * B
    return u, v, D / det, -B / det, A / det, torch.sigmoid(lg), D


def _weights(geo, sel, rows, cols, W):
    """Unclamped blend weights (pixels x entries) and the pixel offsets."""
    u, v, a, b, c, o = (x[sel] for x in geo[:6])
    du = torch.remainder(cols[:, None] - u[None, :] + W / 2, W) - W / 2
    dv = rows[:, None] - v[None, :]
    w = o * torch.exp(-0.5 * (a * du * du + 2 * b * du * dv + c * dv * dv))
    return w, du, dv


def _composite(geo, radiance, nrow, grid):
    """One view's rows (pixels x nrow complex) and the entries it composites.
    geo: projected entries in depth order; radiance(sel) -> (entries, nrow, 2)."""
    H, W = grid.H, grid.W
    dev = geo[0].device
    # entries whose ellipse {w >= 1/255} reaches the grid's rows
    qmax = 2 * torch.log((geo[5] / ALPHA_MIN).clamp(min=1.0))
    rv = torch.sqrt(qmax * geo[6]) + 1e-6
    ent = torch.nonzero((geo[5] >= ALPHA_MIN) & (geo[1] + rv >= 0) & (geo[1] - rv <= H - 1)).reshape(-1)
    C = torch.zeros((H * W, nrow * 2), dtype=torch.float64, device=dev)
    px = torch.arange(H * W, device=dev)
    T = torch.ones(H * W, dtype=torch.float64, device=dev)
    used, at = [], 0
    while at < ent.numel() and px.numel():
        sel = ent[at:at + min(max(CELLS // px.numel(), 256), 1 << 15)]
        at += sel.numel()
        w, _, _ = _weights(geo, sel, (px // W).double(), (px % W).double(), W)
        w = torch.where(w >= ALPHA_MIN, w.clamp(max=W_MAX), 0.0)
        cum = torch.cumprod(1 - w, 1)
        before = torch.cat([torch.ones_like(cum[:, :1]), cum[:, :-1]], 1) * T[:, None]
        tw = torch.where(before >= T_EPS, before * w, 0.0)
        hit = torch.nonzero((tw > 0).any(0)).reshape(-1)
        if hit.numel():
            used.append(sel[hit])
            C.index_add_(0, px, tw[:, hit] @ radiance(sel[hit]).reshape(hit.numel(), -1))
        T = T * cum[:, -1]
        keep = T >= T_EPS     # (an excluded entry only lowers a product that has already stopped)
        px, T = px[keep], T[keep]
    return C, torch.cat(used) if used else ent[:0]


def _pull_back(geo, used, s, C, G, grid):
    """Gradients of sum(C . G) in one view over its used entries, by (u, v, a,
    b, c, o) and by the radiance: dL/dw_i = T_i a_i - (sum_k>i T_k w_k a_k) /
    (1 - w_i), a_i the radiance's product with the pixel's G; nothing through
    a clamped weight."""
    W = grid.W
    n = used.numel()
    out = [torch.zeros(n, dtype=torch.float64, device=s.device) for _ in range(6)]
    gs = torch.zeros((n, s.shape[1] * 2), dtype=torch.float64, device=s.device)
    sf = s.reshape(n, -1)
    _, _, ca, cb, cc, o = (x[used] for x in geo[:6])
    step = max(CELLS // max(n, 1), 1)
    for p0 in range(0, G.shape[0], step):
        px = torch.arange(p0, min(p0 + step, G.shape[0]), device=s.device)
        g = G[px]
        raw, du, dv = _weights(geo, used, (px // W).double(), (px % W).double(), W)
        w = torch.where(raw >= ALPHA_MIN, raw.clamp(max=W_MAX), 0.0)
        cum = torch.cumprod(1 - w, 1)
        before = torch.cat([torch.ones_like(cum[:, :1]), cum[:, :-1]], 1)
        tw = torch.where(before >= T_EPS, before * w, 0.0)
        a = g @ sf.T
        rest = (C[px] * g).sum(1, keepdim=True) - torch.cumsum(tw * a, 1)
        gw = torch.where(tw > 0, before * a - rest / (1 - w), 0.0)
        gs += tw.T @ g
        gw = torch.where(raw > W_MAX, 0.0, gw) * raw      # dL/dw times w
        gq = -0.5 * gw
        out[0] += (-gq * (2 * ca * du + 2 * cb * dv)).sum(0)
        out[1] += (-gq * (2 * cb * du + 2 * cc * dv)).sum(0)
        out[2] += (gq * du * du).sum(0)
        out[3] += (2 * gq * du * dv).sum(0)
        out[4] += (gq * dv * dv).sum(0)
        out[5] += (gw / o).sum(0)
    return out, gs.reshape(s.shape)


def _mlp_radiance(feat, mlp, rx):
    """Radiance (entries, receivers, 2) of the conditioning MLP."""
    W1, b1, W2, b2, W3, b3 = _unflat(mlp)
    ang = rx[:, :, None] * 2.0 ** torch.arange(6, dtype=torch.float64, device=rx.device)
    enc = torch.stack([torch.sin(ang), torch.cos(ang)], 3).reshape(rx.shape[0], -1)
    loc, glo = feat @ W1[:, 36:].T + b1, enc @ W1[:, :36].T
    out = [torch.relu(torch.relu(loc[:, None, :] + glo[None, j:j + 256, :]) @ W2.T + b2) @ W3.T + b3
           for j in range(0, rx.shape[0], 256)]
    return torch.cat(out, 1)


def _unflat(v):
    out, at = [], 0
    for shape in scenes.MLP_SHAPES:
        n = math.prod(shape)
        out.append(v[at:at + n].reshape(shape))
        at += n
    return out


def _occupancy(p, G):
    """Occupancy grid (z, y, x) and its box: 1 - prod (1 - o e^(-d^2 / 2 s^2))
    over the Gaussians within 2 s of a voxel centre."""
    m, sig = p["means"], torch.exp(p["log_scales"].max(1).values)
    o = torch.sigmoid(p["logits"])
    lo, hi = m.min(0).values, m.max(0).values
    hi = torch.where(hi - lo >= 1e-6, hi, lo + 1e-6)
    vs = (hi - lo) / G
    acc = torch.zeros(G * G * G, dtype=torch.float64, device=m.device)
    first = torch.floor((m - 2 * sig[:, None] - lo) / vs).long() - 1
    span = (torch.floor((m + 2 * sig[:, None] - lo) / vs).long() + 2 - first)
    for k in torch.split(torch.argsort(sig), 256):     # Gaussians of similar size together
        n = [int(x) for x in span[k].max(0).values]
        ix = [first[k, a][:, None] + torch.arange(n[a], device=m.device) for a in range(3)]
        d2 = [(lo[a] + (ix[a] + 0.5) * vs[a] - m[k, a][:, None]) ** 2 for a in range(3)]
        ok = [(x >= 0) & (x < G) for x in ix]
        dd = d2[2][:, :, None, None] + d2[1][:, None, :, None] + d2[0][:, None, None, :]
        s2 = (sig[k] ** 2)[:, None, None, None]
        use = ((dd <= 4 * s2) & ok[2][:, :, None, None] & ok[1][:, None, :, None] & ok[0][:, None, None, :])
        at = ((ix[2][:, :, None, None] * G + ix[1][:, None, :, None]) * G + ix[0][:, None, None, :])[use]
        val = torch.log1p(-o[k][:, None, None, None] * torch.exp(-0.5 * dd / s2))[use]
        acc.index_add_(0, at, val)
    return -torch.expm1(acc), lo, hi


def _basis(kind, lmax, d):
    """Directional basis (entries, components) as complex numbers."""
    d = d / d.norm(dim=1, keepdim=True)
    x, s, ph = d[:, 2], torch.hypot(d[:, 0], d[:, 1]), torch.atan2(d[:, 1], d[:, 0])
    P, pmm = {}, torch.ones_like(x)
    for m in range(lmax + 1):
        pmm = pmm * (2 * m - 1) * s if m else pmm
        P[m, m] = pmm
        if m < lmax:
            P[m + 1, m] = (2 * m + 1) * x * pmm
        for l in range(m + 2, lmax + 1):
            P[l, m] = ((2 * l - 1) * x * P[l - 1, m] - (l + m - 1) * P[l - 2, m]) / (l - m)
    out = []
    for l in range(lmax + 1):
        for m in range(-l, l + 1):
            a = abs(m)
            n = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - a) / math.factorial(l + a)) * P[l, a]
            if kind == scenes.BASIS_FLE:
                out.append(torch.polar(n, m * ph) if m else torch.complex(n, torch.zeros_like(n)))
            else:
                n = n if m == 0 else math.sqrt(2.0) * n * (torch.cos(a * ph) if m > 0 else torch.sin(a * ph))
                out.append(torch.complex(n, torch.zeros_like(n)))
    return torch.stack(out, 1)


class _Cond:
    """The conditioned radiance in 64 bits."""

    def __init__(self, model, p, rx):
        self.m, self.means = model, p["means"]
        dev, at, parts = rx.device, 0, []
        for shape in scenes.rxcond_shapes(model.lmax, model.C, model.F, model.H):
            n = math.prod(shape)
            parts.append(model.params[at:at + n].reshape(shape).double())
            at += n
        freq, emb, *g = parts[:8]
        self.loc = parts[8:]
        ang = rx @ freq.T
        gam = torch.stack([torch.sin(ang), torch.cos(ang)], 2).reshape(rx.shape[0], -1)
        dn = max(model.lmax, 1)
        lm = torch.tensor([[l / dn, m / dn] for l in range(model.lmax + 1) for m in range(-l, l + 1)],
                          dtype=torch.float64, device=dev)
        x = torch.cat([gam[:, None, :].expand(-1, model.L, -1),
                       torch.cat([lm, emb], 1)[None].expand(rx.shape[0], -1, -1)], 2)
        self.glob = self._mlp(x, g).reshape(rx.shape[0], model.L, model.C, 4)
        self.occ, self.lo, self.hi = _occupancy(p, model.G)

    @staticmethod
    def _mlp(x, w):
        return torch.relu(torch.relu(x @ w[0].T + w[1]) @ w[2].T + w[3]) @ w[4].T + w[5]

    def __call__(self, idx, rx, js, centre):
        """Radiance (entries, receivers x channels, 2) of Gaussians idx for receivers js."""
        m, G = self.m, self.m.G
        p, r = self.means[idx][:, None, :], rx[js][None, :, :]
        t = 0.05 + (0.9 * torch.arange(m.S, dtype=torch.float64, device=rx.device)) / (m.S - 1)
        q = p[:, :, None, :] + t[:, None] * (r - p)[:, :, None, :]
        cell = torch.floor((q - self.lo) * (G / (self.hi - self.lo)))
        ok = ((cell >= 0) & (cell <= G - 1)).all(3)
        cell = cell.clamp(0, G - 1).long()
        V = torch.where(ok, self.occ[(cell[..., 2] * G + cell[..., 1]) * G + cell[..., 0]], 0.0)
        d = (r - p).norm(dim=2, keepdim=True)
        f = torch.cat([(r - p) / d.clamp(min=1e-300), d, (1 - V).prod(2, keepdim=True), V.mean(2, keepdim=True)], 2)
        ab = self._mlp(f, self.loc).reshape(*f.shape[:2], m.C, 4)
        B = _basis(m.kind, m.lmax, self.means[idx] - centre)
        co = torch.view_as_complex(m.coeffs[idx].double())                         # E, L, C
        ga = torch.complex(1 + self.glob[js][..., 0], self.glob[js][..., 1])       # J, L, C
        gb = torch.complex(self.glob[js][..., 2], self.glob[js][..., 3])
        phi = ga[None] * co[:, None] + gb[None]
        s = (torch.complex(1 + ab[..., 0], ab[..., 1]) * (phi * B[:, None, :, None]).sum(2)
             + torch.complex(ab[..., 2], ab[..., 3]) * B.sum(1)[:, None, None])
        return torch.view_as_real(s).reshape(idx.numel(), -1, 2)


def exact(case, seed):
    V = case["Q"] if case["mode"] == "tx" else case["N"]
    if V * case["K"] > EXACT_MOST:
        return None
    p32, tx, rx32, off, g = _inputs(case, seed)
    grid = _grid(case)
    train = case["op"] in ("train", "autograd")
    cond = _Cond(_cond_model(case, g), {k: x.double() for k, x in p32.items()}, rx32.double()) \
        if case["op"] == "rxcond" else None
    Y = _targets(case, g).double() if train else None
    p = {k: x.double() for k, x in p32.items()}
    rx, ch, px = rx32.double(), case.get("channels", 1), grid.H * grid.W
    C = torch.zeros((case["N"], ch * 2, px), dtype=torch.float64, device=rx.device)
    grads = {k: torch.zeros_like(x) for k, x in p.items()}
    for v in range(V):
        js = torch.arange(off[v], off[v + 1], device=rx.device) if off else torch.tensor([v], device=rx.device)
        if not js.numel():
            continue
        c32 = tx[v] if off else rx32[v]
        c = c32.double()
        order = _depth_order(p32["means"], c32)
        with torch.no_grad():
            geo = _project(p, order, c, grid)

        def radiance(sel, q=p):
            i = order[sel]
            if cond is not None:
                return torch.cat([cond(e, rx, js, c) for e in torch.split(i, max(1, (1 << 23) // (js.numel() * 16 * 7
                                  + js.numel() * cond.m.L * ch * 4)))], 0)
            if "mlp" in q:
                return _mlp_radiance(q["features"][i], q["mlp"], rx[js])
            return q["radiance"][i][:, None, :].expand(-1, js.numel(), -1)

        Cv, used = _composite(geo, radiance, js.numel() * ch, grid)
        C[js] = Cv.reshape(px, js.numel(), ch * 2).permute(1, 2, 0)
        if train:
            G = 2 * (C[js] - Y[js].reshape(js.numel(), 2, px))
            if case["op"] == "autograd":
                G = G + POWER_WEIGHT * 2 * C[js]
            G = G.permute(2, 0, 1).reshape(px, -1)
            leaf = {k: (x if k == "mlp" else x[order[used]]).detach().requires_grad_(True) for k, x in p.items()}
            here = torch.arange(used.numel(), device=rx.device)
            proj = _project(leaf, here, c, grid)
            s = _mlp_radiance(leaf["features"], leaf["mlp"], rx[js]) if "mlp" in leaf else \
                leaf["radiance"][:, None, :].expand(-1, js.numel(), -1)
            gg, gs = _pull_back(geo, used, s.detach(), Cv, G, grid)
            got = torch.autograd.grad([*proj[:6], s], list(leaf.values()), [*gg, gs])
            for k, x in zip(leaf, got):
                if k == "mlp":
                    grads[k] += x
                else:
                    grads[k].index_add_(0, order[used], x)
    P = C.reshape(case["N"], ch, -1).square().sum(2)
    if case["op"] == "rxcond":
        return [C.reshape(case["N"], ch, 2, grid.H, grid.W), P]
    out = [C.reshape(case["N"], 2, grid.H, grid.W), P.reshape(-1)]
    return out + [grads[k] for k in p] if train else out
