"""Timed cases of the library: stereo frames, batches, the serving runtime and
the differentiable head, through the package's public entry points.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs and handles a program holds before the call
    run(state)           one pass; returns its outputs
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    float outputs in 64 bits (plain torch)

A case is a dict of plain values.  ``kind`` says which entry point it times:

    frame       Stereo.disparity, one pair
    noalloc     Stereo.disparity_noalloc, one pair
    batch       Stereo.disparity_batch, n pairs of one shape
    serve       Server.submit / poll, a burst of frames of mixed shapes
    soft        soft_disparity without gradients, n float pairs
    train       soft_disparity + l1_loss + gradients
    head        soft_disparity inside a larger network: gradients of d_hat
                given by what follows it

Images follow the recipe of ``paper_2212_00488_amd/synth.py`` (planar Voronoi
disparity segments, coloured regions, noise, z-buffered forward warp), drawn
on the GPU.
"""

from __future__ import annotations

import torch

from paper_2212_00488_amd import Stereo
from paper_2212_00488_amd.binding import F_FULL_RES, default_params
from paper_2212_00488_amd.serve import Server
from paper_2212_00488_amd.soft import l1_loss, soft_disparity

DEV = "cuda:0"

# learnable weights of the head: lambda_AD, lambda_census
LAMBDAS = (10.0, 30.0)

# frames of one burst of the serving case: the shapes of the served stream
SERVED = ((640, 480, 64), (1436, 992, 145), (640, 480, 64), (1920, 1080, 256),
          (1436, 992, 145), (640, 480, 64), (1436, 992, 145), (1920, 1080, 256))


def _case(kind, W, H, dmax, n=1, **options):
    c = dict(kind=kind, W=W, H=H, dmax=dmax, n=n, arm_x=21, arm_y=31, arm_x_r=-1, fill_mode=0,
             cost_scale=1024, full_res=False)
    c.update(options)
    return c


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # the smallest frame of the test workloads: one robot or drone camera,
        # where launches and latency count
        named("frame_320x240_d32", "frame", 320, 240, 32),
        # a serving loop that forbids allocation, on VGA frames
        named("noalloc_640x480_d64", "noalloc", 640, 480, 64),
        # a cropped, rectified camera image: odd sides, an odd range, the
        # simpler fill and a separate cap for the right image
        named("frame_1237x823_d121", "frame", 1237, 823, 121, fill_mode=1, arm_x_r=15),
        # the size and range the paper times
        named("frame_1436x992_d145", "frame", 1436, 992, 145),
        # the largest served frame
        named("frame_2872x1984_d290", "frame", 2872, 1984, 290),
        # the method on the original images, with the caps the paper uses there
        named("fullres_1436x992_d145", "frame", 1436, 992, 145, arm_x=41, arm_y=61,
              cost_scale=512, full_res=True),
        # eight full-HD cameras or frames in one launch sequence
        named("batch8_1920x1080_d256", "batch", 1920, 1080, 256, n=8),
        # a burst of host frames of mixed shapes through the serving runtime,
        # copies in and out included
        named("serve_burst_8", "serve", 1920, 1080, 256, n=8),
        # inference with the soft-argmin head on a VGA pair
        named("soft_640x480_d64", "soft", 640, 480, 64),
        # training step on one small crop
        named("train_320x240_d32", "train", 320, 240, 32),
        # training step of four pairs at the paper's size
        named("train_4x1436x992_d145", "train", 1436, 992, 145, n=4),
        # the head inside a larger network, four full-HD pairs
        named("head_4x1920x1080_d256", "head", 1920, 1080, 256, n=4),
    ]


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "noalloc", "fullres", "batch", "soft", "train",
                       "train", "head"])
    most = {"frame": 2872 * 1984 * 290, "noalloc": 1436 * 992 * 145, "fullres": 1436 * 992 * 145,
            "batch": 8 * 1920 * 1080 * 256}.get(kind, 4 * 1436 * 992 * 145)
    widest = {"frame": 2872, "batch": 1920, "fullres": 1436, "noalloc": 1436}.get(kind, 1920)
    n = 1
    if kind == "batch":
        n = rng.randint(2, 8)
    elif kind in ("soft", "train", "head"):
        n = rng.randint(1, 4)
    while True:
        W = int(round(320 * (widest / 320) ** rng.random()))
        H = max(200, int(round(W * rng.uniform(0.5, 0.8))))
        # the key of a full-resolution aggregate leaves 8 bits for the disparity
        dmax = min(256 if kind == "fullres" else 290, max(16, int(round(W / rng.uniform(5, 12)))))
        if n * W * H * dmax <= most:
            break
    opt = {}
    if kind == "fullres":
        opt = dict(full_res=True, cost_scale=512, arm_x=41, arm_y=61)
    elif kind in ("frame", "noalloc", "batch"):
        opt["fill_mode"] = rng.choice([0, 0, 0, 1, 2])
        if rng.random() < 0.2:
            opt["arm_x_r"] = rng.randint(11, 21)
        if rng.random() < 0.2:  # the sweep of the caps
            opt.update(arm_x=rng.choice([11, 31, 41]), arm_y=rng.choice([21, 41, 61]),
                       cost_scale=512)
    return _case("frame" if kind == "fullres" else kind, W, H, dmax, n, **opt)


# ------------------------------------------------------------------ inputs
def _nearest(points, W, H):
    """Index of the nearest of [K][2] points for every pixel centre."""
    xs = torch.arange(W, device=DEV, dtype=torch.float32) + 0.5
    out = torch.empty((H, W), dtype=torch.int64, device=DEV)
    dx = (xs[:, None] - points[None, :, 0]) ** 2
    for y in range(0, H, 128):
        ys = torch.arange(y, min(H, y + 128), device=DEV, dtype=torch.float32) + 0.5
        dy = (ys[:, None] - points[None, :, 1]) ** 2
        out[y:y + 128] = (dx[None] + dy[:, None]).argmin(dim=2)
    return out


def _pair(W, H, dmax, gen):
    """left, right uint8 [H][W][3], gt int16 [H][W], nonocc uint8 [H][W]."""
    def uniform(lo, hi, *shape):
        return torch.rand(*shape, device=DEV, generator=gen) * (hi - lo) + lo

    K = 6 if W * H < 300000 else 40
    size = torch.tensor([W, H], device=DEV, dtype=torch.float32)
    seg_pts, col_pts = uniform(0, 1, K, 2) * size, uniform(0, 1, 4 * K, 2) * size
    c0, slope = uniform(0, dmax - 1, K), uniform(-0.15, 0.15, K, 2)
    slope[0::2] = 0.0
    seg, cell = _nearest(seg_pts, W, H), _nearest(col_pts, W, H)
    ys = torch.arange(H, device=DEV, dtype=torch.float32)[:, None]
    xs = torch.arange(W, device=DEV, dtype=torch.float32)[None, :]
    d = c0[seg] + slope[seg, 0] * (xs - seg_pts[seg, 0]) + slope[seg, 1] * (ys - seg_pts[seg, 1])
    gt = d.round().clamp(0, dmax - 1).to(torch.int64)
    region = seg * (4 * K) + cell
    mean = uniform(0, 255, 4 * K * K, 3)
    grad = uniform(-0.5, 0.5, 4 * K * K, 2, 3)
    flat = uniform(0, 1, 4 * K * K) < 0.1
    grad[flat] = 0.0
    sigma = torch.where(flat, 0.5, 2.0)
    img = (mean[region] + grad[region, 0] * (xs - col_pts[cell, 0])[..., None]
           + grad[region, 1] * (ys - col_pts[cell, 1])[..., None])
    img = img + torch.randn(H, W, 3, device=DEV, generator=gen) * sigma[region][..., None]
    left = img.round().clamp(0, 255).to(torch.uint8)
    # forward warp: the larger disparity, then the larger x, wins a target
    xi = torch.arange(W, device=DEV)[None, :].expand(H, W)
    yi = torch.arange(H, device=DEV)[:, None].expand(H, W)
    tx = xi - gt
    ok = tx >= 0
    key = torch.full((H * W,), -1, dtype=torch.int64, device=DEV)
    src = gt * W + xi
    key.scatter_reduce_(0, (yi * W + tx)[ok], src[ok], "amax")
    right = torch.randint(0, 256, (H * W, 3), device=DEV, generator=gen).to(torch.uint8)
    hit = key >= 0
    rows = yi.reshape(-1)[hit]
    right[hit] = left[rows, key[hit] % W]
    nonocc = torch.zeros((H, W), dtype=torch.uint8, device=DEV)
    nonocc[ok] = (key[(yi * W + tx)[ok]] == src[ok]).to(torch.uint8)
    return left, right.view(H, W, 3), gt.to(torch.int16), nonocc


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _float_pairs(case, seed):
    """Float batches left, right [n][H][W][3] in [0, 1], gt, nonocc, and an
    upstream gradient of d_hat."""
    gen = _generator(seed)
    W, H, n = case["W"], case["H"], case["n"]
    pairs = [_pair(W, H, case["dmax"], gen) for _ in range(n)]

    def image(k):
        v = torch.stack([p[k] for p in pairs]).float().div_(255.0)
        # no two intensities tie exactly
        v += (torch.rand(v.shape, device=DEV, generator=gen) - 0.5) * 0.004
        return v.clamp_(0.0, 1.0)

    left, right = image(0), image(1)
    gt, nonocc = (torch.stack([p[k] for p in pairs]).contiguous() for k in (2, 3))
    X, Y = (W + 1) // 2, (H + 1) // 2
    g_dhat = torch.randn(n, Y, X, device=DEV, generator=gen) / (n * X * Y)
    return left, right, gt, nonocc, g_dhat


_kept = {}


def _context():
    """The program's library context: made once, scratch cached inside."""
    if "ctx" not in _kept:
        _kept["ctx"] = Stereo(0)
    return _kept["ctx"]


def _server():
    if "server" not in _kept:
        _kept["server"] = Server(0)
    return _kept["server"]


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, kind=kind)
    if kind in ("soft", "train", "head"):
        left, right, gt, nonocc, g_dhat = _float_pairs(case, seed)
        lam = torch.tensor(LAMBDAS, dtype=torch.float32, device=DEV)
        if kind != "soft":
            for t in (left, right, lam):
                t.requires_grad_(True)
        st.update(ctx=_context(), left=left, right=right, lam=lam, gt=gt, nonocc=nonocc,
                  g_dhat=g_dhat)
        return st
    gen = _generator(seed)
    if kind == "serve":
        frames = []
        for W, H, dmax in SERVED:
            left, right, _, _ = _pair(W, H, dmax, gen)
            host = [torch.empty((H, W, 3), dtype=torch.uint8, pin_memory=True) for _ in range(2)]
            host[0].copy_(left)
            host[1].copy_(right)
            out = torch.empty((H, W), dtype=torch.int16, pin_memory=True)
            frames.append((host[0].numpy(), host[1].numpy(), dmax, out.numpy(), host, out))
        st.update(server=_server(), frames=frames)
        return st
    pairs = [_pair(case["W"], case["H"], case["dmax"], gen)[:2] for _ in range(case["n"])]
    st.update(ctx=_context(), lefts=[p[0].contiguous() for p in pairs],
              rights=[p[1].contiguous() for p in pairs])
    st["params"] = default_params(arm_x=case["arm_x"], arm_y=case["arm_y"],
                                  arm_x_r=case["arm_x_r"], fill_mode=case["fill_mode"],
                                  cost_scale=case["cost_scale"],
                                  flags=F_FULL_RES if case["full_res"] else 0)
    st["outs"] = [torch.empty((case["H"], case["W"]), dtype=torch.int16, device=DEV)
                  for _ in pairs]
    return st


# ------------------------------------------------------------------- calls
def run(st):
    kind, dmax = st["kind"], st["case"]["dmax"]
    if kind == "frame":
        return st["ctx"].disparity(st["lefts"][0], st["rights"][0], dmax, st["params"],
                                   out=st["outs"][0])
    if kind == "noalloc":
        return st["ctx"].disparity_noalloc(st["lefts"][0], st["rights"][0], dmax, st["params"],
                                           out=st["outs"][0])
    if kind == "batch":
        return st["ctx"].disparity_batch(st["lefts"], st["rights"], dmax, st["params"],
                                         outs=st["outs"])
    if kind == "serve":
        srv, left = st["server"], len(st["frames"])
        for i, (l, r, d, out, _, _) in enumerate(st["frames"]):
            srv.submit(l, r, d, out, i)
        while left:
            for res in srv.poll(64, 100):
                if res["status"]:
                    raise RuntimeError("serve: " + srv.last_error())
                left -= 1
        return [f[3] for f in st["frames"]]
    if kind == "soft":
        with torch.no_grad():
            return soft_disparity(st["ctx"], st["left"], st["right"], st["lam"], dmax)
    inputs = (st["left"], st["right"], st["lam"])
    d_hat = soft_disparity(st["ctx"], *inputs, dmax)
    if kind == "head":
        grads = torch.autograd.grad(d_hat, inputs, st["g_dhat"])
        return dict(d_hat=d_hat.detach(), g_left=grads[0], g_right=grads[1], g_lambdas=grads[2])
    loss = l1_loss(st["ctx"], d_hat, st["gt"], st["nonocc"])
    grads = torch.autograd.grad(loss, inputs)
    return dict(d_hat=d_hat.detach(), loss=loss.detach(), g_left=grads[0], g_right=grads[1],
                g_lambdas=grads[2])


# -------------------------------------------------------------------- work
def work(case):
    """Images in, maps (and gradients) out, each once; operations counted per
    evaluation (x, y, d) of the searched range: 40 for both bases of the
    integer path (cost, two window sums, minimum), 25 for the head's forward
    and 35 more for its adjoint."""
    kind = case["kind"]
    shapes = SERVED if kind == "serve" else [(case["W"], case["H"], case["dmax"])] * case["n"]
    nbytes = flops = 0
    for W, H, dmax in shapes:
        if case["full_res"]:
            X, Y, D = W, H, dmax
        else:
            X, Y, D = (W + 1) // 2, (H + 1) // 2, (dmax + 1) // 2
        if kind in ("soft", "train", "head"):
            nbytes += 2 * W * H * 12 + X * Y * 4
            flops += X * Y * D * 25
            if kind != "soft":
                nbytes += 2 * W * H * 12 + (X * Y * 4 if kind == "head" else X * Y * 3)
                flops += X * Y * D * 35
        else:
            nbytes += 2 * W * H * 3 + W * H * 2
            flops += X * Y * D * 40
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------- the head in 64 bits
def _half(v, H, W):
    """3x3 sums at (2x, 2y), borders clamped, of a [H][W] plane."""
    Y, X = (H + 1) // 2, (W + 1) // 2
    ys, xs = torch.arange(Y, device=DEV) * 2, torch.arange(X, device=DEV) * 2
    out = 0
    for j in (-1, 0, 1):
        rows = v[(ys + j).clamp(0, H - 1)]
        for i in (-1, 0, 1):
            out = out + rows[:, (xs + i).clamp(0, W - 1)]
    return out


def _integer_half(rgb, H, W):
    q = torch.floor(rgb * 255.0 + 0.5).clamp(0, 255).to(torch.int64)  # float32 steps
    g = (77 * q[..., 0] + 150 * q[..., 1] + 29 * q[..., 2] + 128) >> 8
    return (_half(g, H, W) + 4) // 9


def _census(h):
    Y, X = h.shape
    ys, xs = torch.arange(Y, device=DEV), torch.arange(X, device=DEV)
    out = torch.zeros_like(h)
    for k, (i, j) in enumerate(((-1, -1), (1, -1), (-2, 0), (2, 0), (-1, 1), (1, 1))):
        nb = h[(ys + j).clamp(0, Y - 1)][:, (xs + i).clamp(0, X - 1)]
        out |= (nb < h).to(torch.int64) << k
    return out


def _arm(h, axis, sign, cap, delta=13):
    n = h.shape[axis]
    pos = torch.arange(n, device=DEV)
    pos = pos[:, None] if axis == 0 else pos[None, :]
    alive, length = torch.ones_like(h, dtype=torch.bool), torch.zeros_like(h)
    for t in range(1, cap + 1):
        inside = (pos + sign * t >= 0) & (pos + sign * t < n)
        alive = alive & inside & ((torch.roll(h, -sign * t, axis) - h).abs() < delta)
        length += alive.to(torch.int64)
    return length


def _window(v, lo, hi, axis):
    """Sums of v[d] over [pos - lo, pos + hi] along axis (1: y, 2: x)."""
    P = torch.nn.functional.pad(v.cumsum(axis), (1, 0) if axis == 2 else (0, 0, 1, 0))
    n = v.shape[axis]
    pos = torch.arange(n, device=DEV)
    pos = pos[:, None] if axis == 1 else pos[None, :]
    a = (pos + hi + 1).expand(lo.shape)[None].expand(v.shape[0], -1, -1)
    b = (pos - lo).expand(lo.shape)[None].expand(v.shape[0], -1, -1)
    return P.gather(axis, a) - P.gather(axis, b)


def _soft64(left, right, lam, dmax, H, W, feats, tau=0.1):
    """d_hat [Y][X] of one pair, float64."""
    cl, cr, m, n, M, N = feats
    wgt = torch.tensor([77.0, 150.0, 29.0], dtype=torch.float64, device=DEV) / 256.0
    hl, hr = (_half((v * wgt).sum(-1), H, W) / 9.0 for v in (left, right))
    Y, X = hl.shape
    D = (dmax + 1) // 2
    xs = torch.arange(X, device=DEV)
    planes = []
    for d in range(D):
        src = (xs - d).clamp(min=0)
        bits = cl ^ cr[:, src]
        ham = sum((bits >> k) & 1 for k in range(6)).to(torch.float64)
        c = (1 - torch.exp(-255.0 * (hl - hr[:, src]).abs() / lam[0])) + (1 - torch.exp(-ham / lam[1]))
        planes.append(torch.where(xs[None, :] >= d, c, torch.full_like(c, 2.0)))
    ca = _window(_window(torch.stack(planes), m, n, 2), M, N, 1)
    ones = torch.ones(1, Y, X, dtype=torch.float64, device=DEV)
    area = _window(_window(ones, m, n, 2), M, N, 1)
    p = torch.softmax(-(ca / area) / tau, dim=0)
    return (p * torch.arange(D, dtype=torch.float64, device=DEV)[:, None, None]).sum(0)


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("soft", "train", "head"):
        return None  # whole numbers
    W, H, n = case["W"], case["H"], case["n"]
    left, right, gt, nonocc, g_dhat = _float_pairs(case, seed)
    grad = kind != "soft"
    lam = torch.tensor(LAMBDAS, dtype=torch.float64, device=DEV, requires_grad=grad)
    d_hat, g_left, g_right, loss = [], [], [], 0.0
    g_lam = torch.zeros(2, dtype=torch.float64, device=DEV)
    for i in range(n):  # one pair at a time: its volumes are freed before the next
        hl, hr = _integer_half(left[i], H, W), _integer_half(right[i], H, W)
        feats = (_census(hl), _census(hr), _arm(hl, 1, -1, 21), _arm(hl, 1, 1, 21),
                 _arm(hl, 0, -1, 31), _arm(hl, 0, 1, 31))
        l, r = (t[i].double().requires_grad_(grad) for t in (left, right))
        with torch.set_grad_enabled(grad):
            d = _soft64(l, r, lam, case["dmax"], H, W, feats)
            if kind == "train":
                diff = (2.0 * d - gt[i, ::2, ::2].double()).abs()
                mask = nonocc[i, ::2, ::2] != 0
                one = diff[mask].sum() / max(int(mask.sum()), 1) / n
            elif kind == "head":
                one = (d * g_dhat[i].double()).sum()
        d_hat.append(d.detach())
        if grad:
            gl, gr, gk = torch.autograd.grad(one, (l, r, lam))
            loss += one.detach()
            g_lam += gk
            g_left.append(gl)
            g_right.append(gr)
    d_hat = torch.stack(d_hat)
    if not grad:
        return d_hat
    out = dict(d_hat=d_hat, g_left=torch.stack(g_left), g_right=torch.stack(g_right),
               g_lambdas=g_lam)
    if kind == "train":
        out["loss"] = loss.reshape(1)
    return out
