"""GPU parity of the soft-argmin head against the FP64 oracle (oracle/soft.py).

Tolerances follow from the kernel's arithmetic: costs enter the aggregate in
fixed point with 2^-19 resolution (k = 18 for the default arms), so the mean
cost is within 2^-19 of the exact one and a logit (mean / tau) within
2e-5; the rest is float32 (relative 1e-6 per operation).  d_hat is compared
to 1e-3 absolute, the loss to 1e-4 relative and every gradient to 1e-3
relative to its largest magnitude (and in norm).
"""

import numpy as np
import pytest
import torch

from oracle import soft as osoft
from paper_2212_00488_amd import Stereo
from paper_2212_00488_amd.binding import soft_default_params
from paper_2212_00488_amd.soft import l1_loss, soft_disparity
from paper_2212_00488_amd.synth import make_pair

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    c = Stereo(0)
    yield c
    c.close()


def float_pairs(n, W, H, dmax, seed, noise=0.0):
    """n synthetic pairs as float32 [0,1] images (plus GT and mask); noise
    adds small uniform jitter so that no two intensities tie exactly."""
    rng = np.random.default_rng(seed)
    L, R, G, M = [], [], [], []
    for i in range(n):
        p = make_pair(W, H, dmax, segments=4, seed=seed + i)
        l = p.left.astype(np.float32) / np.float32(255.0)
        r = p.right.astype(np.float32) / np.float32(255.0)
        if noise:
            l = np.clip(l + rng.uniform(-noise, noise, l.shape).astype(np.float32), 0, 1)
            r = np.clip(r + rng.uniform(-noise, noise, r.shape).astype(np.float32), 0, 1)
        L.append(l.astype(np.float32))
        R.append(r.astype(np.float32))
        G.append(p.gt)
        M.append(p.nonocc)
    return np.stack(L), np.stack(R), np.stack(G), np.stack(M)


def to_dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return t.to(dtype) if dtype is not None else t


def sp_from(p: osoft.SoftParams, slab=0):
    return soft_default_params(tau=p.tau, color_delta=p.color_delta, arm_x=p.arm_x,
                               arm_y=p.arm_y, slab=slab)


def run_gpu(ctx, L, R, G, M, dmax, p, lam=None, slab=0):
    lam = lam if lam is not None else (p.lambda_ad, p.lambda_census)
    left = to_dev(L).requires_grad_(True)
    right = to_dev(R).requires_grad_(True)
    lambdas = torch.tensor(lam, dtype=torch.float32, device=DEV, requires_grad=True)
    d_hat = soft_disparity(ctx, left, right, lambdas, dmax, sp_from(p, slab))
    loss = l1_loss(ctx, d_hat, to_dev(G.astype(np.int16)), to_dev(M.astype(np.uint8)))
    loss.backward()
    torch.cuda.synchronize()
    return (d_hat.detach().cpu().numpy(), float(loss.detach().cpu()[0]),
            left.grad.cpu().numpy(), right.grad.cpu().numpy(), lambdas.grad.cpu().numpy())


def oracle_dhat(L, R, dmax, p):
    out = []
    for i in range(len(L)):
        r = osoft.forward(torch.tensor(L[i], dtype=torch.float64),
                          torch.tensor(R[i], dtype=torch.float64), dmax,
                          torch.tensor(p.lambda_ad, dtype=torch.float64),
                          torch.tensor(p.lambda_census, dtype=torch.float64), p)
        out.append(r["d_hat"].numpy())
    return np.stack(out)


def assert_grad_close(g, r, name, rel=1e-3, floor=1e-2, rel_elem=5e-3):
    """Max error within rel of the largest reference magnitude, the norm of
    the error within rel of the reference's norm, and every entry whose
    reference magnitude is at least floor x the largest within rel_elem of
    itself (the per-entry check sees errors on smaller entries that the
    first two hide)."""
    scale = float(np.abs(r).max())
    assert scale > 0, name
    err = float(np.abs(g - r).max())
    assert err <= rel * scale, f"{name}: max err {err:.3e} vs {rel} x {scale:.3e}"
    nerr = float(np.linalg.norm((g - r).ravel()) / np.linalg.norm(r.ravel()))
    assert nerr <= rel, f"{name}: norm rel err {nerr:.3e}"
    big = np.abs(r) >= floor * scale
    eel = float((np.abs(g - r)[big] / np.abs(r)[big]).max())
    print(f"[grad] {name}: max err {err / scale:.2e} of max, worst entry above "
          f"{floor:g} x max {eel:.2e} relative ({int(big.sum())} entries)", flush=True)
    assert eel <= rel_elem, f"{name}: entry rel err {eel:.3e} above {floor} x max"


@pytest.mark.parametrize("case", [
    dict(W=64, H=48, dmax=32, n=2, seed=500),          # the FD configuration (D = 16)
    # the same with the adjoint in slabs of 3 and of 5 disparities (6 and 4
    # slabs, the last ones short): slab offsets and per-slab lambda partials
    dict(W=64, H=48, dmax=32, n=2, seed=500, slab=3),
    dict(W=64, H=48, dmax=32, n=2, seed=500, slab=5),
    dict(W=67, H=41, dmax=20, n=1, seed=510),          # odd sizes, ragged strip and band
    dict(W=67, H=41, dmax=20, n=1, seed=510, slab=4),
    dict(W=150, H=30, dmax=40, n=3, seed=520),         # three strips
])
def test_forward_loss_and_gradients_match_oracle(ctx, case):
    W, H, dmax, n, seed = case["W"], case["H"], case["dmax"], case["n"], case["seed"]
    L, R, G, M = float_pairs(n, W, H, dmax, seed, noise=0.002)
    p = osoft.SoftParams()
    print(f"[soft] {W}x{H} Dmax={dmax} n={n} slab={case.get('slab', 0)}", flush=True)
    d_hat, loss, gl, gr, glam = run_gpu(ctx, L, R, G, M, dmax, p, slab=case.get("slab", 0))
    ref = oracle_dhat(L, R, dmax, p)
    assert np.all(np.isfinite(d_hat))
    assert float(np.abs(d_hat - ref).max()) <= 1e-3
    rloss, rgl, rgr, rglam = osoft.loss_and_grads(list(L), list(R), list(G), list(M), dmax, p)
    assert abs(loss - rloss) <= 1e-4 * abs(rloss)
    assert_grad_close(gl, rgl, "g_left")
    assert_grad_close(gr, rgr, "g_right")
    for k in range(2):
        assert abs(glam[k] - rglam[k]) <= 1e-3 * abs(rglam[k]), (k, glam, rglam)


def test_arm_and_temperature_variants_match_oracle(ctx):
    L, R, G, M = float_pairs(1, 70, 36, 24, 530, noise=0.002)
    for p in (osoft.SoftParams(tau=0.3, arm_x=5, arm_y=4, color_delta=30),
              osoft.SoftParams(tau=0.05, arm_x=31, arm_y=63),
              osoft.SoftParams(arm_x=0, arm_y=0)):
        d_hat, loss, gl, gr, glam = run_gpu(ctx, L, R, G, M, 24, p)
        ref = oracle_dhat(L, R, 24, p)
        assert float(np.abs(d_hat - ref).max()) <= 1e-3, p
        rloss, rgl, rgr, rglam = osoft.loss_and_grads(list(L), list(R), list(G), list(M), 24, p)
        assert_grad_close(gl, rgl, f"g_left {p}")
        assert_grad_close(gr, rgr, f"g_right {p}")
        for k in range(2):
            assert abs(glam[k] - rglam[k]) <= 1e-3 * abs(rglam[k]) + 1e-9, (p, k, glam, rglam)


def test_lambda_gradient_matches_gpu_central_differences(ctx):
    """Central differences of the GPU forward itself for both lambdas, a
    coarse check of the adjoint on the kernels alone (the 1e-3 checks above
    compare against the FP64 reference gradient, itself pinned by float64
    central differences).  The differenced function is a fixed random linear
    functional of d_hat (the L1 loss has kinks a finite step crosses), summed
    in float64 on the host; its gradient comes from the adjoint with g_dhat =
    the weights.  The float32 forward with fixed-point costs carries about
    1e-5 of noise per d_hat, about 4e-4 in the functional, so a step of 1e-2
    lambda leaves about 1% of noise and truncation: tolerance 1.5e-2 (the
    check against the FP64 reference gradient above is the 1e-3 one)."""
    L, R, G, M = float_pairs(2, 64, 48, 32, 540, noise=0.002)
    p = osoft.SoftParams()
    w = np.random.default_rng(541).standard_normal((2, 24, 32)).astype(np.float32)
    left, right = to_dev(L), to_dev(R)
    lam = torch.tensor([p.lambda_ad, p.lambda_census], dtype=torch.float32, device=DEV,
                       requires_grad=True)
    d = soft_disparity(ctx, left, right, lam, 32, sp_from(p))
    (d * to_dev(w)).sum().backward()
    glam = lam.grad.cpu().numpy()
    base = np.array([p.lambda_ad, p.lambda_census])

    def f(lv):
        with torch.no_grad():
            lt = torch.tensor(lv, dtype=torch.float32, device=DEV)
            dh = soft_disparity(ctx, left, right, lt, 32, sp_from(p)).cpu().numpy()
        return float(np.sum(dh.astype(np.float64) * w))

    for k in range(2):
        e = np.zeros(2)
        e[k] = 1e-2 * base[k]
        fd = (f(base + e) - f(base - e)) / (2 * e[k])
        assert abs(fd - glam[k]) <= 1.5e-2 * abs(glam[k]) + 1e-6, (k, fd, glam[k])


def test_backward_is_deterministic_and_batch_matches_single(ctx):
    L, R, G, M = float_pairs(3, 96, 40, 30, 550, noise=0.002)
    p = osoft.SoftParams()
    a = run_gpu(ctx, L, R, G, M, 30, p)
    for rep in range(9):  # ten runs in all, the same bits each time
        b = run_gpu(ctx, L, R, G, M, 30, p)
        for u, v in zip(a, b):
            assert np.array_equal(np.asarray(u), np.asarray(v)), rep
    # pair 1 alone: same d_hat (chunk sums may group differently) and, with the
    # loss of one pair instead of the mean of three, 3x the image gradients
    s = run_gpu(ctx, L[1:2], R[1:2], G[1:2], M[1:2], 30, p)
    assert float(np.abs(s[0][0] - a[0][1]).max()) <= 1e-5
    assert_grad_close(s[2][0], 3.0 * a[2][1], "single vs batch g_left", rel=1e-4)


def launch_step(ctx, L, R, G, M, dmax, p):
    """Forward + loss + backward enqueued on the current stream, no wait."""
    left = to_dev(L).requires_grad_(True)
    right = to_dev(R).requires_grad_(True)
    lambdas = torch.tensor((p.lambda_ad, p.lambda_census), dtype=torch.float32, device=DEV,
                           requires_grad=True)
    d_hat = soft_disparity(ctx, left, right, lambdas, dmax, sp_from(p))
    loss = l1_loss(ctx, d_hat, to_dev(G.astype(np.int16)), to_dev(M.astype(np.uint8)))
    loss.backward()
    return d_hat, loss, left, right, lambdas


def test_ten_training_steps_bit_identical_at_paper_size(ctx):
    """4 x 1436x992, Dmax = 145: ten forward + loss + backward steps (the
    saved-weights path) give the same d_hat, loss and gradients bit for bit."""
    L, R, G, M = float_pairs(4, 1436, 992, 145, 400)
    p = osoft.SoftParams()
    first = None
    for rep in range(10):
        d_hat, loss, left, right, lam = launch_step(ctx, L, R, G, M, 145, p)
        torch.cuda.synchronize()
        got = (d_hat.detach().cpu().numpy(), loss.detach().cpu().numpy(),
               left.grad.cpu().numpy(), right.grad.cpu().numpy(), lam.grad.cpu().numpy())
        if first is None:
            first = got
            continue
        for u, v in zip(got, first):
            assert np.array_equal(u, v), rep


def test_two_streams_equal_serial_runs(ctx):
    """Forward + backward of two batches in flight on two streams at once
    (each stream has its own plan and loss scratch) equal the same runs made
    one after the other, bit for bit."""
    A = float_pairs(2, 96, 40, 30, 560, noise=0.002)
    B = float_pairs(1, 80, 48, 24, 570, noise=0.002)
    p = osoft.SoftParams()
    serial = [run_gpu(ctx, *A, 30, p), run_gpu(ctx, *B, 24, p)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(2):
        torch.cuda.synchronize()
        live = []
        for i, (case, dmax) in enumerate(((A, 30), (B, 24))):
            with torch.cuda.stream(streams[i]):
                live.append(launch_step(ctx, *case, dmax, p))
        torch.cuda.synchronize()
        for i, (d_hat, loss, left, right, lam) in enumerate(live):
            got = (d_hat.detach().cpu().numpy(), float(loss.detach().cpu()[0]),
                   left.grad.cpu().numpy(), right.grad.cpu().numpy(), lam.grad.cpu().numpy())
            for u, v in zip(got, serial[i]):
                assert np.array_equal(np.asarray(u), np.asarray(v)), (rep, i)


def test_paper_size_batch_rows_match_oracle(ctx):
    """4 x 1436x992, Dmax = 145 (the differentiable configuration): d_hat of
    a band of rows against the oracle run on a crop of rows wide enough that
    the band's features, windows and borders are those of the full image."""
    W, H, dmax = 1436, 992, 145
    L, R, G, M = float_pairs(4, W, H, dmax, 400)
    p = osoft.SoftParams()
    lambdas = torch.tensor([p.lambda_ad, p.lambda_census], dtype=torch.float32, device=DEV,
                           requires_grad=True)
    left = to_dev(L).requires_grad_(True)
    right = to_dev(R).requires_grad_(True)
    d_hat = soft_disparity(ctx, left, right, lambdas, dmax, sp_from(p))
    loss = l1_loss(ctx, d_hat, to_dev(G.astype(np.int16)), to_dev(M.astype(np.uint8)))
    loss.backward()
    torch.cuda.synchronize()
    dh = d_hat.detach().cpu().numpy()
    assert np.all(np.isfinite(dh)) and dh.min() >= 0 and dh.max() <= 72
    assert np.all(np.isfinite(left.grad.cpu().numpy()))
    assert np.all(np.isfinite(right.grad.cpu().numpy()))
    assert np.all(np.isfinite(lambdas.grad.cpu().numpy()))
    y0, y1 = 240, 256                    # half-res rows checked (band boundary at 248)
    ya, yb = y0 - 36, y1 + 36            # crop in half-res rows
    for i in (0, 3):
        Lc = L[i, 2 * ya:2 * yb]
        Rc = R[i, 2 * ya:2 * yb]
        ref = oracle_dhat(Lc[None], Rc[None], dmax, p)[0]
        got = dh[i, y0:y1]
        assert float(np.abs(got - ref[y0 - ya:y1 - ya]).max()) <= 1e-3


def test_feature_reuse_in_interleaved_backwards(ctx):
    """The autograd backward reuses the forward's features and weights when
    the plan still holds them: forward A, forward B (other tensors, same
    shape, same plan, whose weights replace A's), then the backward of A must
    recompute A's features and aggregate and give A's gradients, as must B's
    backward after it (A's backward recomputed the slabs over B's weights).
    The reference runs took the saved-weights path, these the recomputing
    one: equal to float rounding."""
    p = osoft.SoftParams()
    A = float_pairs(1, 96, 40, 30, 570, noise=0.002)
    B = float_pairs(1, 96, 40, 30, 571, noise=0.002)
    ref_a = run_gpu(ctx, *A, 30, p)
    ref_b = run_gpu(ctx, *B, 30, p)
    outs = []
    for L, R, G, M in (A, B):
        left = to_dev(L).requires_grad_(True)
        right = to_dev(R).requires_grad_(True)
        lam = torch.tensor((p.lambda_ad, p.lambda_census), dtype=torch.float32, device=DEV,
                           requires_grad=True)
        d = soft_disparity(ctx, left, right, lam, 30, sp_from(p))
        loss = l1_loss(ctx, d, to_dev(G.astype(np.int16)), to_dev(M.astype(np.uint8)))
        outs.append((loss, left, right, lam))
    for (loss, left, right, lam), ref, nm in zip(outs, (ref_a, ref_b), "AB"):
        loss.backward()
        torch.cuda.synchronize()
        assert_grad_close(left.grad.cpu().numpy(), ref[2], f"{nm} g_left", rel=1e-5,
                          rel_elem=1e-4)
        assert_grad_close(right.grad.cpu().numpy(), ref[3], f"{nm} g_right", rel=1e-5,
                          rel_elem=1e-4)
        g = lam.grad.cpu().numpy()
        assert np.all(np.abs(g - ref[4]) <= 1e-5 * np.abs(ref[4])), (nm, g, ref[4])


def soft_grads(ctx, left, right, lam, dmax, p, g_dhat, fwd_flags, bwd_flags, slab=0):
    """Forward then backward through the C ABI with the given flags."""
    fp = sp_from(p, slab)
    fp.flags = fwd_flags
    d_hat, lse2 = ctx.soft_forward(left, right, lam, dmax, fp)
    bp = sp_from(p, slab)
    bp.flags = bwd_flags
    gl, gr, glam = ctx.soft_backward(left, right, lam, dmax, d_hat, lse2, g_dhat, bp)
    torch.cuda.synchronize()
    return d_hat.cpu().numpy(), gl.cpu().numpy(), gr.cpu().numpy(), glam.cpu().numpy()


def test_saved_weights_path_matches_recompute(ctx):
    """The backward that forms dL/dCA from the forward's saved weights
    (k_soft_tcolw) equals the one that recomputes the aggregate per slab
    (k_soft_agg, k_soft_tcol) to float rounding, on the FD configuration and
    on odd sizes with three strips; with the slab smaller than D the forward
    cannot save the weights and both calls take the recomputing path, bit
    for bit."""
    from paper_2212_00488_amd.binding import SOFT_F_REUSE_FEATURES, SOFT_F_SAVE_WEIGHTS
    p = osoft.SoftParams()
    for (n, W, H, dmax, seed) in ((2, 64, 48, 32, 580), (3, 150, 30, 40, 581), (1, 67, 41, 20, 582)):
        L, R, G, M = float_pairs(n, W, H, dmax, seed, noise=0.002)
        left, right = to_dev(L), to_dev(R)
        lam = torch.tensor((p.lambda_ad, p.lambda_census), dtype=torch.float32, device=DEV)
        X, Y = (W + 1) // 2, (H + 1) // 2
        g = to_dev(np.random.default_rng(seed).standard_normal((n, Y, X)).astype(np.float32))
        print(f"[soft] saved weights vs recompute {W}x{H} Dmax={dmax} n={n}", flush=True)
        rec = soft_grads(ctx, left, right, lam, dmax, p, g, 0, SOFT_F_REUSE_FEATURES)
        sav = soft_grads(ctx, left, right, lam, dmax, p, g, SOFT_F_SAVE_WEIGHTS,
                         SOFT_F_REUSE_FEATURES)
        assert np.array_equal(rec[0], sav[0])
        assert_grad_close(sav[1], rec[1], "saved g_left", rel=1e-5, rel_elem=1e-4)
        assert_grad_close(sav[2], rec[2], "saved g_right", rel=1e-5, rel_elem=1e-4)
        assert np.all(np.abs(sav[3] - rec[3]) <= 1e-5 * np.abs(rec[3])), (sav[3], rec[3])
        # slabs of 3: nothing saved, the same recomputing path both times
        a = soft_grads(ctx, left, right, lam, dmax, p, g, 0, SOFT_F_REUSE_FEATURES, slab=3)
        b = soft_grads(ctx, left, right, lam, dmax, p, g, SOFT_F_SAVE_WEIGHTS,
                       SOFT_F_REUSE_FEATURES, slab=3)
        for u, v in zip(a, b):
            assert np.array_equal(u, v)


def test_saved_weights_dropped_by_a_later_forward(ctx):
    """A forward that saves weights, then new data written into the same
    tensors and a forward without saving: the backward (same pointers,
    REUSE_FEATURES) must not take the first forward's weights; its gradients
    are those of the new data."""
    from paper_2212_00488_amd.binding import SOFT_F_REUSE_FEATURES, SOFT_F_SAVE_WEIGHTS
    p = osoft.SoftParams()
    A = float_pairs(1, 96, 40, 30, 590, noise=0.002)
    B = float_pairs(1, 96, 40, 30, 591, noise=0.002)
    lam = torch.tensor((p.lambda_ad, p.lambda_census), dtype=torch.float32, device=DEV)
    g = to_dev(np.random.default_rng(592).standard_normal((1, 20, 48)).astype(np.float32))
    lb, rb = to_dev(B[0]), to_dev(B[1])
    ref = soft_grads(ctx, lb, rb, lam, 30, p, g, 0, 0)
    left, right = to_dev(A[0]), to_dev(A[1])
    fp = sp_from(p)
    fp.flags = SOFT_F_SAVE_WEIGHTS
    ctx.soft_forward(left, right, lam, 30, fp)
    left.copy_(lb)
    right.copy_(rb)
    got = soft_grads(ctx, left, right, lam, 30, p, g, 0, SOFT_F_REUSE_FEATURES)
    for u, v in zip(got, ref):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("case", [
    # 135 disparities: two slabs, whose terms the backward forms from saved CA
    dict(W=290, H=14, dmax=270, n=1, seed=600),
    # 768 half rows: three bands of k_soft_agg with 382 rows at most (24 a wave).
    # 4 columns only: among many pixels some pair of half-image intensities is
    # nearer than float rounding, and the sign of its difference is not the oracle's
    dict(W=8, H=1536, dmax=4, n=1, seed=601, arm_y=63),
    # bands with 17 and 18 rows a wave, two strips, the second of one column
    dict(W=130, H=440, dmax=10, n=1, seed=602),
])
def test_slabs_and_bands_match_oracle(ctx, case):
    """The largest arrangements of k_soft_agg and the slabs beyond one, saved and
    computed again, against the oracle."""
    W, H, dmax, n, seed = case["W"], case["H"], case["dmax"], case["n"], case["seed"]
    p = osoft.SoftParams(**({"arm_y": case["arm_y"]} if "arm_y" in case else {}))
    L, R, G, M = float_pairs(n, W, H, dmax, seed, noise=0.002)
    print(f"[soft] slabs and bands {W}x{H} Dmax={dmax}", flush=True)
    ref = oracle_dhat(L, R, dmax, p)
    rloss, rgl, rgr, rglam = osoft.loss_and_grads(list(L), list(R), list(G), list(M), dmax, p)
    for slab in (0, 7):
        d_hat, loss, gl, gr, glam = run_gpu(ctx, L, R, G, M, dmax, p, slab=slab)
        assert float(np.abs(d_hat - ref).max()) <= 1e-3
        assert_grad_close(gl, rgl, "g_left")
        assert_grad_close(gr, rgr, "g_right")
        for k in range(2):
            assert abs(glam[k] - rglam[k]) <= 1e-3 * abs(rglam[k]) + 1e-9, (k, glam, rglam)


def test_scratch_cap_shrinks_the_planes(ctx):
    """Under smaller and smaller scratch caps a plan holds the weights of all D, of
    a slab, of smaller slabs, and at last is refused; the map stays the same and
    the gradients stay those of the uncapped plan to float rounding (sums over
    slabs of other sizes; dL/dlambda's terms cancel by three digits)."""
    from paper_2212_00488_amd.binding import SOFT_F_REUSE_FEATURES, SOFT_F_SAVE_WEIGHTS, StereoError
    p, dmax = osoft.SoftParams(), 128
    L, R, G, M = float_pairs(1, 150, 60, dmax, 610, noise=0.002)
    left, right = to_dev(L), to_dev(R)
    lam = torch.tensor((p.lambda_ad, p.lambda_census), dtype=torch.float32, device=DEV)
    g = to_dev(np.random.default_rng(610).standard_normal((1, 30, 75)).astype(np.float32))
    ref = soft_grads(ctx, left, right, lam, dmax, p, g, SOFT_F_SAVE_WEIGHTS, SOFT_F_REUSE_FEATURES)
    # planes of all 64 disparities take 2 x 600 kB
    ran, refused = 0, 0
    for cap in (4000, 2200, 1700, 1400, 1200, 1000, 900, 800, 100):
        small = Stereo(0, mem_cap=cap * 1000)
        try:
            got = soft_grads(small, left, right, lam, dmax, p, g, SOFT_F_SAVE_WEIGHTS,
                             SOFT_F_REUSE_FEATURES)
        except StereoError:
            refused += 1
            continue
        finally:
            small.close()
        ran += 1
        assert np.array_equal(got[0], ref[0])
        assert_grad_close(got[1], ref[1], f"g_left, cap {cap} kB", rel=1e-5, rel_elem=1e-4)
        assert_grad_close(got[2], ref[2], f"g_right, cap {cap} kB", rel=1e-5, rel_elem=1e-4)
        assert np.all(np.abs(got[3] - ref[3]) <= 1e-4 * np.abs(ref[3])), (cap, got[3], ref[3])
    assert ran >= 3 and refused >= 1, (ran, refused)


@pytest.mark.parametrize("case", [
    dict(W=128, H=10, dmax=32, seed=620),              # one full strip, one tile of 16
    dict(W=130, H=10, dmax=34, seed=621, arm_x=31),    # one column more, one disparity more
    dict(W=190, H=10, dmax=66, seed=622, arm_x=31),    # sources of both tiles past the image
    dict(W=194, H=10, dmax=34, seed=623, arm_x=16),
    # two full strips, no remainder row; an input whose half-image differences
    # stay away from 0 (at seed 624 one is 2.5e-8, below float rounding, and its
    # sign is not the oracle's)
    dict(W=256, H=8, dmax=30, seed=625, arm_x=0),
])
def test_horizontal_adjoint_edges_match_oracle(ctx, case):
    """k_soft_tr at the edges of its strips (64 columns, sources 32 further on
    either side), tiles (16 disparities) and blocks (4 rows)."""
    W, H, dmax, seed = case["W"], case["H"], case["dmax"], case["seed"]
    p = osoft.SoftParams(**({"arm_x": case["arm_x"]} if "arm_x" in case else {}))
    L, R, G, M = float_pairs(1, W, H, dmax, seed, noise=0.002)
    print(f"[soft] horizontal adjoint {W}x{H} Dmax={dmax}", flush=True)
    rloss, rgl, rgr, rglam = osoft.loss_and_grads(list(L), list(R), list(G), list(M), dmax, p)
    d_hat, loss, gl, gr, glam = run_gpu(ctx, L, R, G, M, dmax, p)
    assert_grad_close(gl, rgl, "g_left")
    assert_grad_close(gr, rgr, "g_right")
    for k in range(2):
        assert abs(glam[k] - rglam[k]) <= 1e-3 * abs(rglam[k]) + 1e-9, (k, glam, rglam)


def test_adjoint_terms_keep_their_unit_at_a_mantissa_of_ones():
    """k_soft_tr's terms are rounded to 2^(e-24), 2^(e-1) <= the largest |dL/dCA_x|
    of a row's sources < 2^e: also where that largest value is all ones in its
    mantissa, just below 2^e.  Constant images, so that every quantity below is
    exact in floats: column A's three sources add up to a largest value of S units
    of 2^(e-24), S = 2^24 - 2, 2^24 - 1 and 2^24, and column B's is 0.8 of 2^(e-23)
    with e of the first two: one unit there, none for the third."""
    f = np.float32
    W, H, X, Y, arm_y, tau = 256, 160, 128, 80, 2, f(0.2)
    p = soft_default_params(tau=float(tau), arm_x=0, arm_y=arm_y)
    left = torch.full((1, H, W, 3), 1e-20, device=DEV)
    right = torch.zeros((1, H, W, 3), device=DEV)
    lam = torch.tensor((255.0, 30.0), device=DEV)
    A, B = 40, 48

    def const(g):  # A of k_soft_bprep for a g_dhat, |S| = 5
        return f(f(-g * f(f(1) / f(2 * arm_y + 1))) * f(f(1) / tau))

    def g_for(value):  # a g_dhat whose dL/dCA at d = 1 is exactly value
        g = f(-value * 4)
        for _ in range(64):
            got = const(g) * f(0.25)
            if got == f(value):
                return g
            g = np.nextafter(g, f(-np.inf) if got < value else f(np.inf))
        return None

    # terms of column A: q units of 2^-25 (all below 2^23: 2^-2 is the column's scale)
    g = np.zeros((1, Y, X), f)
    rows, units = [], []
    y = 6
    for S in (2**24 - 2, 2**24 - 1, 2**24):
        for q1 in (6710886, 7000001, 7300000):
            q2 = 5000000 + q1 % 1000
            qs = (q1, q2, S - q1 - q2)
            gs = [g_for(q * 2.0**-25) for q in qs]
            if None in gs or max(qs) >= 2**23:
                continue
            g[0, y - 1:y + 2, A] = gs
            g[0, y, B] = f(-0.8 * 2.0**-22)
            rows.append(y)
            units.append(S)
            y += 8
    assert set(units) == {2**24 - 2, 2**24 - 1, 2**24}, units
    c = Stereo(0)
    d_hat, lse2 = c.soft_forward(left, right, lam, 4, p)
    assert float((d_hat[0, :, 1:] - 0.5).abs().max()) == 0.0
    gl, gr, _ = c.soft_backward(left, right, lam, 4, d_hat, lse2, torch.from_numpy(g).to(DEV), p)
    torch.cuda.synchronize()
    c.close()
    # half-image gradient from the red channel of the pixel at even coordinates
    half = gr[0, ::2, ::2, 0].cpu().numpy().astype(np.float64) * (2304.0 / 77.0)
    for y, S in zip(rows, units):
        # right pixel x - 1 takes -dL/dC(x, d = 1)
        a, b = -half[y, A - 1], -half[y, B - 1]
        print(f"[soft] S = 2^24 - {2**24 - S}: A {a!r}, B {b!r}", flush=True)
        assert abs(a - S * 2.0**-25) <= 2.0**-22 * a, (S, a)
        exp = 2.0**-24 if S < 2**24 else 0.0
        assert abs(b - exp) <= 2.0**-40, (S, b, exp)


# ------------------------------------------------------- scratch under a cap


def device_bytes_free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


class HeadCall:
    """Device inputs of one call of the head, made before any memory is counted;
    the outputs are torch's and stay in its cache."""

    def __init__(self, n, W, H, dmax, seed, slab=0):
        g = torch.Generator().manual_seed(seed)
        self.left = torch.rand((n, H, W, 3), generator=g).to(DEV)
        self.right = torch.rand((n, H, W, 3), generator=g).to(DEV)
        self.g = torch.randn((n, (H + 1) // 2, (W + 1) // 2), generator=g).to(DEV)
        self.lam = torch.tensor((10.0, 30.0), device=DEV)
        self.dmax, self.slab = dmax, slab

    def forward(self, ctx, flags=0):
        d_hat, lse2 = ctx.soft_forward(self.left, self.right, self.lam, self.dmax,
                                       soft_default_params(flags=flags, slab=self.slab))
        return d_hat, lse2

    def backward(self, ctx, d_hat, lse2, flags=0):
        return ctx.soft_backward(self.left, self.right, self.lam, self.dmax, d_hat, lse2, self.g,
                                 soft_default_params(flags=flags, slab=self.slab))

    def step(self, ctx, save=True):
        from paper_2212_00488_amd.binding import SOFT_F_REUSE_FEATURES, SOFT_F_SAVE_WEIGHTS
        d_hat, lse2 = self.forward(ctx, SOFT_F_SAVE_WEIGHTS if save else 0)
        out = (d_hat,) + self.backward(ctx, d_hat, lse2, SOFT_F_REUSE_FEATURES)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]


def taken_by(ctx, free0):
    return free0 - device_bytes_free()


def test_cap_frees_idle_plans_before_smaller_slabs():
    """A cap that holds one plan of two shapes trained in turn: each call frees
    the idle plan and runs its shape with the slabs of a context without a cap
    (the scratch it takes, and every bit of its results), not with smaller ones
    beside the idle plan."""
    calls = [HeadCall(1, 640, 480, 64, 630), HeadCall(1, 620, 496, 64, 631)]
    ref, alone = [], []
    for h in calls:
        for _ in range(2):  # the first time loads kernels
            free0 = device_bytes_free()
            c = Stereo(0)
            r = h.step(c)
            taken = taken_by(c, free0)
            c.close()
        ref.append(r)
        alone.append(taken)
    print(f"[soft] scratch of each shape alone: {alone}", flush=True)
    assert min(alone) > 20 << 20
    free0 = device_bytes_free()
    c = Stereo(0, mem_cap=int(1.75 * max(alone)))
    for k in (0, 1, 0, 1):
        got = calls[k].step(c)
        taken = taken_by(c, free0)
        print(f"[soft] shape {k}: scratch {taken}", flush=True)
        assert abs(taken - alone[k]) <= 4 << 20, (k, taken, alone)
        for u, v in zip(got, ref[k]):
            assert np.array_equal(u, v)
    c.close()


def test_weight_planes_of_all_disparities_only_for_a_backward():
    """4 x 1920x1080, 128 disparities: a forward that saves nothing takes the
    slab's planes only (at most 1 GiB beside the pixel planes); the first one that
    saves its weights adds the planes of the other disparities."""
    from paper_2212_00488_amd.binding import SOFT_F_SAVE_WEIGHTS
    h = HeadCall(4, 1920, 1080, 256, 632)
    c = Stereo(0)
    h.forward(c)  # kernels, and the outputs' memory in torch's cache
    c.close()
    free0 = device_bytes_free()
    c = Stereo(0)
    h.forward(c)
    plain = taken_by(c, free0)
    h.forward(c, SOFT_F_SAVE_WEIGHTS)
    saving = taken_by(c, free0)
    c.close()
    print(f"[soft] scratch without saving {plain}, with {saving}", flush=True)
    plane = 4 * 540 * 960 * 4  # of one disparity
    assert plain <= (1 << 30) + 60 * plane // 2, plain
    assert saving >= plain + 32 * plane, (plain, saving)


def test_optional_weight_planes_give_way():
    """256 disparities (two slabs), two shapes under a cap that holds both plans
    and the further weight planes of one: these go to the shape in use, the other
    one's once it has not been used since; a pair of the integer path that needs
    their room gets it; and the gradients are the same bits throughout."""
    calls = [HeadCall(1, 1100, 400, 512, 640), HeadCall(1, 1090, 404, 512, 641)]
    ref, base, full = [], [], []
    for h in calls:
        for _ in range(2):
            free0 = device_bytes_free()
            c = Stereo(0)
            h.forward(c)
            b = taken_by(c, free0)
            r = h.step(c)
            f = taken_by(c, free0)
            c.close()
        ref.append(r)
        base.append(b)
        full.append(f)
    print(f"[soft] plan {base}, with the weights of all disparities {full}", flush=True)
    rest = min(f - b for f, b in zip(full, base))
    assert rest >= 40 << 20
    free0 = device_bytes_free()
    c = Stereo(0, mem_cap=sum(base) + rest + (16 << 20))
    # (shape, who holds the further planes after the step)
    for k, owner in ((0, 0), (1, 0), (1, 1), (0, 1), (1, 1), (0, 1), (0, 0)):
        got = calls[k].step(c)
        taken = taken_by(c, free0)
        other = full[owner] + (base[1 - owner] if taken > full[owner] + (8 << 20) else 0)
        print(f"[soft] shape {k}: scratch {taken}", flush=True)
        assert abs(taken - other) <= 8 << 20, (k, owner, taken, base, full)
        for u, v in zip(got, ref[k]):
            assert np.array_equal(u, v)
    # the integer path takes their room, not STEREO_ENOMEM
    g = torch.Generator().manual_seed(9)
    lt = torch.randint(0, 256, (992, 1436, 3), dtype=torch.uint8, generator=g).to(DEV)
    big = c.disparity(lt, lt, 145)
    torch.cuda.synchronize()
    alone = Stereo(0)
    assert torch.equal(big, alone.disparity(lt, lt, 145))
    alone.close()
    for u, v in zip(calls[0].step(c), ref[0]):
        assert np.array_equal(u, v)
    c.close()


def test_training_step_captured_after_a_plain_forward():
    """A plan whose calls saved nothing so far, then forward with saving and
    backward captured in a graph (where nothing can be allocated): each replay
    gives the eager gradients, with one slab and with two."""
    from paper_2212_00488_amd.binding import SOFT_F_REUSE_FEATURES, SOFT_F_SAVE_WEIGHTS
    for W, H, dmax, seed in ((96, 40, 32, 650), (290, 20, 270, 651)):
        print(f"[soft] captured step {W}x{H} Dmax={dmax}", flush=True)
        h = HeadCall(1, W, H, dmax, seed)
        c, s = Stereo(0), torch.cuda.Stream()
        ref = h.step(c, save=False)
        with torch.cuda.stream(s):
            h.forward(c)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            d_hat, lse2 = h.forward(c, SOFT_F_SAVE_WEIGHTS)
            out = (d_hat,) + h.backward(c, d_hat, lse2, SOFT_F_REUSE_FEATURES)
        for k in range(3):
            for t in out:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out[0].cpu().numpy(), ref[0])
            for t, r, nm in zip(out[1:], ref[1:], ("g_left", "g_right", "g_lambdas")):
                t = t.cpu().numpy()
                assert np.abs(t - r).max() <= 1e-5 * np.abs(r).max(), (k, nm)
            h.step(c)  # eager work between the replays
        del graph
        torch.cuda.synchronize()
        c.close()
