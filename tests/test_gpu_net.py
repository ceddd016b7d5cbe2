"""GPU parity of the learned-initial-guess network with the oracle (oracle/convnet.py).

Bars (bfloat16 storage, fp32 accumulation on both sides of the rounding points the oracle
emulates): features within one bfloat16 step of the rounded oracle features; target and guess
maps within float32 / float64 rounding; network output within 1e-2 (relative norm) of the
rounded oracle; every layer's weight and bias gradient within 3e-2 (relative norm), the whole
gradient's cosine with the oracle's above 0.999.
"""
import numpy as np
import pytest
import torch

from oracle import convnet as cn
from oracle import dda as odda
from paper_0704_0037_amd import inputs

pytestmark = pytest.mark.gpu


def _dda():
    from paper_0704_0037_amd import dda
    return dda


def _particles(G):
    return [
        (inputs.ellipsoid_mask((12, 9, 7), (6, 4.5, 3.5)), 1.5 + 0.02j, 0.4, inputs.beams_for_orientations(1, seed=2)[1]),
        (inputs.sphere_mask(G - 2), 1.8, 0.3, inputs.beams_for_orientations(1, seed=5)[0]),
    ]


def _params(seed):
    p = cn.init_params(seed).astype(np.float64)
    rng = np.random.default_rng(seed + 100)
    return cn.flatten([(W, rng.standard_normal(b.shape) * 0.05) for W, b in cn.unflatten(p)]).astype(np.float32)


def _bf16_to_np(t):
    return t.float().cpu().numpy().astype(np.float64)


def test_features_target_guess_maps():
    dda = _dda()
    G = 16
    p = _params(1)
    for mask, m, kd, beam in _particles(G):
        with dda.Context(mask, m, kd) as ctx, dda.Net(G, p, max_batch=1) as net:
            f = _bf16_to_np(net.features(ctx, beam)).reshape(G, G, G, 16)
            fo = cn.bf16(cn.features(mask, m, kd, beam.prop, beam.pol, G))
            step = np.maximum(np.abs(fo), 1e-6) * 2.0 ** -7
            assert np.all(np.abs(f - fo) <= step)
            alpha = odda.alpha_ldr(m, kd, beam.prop, beam.pol)
            beta = odda.beta_of_alpha(alpha)
            x = inputs.random_vector(ctx.n, seed=4)
            t = net.target(ctx, beam, torch.from_numpy(x).cuda()).cpu().numpy().reshape(G, G, G, 6)
            to = cn.target(mask, kd, beta, beam.prop, beam.pol, x.T, G)
            assert np.abs(t - to).max() < 1e-6 * np.abs(to).max()
            feat = net.features(ctx, beam).reshape(1, G ** 3, 16)
            out = net.forward(feat)
            x0 = net.guess(ctx, [beam], feat)[0].cpu().numpy().T
            x0o = cn.guess(mask, kd, beta, beam.prop, beam.pol, out[0].cpu().numpy().astype(np.float64), G)
            assert np.abs(x0 - x0o).max() < 1e-12 * np.abs(x0o).max()


def _batch(net, G, solved=False):
    """Features and targets of the two particles; targets from random vectors or from solutions."""
    dda = _dda()
    feats, tgts, masks = [], [], []
    for i, (mask, m, kd, beam) in enumerate(_particles(G)):
        with dda.Context(mask, m, kd) as ctx:
            feats.append(net.features(ctx, beam))
            if solved:
                x = ctx.solve([beam], tol=1e-6)[0][0].contiguous()
            else:
                x = torch.from_numpy(inputs.random_vector(ctx.n, seed=10 + i) * 0.3).cuda()
            tgts.append(net.target(ctx, beam, x))
    feat = torch.stack(feats)
    tgt = torch.stack(tgts)
    f_np = _bf16_to_np(feat).reshape(-1, G, G, G, 16)
    t_np = tgt.cpu().numpy().astype(np.float64).reshape(-1, G, G, G, 6)
    return feat, tgt, f_np, t_np, f_np[..., 0]


def test_forward_matches_oracle():
    dda = _dda()
    G = 16
    p = _params(2)
    with dda.Net(G, p, max_batch=2) as net:
        feat, tgt, f_np, t_np, m_np = _batch(net, G)
        out = net.forward(feat).cpu().numpy().astype(np.float64).reshape(-1, G, G, G, 6)
    for s in range(out.shape[0]):
        ref = cn.forward(p, f_np[s], bf16_round=True)["out"]
        assert np.linalg.norm(out[s] - ref) < 1e-2 * np.linalg.norm(ref)


def test_gradient_matches_oracle():
    dda = _dda()
    G = 16
    p = _params(3)
    with dda.Net(G, p, max_batch=2) as net:
        feat, tgt, f_np, t_np, m_np = _batch(net, G)
        loss, g = net.grad(feat, tgt)
    lo, go = cn.loss_and_grad(p, f_np, t_np, m_np, bf16_round=True)
    assert abs(loss - lo) < 1e-2 * lo
    g = g.astype(np.float64)
    assert g @ go / (np.linalg.norm(g) * np.linalg.norm(go)) > 0.999
    off = 0
    for li, (ci, co, *_) in enumerate(cn.LAYERS):
        for n in (27 * ci * co, co):
            a, b = g[off:off + n], go[off:off + n]
            assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(b) + 1e-12, (li, n)
            off += n


def test_training_lowers_the_loss():
    dda = _dda()
    G = 16
    with dda.Net(G, cn.init_params(4), max_batch=2) as net:
        feat, tgt, *_ = _batch(net, G, solved=True)
        l0 = net.train_step(feat, tgt, 2e-3)
        for _ in range(60):
            l = net.train_step(feat, tgt, 2e-3)
        assert l < 0.3 * l0
        p = net.params()
        assert np.all(np.isfinite(p))


def test_initial_guess_check_falls_back_to_zero():
    dda = _dda()
    mask = inputs.sphere_mask(8)
    with dda.Context(mask, 1.5, 0.5) as ctx:
        xz, iz, _ = ctx.solve([inputs.X_POL], tol=1e-8)
        bad = 10 * ctx.rhs(inputs.X_POL).reshape(1, 3, ctx.n)
        xb, ib, st = ctx.solve([inputs.X_POL], tol=1e-8, x0=bad, x0_check=True)
        assert st == 0 and ib[0]["iters"] == iz[0]["iters"]
        assert torch.equal(xb, xz)
        # a good guess is kept
        xg, ig, st = ctx.solve([inputs.X_POL], tol=1e-8, x0=xz, x0_check=True)
        assert st == 0 and ig[0]["iters"] == 0


def test_trained_guess_lowers_the_initial_residual_but_not_the_iterations():
    """What the trained network gains, measured: trained on solver output for small random particles,
    its guess starts held-out solves from a residual at least a quarter below the untrained network's
    (x0 = b), yet QMR from it needs within 10 % of the iterations from a zero guess.  This is the
    negative result of the full-size runs (2,000 training and 200 held-out particles: initial residual
    0.63 against 1.02, iterations x 0.99), asserted so that a change in either direction is seen; plain
    QMR stays the fallback and the judge of convergence (every solve converges)."""
    from paper_0704_0037_amd import learned_guess as lg
    ev, _ = lg.run(grid=48, n_train=600, n_eval=16, epochs=30, batch=8, lr=1e-3, seed=5000, quiet=True)
    assert all(r["status"] == [0, 0, 0] for r in ev["rows"])
    assert ev["mean_res0_guess"] < 0.75 * ev["mean_res0_b"], ev
    assert 0.9 < ev["iteration_ratio"] < 1.1, ev


@pytest.mark.parametrize("G,B,grad", [(8, 1, True), (8, 3, True), (24, 2, True), (40, 1, True), (72, 1, False)])
def test_boxes_on_both_sides_of_the_tiled_kernels(G, B, grad):
    """The tiled kernels take boxes whose side is a multiple of 8 (four rows and steps of eight voxels;
    the planes of 32 channels up to 56, the weight gradient up to 64), the gathering ones the rest:
    levels of 8 4 2 1, 24 12 6 3 and 40 20 10 5 voxels, and 72, where only the 16-channel planes still
    fit.  Bars as above (bfloat16 rounding); a batch gives each of its particles bit for bit."""
    dda = _dda()
    p = _params(6)
    rng = np.random.default_rng(G + B)
    f = rng.standard_normal((B, G, G, G, 16)) * 0.5
    f[..., 0] = rng.random((B, G, G, G)) < 0.4
    f = cn.bf16(f)
    t = (rng.standard_normal((B, G, G, G, 6)) * 0.3).astype(np.float32)
    feat = torch.from_numpy(f.astype(np.float32)).cuda().to(torch.bfloat16).reshape(B, G ** 3, 16)
    with dda.Net(G, p, max_batch=B) as net:
        out = net.forward(feat)
        for s in range(B):
            assert torch.equal(net.forward(feat[s:s + 1].contiguous())[0], out[s])
        if grad:
            loss, g = net.grad(feat, torch.from_numpy(t).cuda().reshape(B, G ** 3, 6))
    ref = cn.forward(p, f[0], bf16_round=True)["out"]
    o = out[0].cpu().numpy().astype(np.float64).reshape(G, G, G, 6)
    assert np.linalg.norm(o - ref) < 1e-2 * np.linalg.norm(ref)
    if not grad:
        return
    lo, go = cn.loss_and_grad(p, f, t.astype(np.float64), f[..., 0], bf16_round=True)
    assert abs(loss - lo) < 1e-2 * lo
    off = 0
    for li, (ci, co, *_) in enumerate(cn.LAYERS):
        for n in (27 * ci * co, co):
            a, b = g[off:off + n].astype(np.float64), go[off:off + n]
            assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(b) + 1e-12, (li, n)
            off += n


def test_memory_of_large_batches_is_the_tensors():
    """The weight gradient's partial sums do not grow with the batch: 4,096 more particles of 8^3 cells take
    the network's tensors (292 bytes a cell: 16 to 64 channels in bfloat16 on four levels) and no 110 KB each
    for sums of their own (a quarter is left for rounding by the allocator)."""
    dda = _dda()
    p = _params(7)
    used = []
    for B in (4096, 8192):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        with dda.Net(8, p, max_batch=B):
            used.append(before - torch.cuda.mem_get_info()[0])
    assert used[1] - used[0] < 1.25 * 4096 * 512 * 292


@pytest.mark.parametrize("G,B", [(8, 2048), (16, 512), (24, 384)])
def test_blocks_that_take_several_tiles(G, B):
    """Weight gradients of batches with more tiles than blocks (one to three a block) against the eight
    parts of the batch, which take one each: the same mask in every part, so the mean over
    eight times the cells scales each part's output gradient by exactly 1/8 and only the order of the
    single-precision sums differs (up to 10^6 products of random sign: 1e-4 of a layer's norm)."""
    dda = _dda()
    g = torch.Generator("cuda").manual_seed(G)
    n = B // 8
    feat = torch.randn((8, n, G ** 3, 16), device="cuda", generator=g) * 0.5
    feat[..., 0] = (torch.rand((n, G ** 3), device="cuda", generator=g) < 0.4).float()
    feat = feat.to(torch.bfloat16)
    tgt = torch.randn((8, n, G ** 3, 6), device="cuda", generator=g) * 0.3
    with dda.Net(G, _params(8), max_batch=B) as net:
        loss, grad = net.grad(feat.reshape(B, G ** 3, 16), tgt.reshape(B, G ** 3, 6))
        parts = [net.grad(feat[i].contiguous(), tgt[i].contiguous()) for i in range(8)]
    ref = np.mean([q.astype(np.float64) for _, q in parts], axis=0)
    assert abs(loss - np.mean([v for v, _ in parts])) < 1e-6 * loss
    off = 0
    for li, (ci, co, *_) in enumerate(cn.LAYERS):
        for k in (27 * ci * co, co):
            a, b = grad[off:off + k].astype(np.float64), ref[off:off + k]
            assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b) + 1e-12, (li, k)
            off += k


@pytest.mark.parametrize("G,grad", [(48, False), (56, False), (64, True)])
def test_largest_boxes_of_the_tiled_kernels(G, grad):
    """Three planes of 32 channels fit 64 KiB up to a side of 48 (56 takes the gathering kernel there), and
    the weight gradient's two staged pairs per thread reach 64.  Bars as above."""
    dda = _dda()
    p = _params(9)
    rng = np.random.default_rng(G)
    f = rng.standard_normal((1, G, G, G, 16)) * 0.5
    f[..., 0] = rng.random((1, G, G, G)) < 0.4
    f = cn.bf16(f)
    t = (rng.standard_normal((1, G, G, G, 6)) * 0.3).astype(np.float32)
    feat = torch.from_numpy(f.astype(np.float32)).cuda().to(torch.bfloat16).reshape(1, G ** 3, 16)
    with dda.Net(G, p, max_batch=1) as net:
        if not grad:
            o = net.forward(feat)[0].cpu().numpy().astype(np.float64).reshape(G, G, G, 6)
            ref = cn.forward(p, f[0], bf16_round=True)["out"]
            assert np.linalg.norm(o - ref) < 1e-2 * np.linalg.norm(ref)
            return
        loss, g = net.grad(feat, torch.from_numpy(t).cuda().reshape(1, G ** 3, 6))
    lo, go = cn.loss_and_grad(p, f, t.astype(np.float64), f[..., 0], bf16_round=True)
    assert abs(loss - lo) < 1e-2 * lo
    off = 0
    for li, (ci, co, *_) in enumerate(cn.LAYERS):
        for n in (27 * ci * co, co):
            a, b = g[off:off + n].astype(np.float64), go[off:off + n]
            assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(b) + 1e-12, (li, n)
            off += n
