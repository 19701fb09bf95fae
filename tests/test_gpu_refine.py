"""GPU parity of the refinement extras (Sec. III-C, Eq. (refine_loss)):
exposure-compensated L1 gradient and opacity pruning, through the C ABI,
against the oracle."""
import numpy as np
import pytest

from gpu_harness import announce
from oracle.refine import exposure, l1_loss_grad, prune
from synth.scenes import multi_agent

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(37, 53), (40, 52)])
def test_l1_loss_grad_matches_oracle(H, W):
    """37 x 53: ragged, one pixel at a time; 40 x 52: four pixels per load."""
    announce(f"refine l1 grad {H}x{W}")
    import torch
    from paper_2605_10760_amd import l1_loss_grad as gpu_grad
    rng = np.random.default_rng(7)
    V = 3
    c = rng.random((V, 3, H, W)).astype(np.float32)
    d = (0.5 + 3 * rng.random((V, H, W))).astype(np.float32)
    tc = rng.random((V, 3, H, W)).astype(np.float32)
    td = (0.5 + 3 * rng.random((V, H, W))).astype(np.float32)
    tc[0, 0, :2] = c[0, 0, :2]  # exact zeros of the residual: subgradient 0
    ex = np.stack([rng.normal(0, 0.3, V), rng.normal(0, 0.1, V)], 1).astype(np.float32)
    t = lambda a: torch.from_numpy(a).cuda()
    for expo in (None, ex):
        a = np.zeros(V) if expo is None else expo[:, 0]
        b = np.zeros(V) if expo is None else expo[:, 1]
        got = gpu_grad(t(c), t(tc), t(d), t(td), None if expo is None else t(expo), 1.75, 0.25)
        torch.cuda.synchronize()
        ref = l1_loss_grad(c, d, tc, td, a, b, 1.75, 0.25)
        # residuals the FP32 and FP64 evaluations could sign differently
        resid = exposure(c, a, b) - tc
        amb = (np.abs(resid) < 1e-5) & (resid != 0)
        gc = got["d_color"].cpu().numpy()
        np.testing.assert_allclose(gc[~amb], ref["d_color"][~amb], rtol=1e-6, atol=0)
        np.testing.assert_allclose(got["d_depth"].cpu().numpy(), ref["d_depth"], rtol=1e-6, atol=0)
        if expo is not None:
            ge = got["d_exposure"].cpu().numpy()
            scale = np.abs(ref["d_color"]).max() * c[0].size
            np.testing.assert_allclose(ge[:, 0], ref["d_a"], atol=1e-5 * scale)
            np.testing.assert_allclose(ge[:, 1], ref["d_b"], atol=1e-5 * scale)
            assert amb.sum() < 20


# several workgroups of 1024 per view, the last one partly filled, four pixels at
# a time and one at a time
@pytest.mark.parametrize("H,W", [(130, 64), (67, 129)])
def test_l1_loss_grad_several_workgroups(H, W):
    test_l1_loss_grad_matches_oracle(H, W)


def test_prune_matches_oracle():
    announce("refine prune")
    import torch
    from paper_2605_10760_amd import SceneTensors, prune as gpu_prune
    wl = multi_agent(scale=0.01, keyframes=1)
    sc = wl.scene
    rng = np.random.default_rng(8)
    o = sc.opacity_logits.copy()
    o[rng.random(o.shape[0]) < 0.3] = -6.0  # sigmoid = 0.0025: pruned
    # logits at and next to logit(0.005) = -5.2933048...
    o[::97] = np.float32(-5.2933048)
    o[1::97] = np.nextafter(np.float32(-5.2933048), np.float32(0))
    o[2::97] = np.nextafter(np.float32(-5.2933048), np.float32(-10))
    sc.opacity_logits = o
    st_ = SceneTensors.from_numpy(sc)
    out = gpu_prune(st_, 0.005)
    idx, offs = prune(o, sc.set_offsets, 0.005)
    np.testing.assert_array_equal(out.set_offsets, offs)
    np.testing.assert_array_equal(out.means.cpu().numpy(), sc.means[idx])
    np.testing.assert_array_equal(out.log_scales.cpu().numpy(), sc.log_scales[idx])
    np.testing.assert_array_equal(out.quats.cpu().numpy(), sc.quats[idx])
    np.testing.assert_array_equal(out.opacity_logits.cpu().numpy(), o[idx])
    np.testing.assert_array_equal(out.colors.cpu().numpy(), sc.colors[idx])
    assert 0 < idx.shape[0] < o.shape[0]


@pytest.mark.parametrize("V,H,W", [(2, 37, 45), (2, 150, 70)])
def test_ssim_grad_matches_oracle(V, H, W):
    """Ragged tiles in both directions (16 x 64 output tiles, 5-pixel halo)."""
    announce(f"refine ssim {V}x{H}x{W}")
    import torch
    from oracle.ssim import ssim, ssim_term_grad
    from paper_2605_10760_amd import ssim_grad
    rng = np.random.default_rng(9)
    c = rng.random((V, 3, H, W)).astype(np.float32)
    tgt = np.clip(c + 0.1 * rng.normal(size=c.shape), 0, 1).astype(np.float32)
    ex = np.array([[0.15, 0.02], [-0.1, -0.03]], np.float32)
    t = lambda a: torch.from_numpy(a).cuda()
    # accumulated onto: small enough that the FP32 sum keeps the gradient digits
    base = (1e-4 * rng.normal(size=c.shape)).astype(np.float32)
    d_color = t(base.copy())
    d_exp = t(np.array([[1.0, 2.0], [3.0, 4.0]], np.float32))
    out = torch.zeros(1, device="cuda")
    ssim_grad(t(c), t(tgt), d_color, t(ex), d_exp, 0.2, ssim_out=out)
    torch.cuda.synchronize()
    ref = ssim_term_grad(c, tgt, ex[:, 0], ex[:, 1], 0.2)
    xt = np.exp(ex[:, 0])[:, None, None, None] * c + ex[:, 1][:, None, None, None]
    assert abs(out.item() - ssim(xt, tgt)) <= 2e-5
    got = d_color.cpu().numpy() - base
    scale = np.abs(ref["d_color"]).max()
    assert np.abs(got - ref["d_color"]).max() <= 1e-3 * scale
    ge = d_exp.cpu().numpy() - np.array([[1.0, 2.0], [3.0, 4.0]])
    sa = np.abs(ref["d_a"]).max()
    np.testing.assert_allclose(ge[:, 0], ref["d_a"], atol=1e-3 * sa)
    np.testing.assert_allclose(ge[:, 1], ref["d_b"], atol=1e-3 * np.abs(ref["d_b"]).max())


def test_ssim_grad_full_size_sampled():
    """The refinement batch's size, 48 views x 3 x 480 x 640: the gradient and
    exposure gradients of three sampled views against the oracle (the window
    stays inside a view, so a view's gradient is the one-view oracle's scaled
    by 1/48), and the batch's mean SSIM against the mean of the 48 one-view
    means the kernel reports."""
    V, H, W = 48, 480, 640
    announce(f"refine ssim full size {V}x3x{H}x{W}")
    import torch
    from oracle.ssim import ssim, ssim_term_grad
    from paper_2605_10760_amd import ssim_grad
    rng = np.random.default_rng(12)
    c = rng.random((V, 3, H, W), dtype=np.float32)
    tgt = np.clip(c + 0.08 * rng.standard_normal(c.shape, dtype=np.float32), 0, 1)
    ex = np.stack([rng.normal(0, 0.1, V), rng.normal(0, 0.02, V)], 1).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d_color = torch.zeros((V, 3, H, W), device="cuda")
    d_exp = torch.zeros((V, 2), device="cuda")
    out = torch.zeros(1, device="cuda")
    ct, tt, et = t(c), t(tgt), t(ex)
    ssim_grad(ct, tt, d_color, et, d_exp, 0.2, ssim_out=out)
    torch.cuda.synchronize()
    per_view = []
    one = torch.zeros(1, device="cuda")
    for v in range(V):
        ssim_grad(ct[v:v + 1], tt[v:v + 1], torch.zeros((1, 3, H, W), device="cuda"), et[v:v + 1],
                  None, 0.2, ssim_out=one)
        per_view.append(one.item())
    assert abs(out.item() - float(np.mean(per_view))) <= 1e-5
    g = d_color.cpu().numpy()
    ge = d_exp.cpu().numpy()
    for v in (0, 23, 47):
        ref = ssim_term_grad(c[v:v + 1], tgt[v:v + 1], ex[v:v + 1, 0], ex[v:v + 1, 1], 0.2)
        xt = np.exp(ex[v, 0]) * c[v:v + 1].astype(np.float64) + ex[v, 1]
        assert abs(per_view[v] - ssim(xt, tgt[v:v + 1])) <= 2e-5
        want = ref["d_color"][0] / V
        assert np.abs(g[v] - want).max() <= 1e-3 * np.abs(want).max(), v
        np.testing.assert_allclose(ge[v, 0], ref["d_a"][0] / V, rtol=1e-3,
                                   atol=1e-4 * abs(ref["d_a"][0] / V))
        np.testing.assert_allclose(ge[v, 1], ref["d_b"][0] / V, rtol=1e-3,
                                   atol=1e-4 * abs(ref["d_b"][0] / V))


# image widths at the edges of the strips of one to four waves (40, 104, 168 and
# 232 output columns), heights at the edges of the row segments (32 rows and
# multiples of four) and below a window
@pytest.mark.parametrize("H,W", [(33, 40), (32, 41), (67, 104), (5, 105), (36, 168), (41, 169),
                                 (64, 232), (35, 233), (1, 1)])
def test_ssim_grad_strip_edges(H, W):
    announce(f"ssim strips {H}x{W}")
    import torch
    from oracle.ssim import ssim, ssim_term_grad
    from paper_2605_10760_amd import ssim_grad
    V = 2
    rng = np.random.default_rng(H * 1000 + W)
    c = rng.random((V, 3, H, W)).astype(np.float32)
    tgt = np.clip(c + 0.1 * rng.standard_normal(c.shape), 0, 1).astype(np.float32)
    ex = np.array([[0.05, 0.01], [-0.08, 0.02]], np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d_color = torch.full((V, 3, H, W), 0.5, device="cuda")
    d_exp = torch.zeros((V, 2), device="cuda")
    out = torch.zeros(1, device="cuda")
    weight = 0.2 * c.size  # gradients of order one next to the 0.5 they add to
    ssim_grad(t(c), t(tgt), d_color, t(ex), d_exp, weight, ssim_out=out)
    ref = ssim_term_grad(c, tgt, ex[:, 0], ex[:, 1], weight)
    xt = np.exp(ex[:, 0])[:, None, None, None] * c.astype(np.float64) + ex[:, 1][:, None, None, None]
    # the variances cancel to about 6e-8 of the squares, against C2 = 9e-4
    assert abs(out.item() - ssim(xt, tgt)) <= 2e-5
    got = d_color.cpu().numpy().astype(np.float64) - 0.5
    assert np.abs(got - ref["d_color"]).max() <= 1e-3 * np.abs(ref["d_color"]).max()
    ge = d_exp.cpu().numpy()
    for k, key in ((0, "d_a"), (1, "d_b")):
        scale = np.abs(ref["d_color"]).sum(axis=(1, 2, 3)).max()
        assert np.abs(ge[:, k] - ref[key]).max() <= 1e-3 * scale, key


@pytest.mark.parametrize("W", [38, 150])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_ssim_grad_non_finite_stays_local(W, bad):
    """A NaN or infinite pixel reaches the gradient within two windows of it
    (10 pixels along each axis) and nowhere else; the rest is the gradient
    without it, to the rounding of sums formed another way."""
    announce(f"ssim non-finite {bad} W={W}")
    import torch
    from paper_2605_10760_amd import ssim_grad
    H = 70
    rng = np.random.default_rng(W)
    c = rng.random((1, 3, H, W)).astype(np.float32)
    tgt = rng.random(c.shape).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    grads = []
    pj, pi = 33, min(W - 1, 101) if W > 100 else 17
    for value in (c[0, 1, pj, pi], bad):
        c[0, 1, pj, pi] = value
        d = torch.zeros((1, 3, H, W), device="cuda")
        ssim_grad(t(c), t(tgt), d, None, None, 1000.0)
        grads.append(d.cpu().numpy()[0])
    near = np.zeros((3, H, W), bool)
    near[1, pj - 10:pj + 11, max(pi - 10, 0):pi + 11] = True
    assert not np.isfinite(grads[1][near]).any()
    np.testing.assert_allclose(grads[1][~near], grads[0][~near], rtol=1e-5, atol=1e-7)


# FP32 roundings between a term and its sum: the product, the sums over a thread's
# pixel group (L1) or four rows (SSIM), the conversion of the thread's FP64 sum, the
# tree over lanes and waves, the workgroups' sums and the exposure factor (1 here)
L1_ROUNDINGS, SSIM_ROUNDINGS = 19, 23


def _sum_err(got, terms):
    """Largest error of the sums got [V] of terms [V, ...] (FP64), relative to the
    sums of their absolute values."""
    want = terms.flatten(1).sum(1)
    return float(((got.double() - want).abs() / terms.flatten(1).abs().sum(1)).max())


def test_l1_exposure_sums_of_a_large_batch():
    """Constant images, whose equal terms let the roundings of a long chain of FP32
    additions add up, in a call that gives a thread 180 of them: the exposure
    gradients against FP64 sums over the gradient images."""
    announce("l1 exposure sums of a large batch")
    import torch
    from paper_2605_10760_amd import l1_loss_grad as gpu_grad
    V, H, W = 256, 384, 640
    c = torch.full((V, 3, H, W), 0.37, device="cuda")
    tc = torch.zeros_like(c)
    ex = torch.zeros((V, 2), device="cuda")
    out = dict(d_color=torch.empty_like(c), d_depth=None, d_exposure=torch.empty_like(ex))
    for k in range(24):
        gpu_grad(c, tc, None, None, ex, 1.0 + k / 17.0, 0.0, out=out)
        g = out["d_color"][:1, :, :1, :1].double().expand(1, 3, H, W)  # every pixel's
        assert bool((out["d_color"] == out["d_color"][0, 0, 0, 0]).all())
        for i, t in enumerate((g * float(c[0, 0, 0, 0]), g)):
            assert _sum_err(out["d_exposure"][:1, i], t) <= L1_ROUNDINGS * 2.0 ** -24, (k, i)


def test_ssim_exposure_sums_of_a_large_batch():
    """The same for SSIM, in a call whose lanes march down 240 rows."""
    announce("ssim exposure sums of a large batch")
    import torch
    from paper_2605_10760_amd import ssim_grad
    V, H, W = 2800, 240, 40
    x = torch.full((V, 3, H, W), 0.71, device="cuda")
    y = torch.full((V, 3, H, W), 0.35, device="cuda")
    ex = torch.zeros((V, 2), device="cuda")
    ws = None
    for k in range(24):
        d = torch.zeros_like(x)
        de = torch.zeros_like(ex)
        ws = ssim_grad(x, y, d, exposure=ex, d_exposure=de, weight=1.0 + k / 17.0, workspace=ws)
        part = d[:4].double()
        for i, t in enumerate((part * float(x[0, 0, 0, 0]), part)):
            assert _sum_err(de[:4, i], t) <= SSIM_ROUNDINGS * 2.0 ** -24, (k, i)


# the strip edges of two to four waves again, in batches of more marches than the
# device has SIMDs (smaller calls go by one-wave strips), and one wave there
@pytest.mark.parametrize("V,H,W,nw", [(172, 33, 40, 1), (172, 5, 41, 2), (58, 37, 104, 2),
                                      (58, 33, 105, 3), (35, 64, 168, 3), (35, 41, 169, 4),
                                      (30, 35, 232, 4), (30, 33, 233, 3)])
def test_ssim_grad_strip_edges_of_batches(V, H, W, nw):
    announce(f"ssim strips of batches {V}x{H}x{W}")
    import torch
    from oracle.ssim import ssim, ssim_term_grad
    from paper_2605_10760_amd import ssim_grad
    rng = np.random.default_rng(H * 1000 + W + V)
    c = rng.random((V, 3, H, W)).astype(np.float32)
    tgt = np.clip(c + 0.1 * rng.standard_normal(c.shape), 0, 1).astype(np.float32)
    ex = np.stack([rng.normal(0, 0.1, V), rng.normal(0, 0.02, V)], 1).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d_color = torch.full((V, 3, H, W), 0.5, device="cuda")
    d_exp = torch.zeros((V, 2), device="cuda")
    out = torch.zeros(1, device="cuda")
    weight = 0.2 * c.size  # gradients of order one next to the 0.5 they add to
    ssim_grad(t(c), t(tgt), d_color, t(ex), d_exp, weight, ssim_out=out)
    xt = np.exp(ex[:, 0])[:, None, None, None] * c.astype(np.float64) + ex[:, 1][:, None, None, None]
    assert abs(out.item() - ssim(xt, tgt)) <= 2e-5
    got = d_color.cpu().numpy().astype(np.float64) - 0.5
    ge = d_exp.cpu().numpy()
    for v in (0, V // 2, V - 1):
        one = slice(v, v + 1)
        ref = ssim_term_grad(c[one], tgt[one], ex[one, 0], ex[one, 1], weight / V)
        want = ref["d_color"][0]
        assert np.abs(got[v] - want).max() <= 1e-3 * np.abs(want).max(), v
        for k, key in ((0, "d_a"), (1, "d_b")):
            assert abs(ge[v, k] - ref[key][0]) <= 1e-3 * np.abs(want).sum(), (v, key)


@pytest.mark.parametrize("V,W", [(58, 104), (35, 168), (30, 232)])
def test_ssim_grad_non_finite_stays_local_in_batches(V, W):
    """As for one view, in workgroups of two to four waves, which agree on the way
    they sum: nothing but the bad pixel's two windows in its own view changes."""
    announce(f"ssim non-finite in batches {V} W={W}")
    import torch
    from paper_2605_10760_amd import ssim_grad
    H = 38
    rng = np.random.default_rng(W)
    c = torch.from_numpy(rng.random((V, 3, H, W)).astype(np.float32)).cuda()
    tgt = torch.from_numpy(rng.random((V, 3, H, W)).astype(np.float32)).cuda()
    v, pj, pi = V // 2, 17, W - 30
    grads = []
    for bad in (False, True):
        if bad:
            c[v, 1, pj, pi] = float("nan")
        d = torch.zeros_like(c)
        ssim_grad(c, tgt, d, None, None, float(c.numel()))
        grads.append(d.clone())
    local = torch.zeros_like(c, dtype=torch.bool)
    local[v, 1, max(pj - 10, 0):pj + 11, max(pi - 10, 0):pi + 11] = True
    a, b = grads
    assert bool(torch.isfinite(a).all()) and bool((torch.isfinite(b) | local).all())
    assert bool(torch.isnan(b[v, 1, pj, pi]))
    assert float(((a - b).abs() * ~local).nan_to_num().max()) <= 1e-3 * float(a.abs().max())
    assert torch.equal(a[:v], b[:v]) and torch.equal(a[v + 1:], b[v + 1:])
