"""The compositing kernels' two forms against each other: a call with many
tiles gives each tile (or pair of tiles) to a wave, one with few tiles gives
each tile to a workgroup of one wave per 8x8 block.  The same views rendered
in one large call and one call per view take the two forms; images, entry
counts and saved last contributors must match bit for bit, gradients to the
rounding of their sums (RERUN_TOL of the tensor's largest value: the sums
run over float atomics in no fixed order in either form)."""
import numpy as np
import pytest

from gpu_harness import (GMAP, GRAD_TOL, IMG_TOL, RERUN_TOL, announce, check_ambiguous_pixels,
                         grad_rel_err)
from oracle.render import Settings, render_backward, render_view
from synth.scenes import ROOM_HI, ROOM_LO, Scene, Views, draw_gaussians, look_at, pinhole

pytestmark = pytest.mark.gpu

PARAMS = ("d_means", "d_log_scales", "d_quats", "d_opacity_logits", "d_colors")


def _case(n, n_views, W, H):
    rng = np.random.default_rng(900 + n)
    scene = Scene(*draw_gaussians(rng, n, ROOM_LO, ROOM_HI), set_offsets=np.array([0, n], np.int64))
    vm = [look_at(rng.uniform(-1, 1, 3) * [1.5, 0.3, 1.0], rng.uniform(-1, 1, 3), 0.2)
          for _ in range(n_views)]
    return scene, Views(np.array(vm, np.float32),
                        np.array([pinhole(W, H, W / 2.0)] * n_views, np.float32),
                        np.zeros(n_views, np.int32), W, H)


# (tile, tiles per backward wave, image size): 5 views of 2,450 16x16 tiles, 65 x
# 33 = 2,145 32x16 tiles (an odd edge on both axes), 49 x 50 8x8 tiles; each
# large call passes 10,000 tiles
@pytest.mark.parametrize("tile,cols,W,H,n_views", [
    ((16, 16), 1, 784, 800, 5), ((16, 16), 2, 777, 795, 5), ((32, 16), 1, 2077, 521, 5),
    ((8, 8), 1, 391, 399, 5)])
def test_wave_and_workgroup_forms(tile, cols, W, H, n_views):
    import torch
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"forms {tile} cols {cols} {W}x{H}")
    scene, views = _case(4000, n_views, W, H)
    tiles = -(-W // tile[0]) * -(-H // tile[1])
    assert tiles <= 2500 and n_views * tiles > 10000
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    rng = np.random.default_rng(5)
    up = [torch.from_numpy((rng.choice([-1.0, 1.0], s) / s[-1]).astype(np.float32)).cuda()
          for s in ((n_views, 3, H, W), (n_views, H, W), (n_views, H, W))]
    big = Rasterizer(W, H, n_views * scene.n, n_views, tile=tile, bwd_cols=cols)
    c, d, a, state, ne = big.forward(st, vt, bg=(0.2, 0.4, 0.6), n_eval=True)
    g = big.backward(st, vt, state, *up, bg=(0.2, 0.4, 0.6))
    dbg = big.debug_export(state, n_views, n_views * scene.n, 0)
    c2, d2, a2, _ = big.forward(st, vt, bg=(0.2, 0.4, 0.6))
    assert torch.equal(c, c2) and torch.equal(d, d2) and torch.equal(a, a2)
    one = Rasterizer(W, H, scene.n, 1, tile=tile, bwd_cols=1)
    total = {k: torch.zeros_like(g[k]) for k in PARAMS}
    for k in range(n_views):
        vk = vt.select([k])
        ck, dk, ak, sk, nk = one.forward(st, vk, bg=(0.2, 0.4, 0.6), n_eval=True)
        assert torch.equal(ck[0], c[k]) and torch.equal(dk[0], d[k]) and torch.equal(ak[0], a[k])
        assert torch.equal(nk[0], ne[k])
        ek = one.debug_export(sk, 1, scene.n, 0)
        np.testing.assert_array_equal(ek["last"][0], dbg["last"][k])
        np.testing.assert_array_equal(ek["t_final"][0], dbg["t_final"][k])
        gk = one.backward(st, vk, sk, *[x[k:k + 1].contiguous() for x in up],
                          bg=(0.2, 0.4, 0.6))
        for q in PARAMS:
            total[q] += gk[q]
        pose = g["d_pose"][k]
        assert float((gk["d_pose"][0] - pose).abs().max()) <= RERUN_TOL * float(pose.abs().max())
    for q in PARAMS:
        err = float((total[q] - g[q]).abs().max())
        assert err <= RERUN_TOL * float(g[q].abs().max()), (q, err)


# 64 views of 33 sort blocks each (2112: past the limit up to which a block walks
# its view's digit counts itself), of 32 (2048: at it)
@pytest.mark.parametrize("n", [65537, 65536])
def test_sort_with_and_without_scan_kernel(n):
    """The depth order of a call on either side of the limit equals that of one
    call per view, bit for bit."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"sort forms {n}")
    W, H, n_views = 64, 48, 64
    scene, views = _case(n, n_views, W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views)
    *_, state = big.forward(st, vt)
    dbg = big.debug_export(state, n_views, n_views * n, 0)
    one = Rasterizer(W, H, n, 1)
    for k in (0, 1, 31, 63):
        *_, sk = one.forward(st, vt.select([k]))
        ek = one.debug_export(sk, 1, n, 0)
        lo, hi = int(dbg["vis_off"][k]), int(dbg["vis_off"][k + 1])
        assert hi - lo == int(ek["vis_off"][1]) > 4096
        np.testing.assert_array_equal(dbg["order"][lo:hi].astype(np.int64) - k * n,
                                      ek["order"].astype(np.int64))


# views of a set: below and from the number on which the key pass queues its pairs
@pytest.mark.parametrize("n,n_views", [(64, 5), (700, 21), (1500, 64)])
def test_key_pass_with_and_without_queue(n, n_views):
    """Splats of all sizes and shapes, most of them across or beyond the image's
    edges or the near plane, some without a finite rectangle; views of any
    scale: the same pairs are visible, with the same depth keys and rectangles,
    as in one call per view."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"key pass forms {n} {n_views}")
    W, H = 72, 40
    scene, views = _case(n, n_views, W, H)
    rng = np.random.default_rng(n)
    scene.log_scales[:] = rng.normal(-2.5, 1.5, (n, 3))
    scene.opacity_logits[:] = rng.normal(-3.0, 2.5, n)
    bad = rng.permutation(n)[:4]
    scene.means[bad[0]] = np.nan
    scene.log_scales[bad[1], 1] = 60.0
    scene.means[bad[2]] = 1e30
    scene.quats[bad[3]] = 0.0
    views.viewmats[1::3, :, :3] *= 1.7
    views.viewmats[2::3, 0, :3] *= 0.4
    views.intrinsics[::4, 0] *= 3.0
    views.intrinsics[3::4, 3] += 25.0
    views.intrinsics[2, 1] *= -1.0
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views)
    *_, state = big.forward(st, vt)
    dbg = big.debug_export(state, n_views, n_views * n, 0)
    one = Rasterizer(W, H, n, 1)
    seen = 0
    for k in range(n_views):
        *_, sk = one.forward(st, vt.select([k]))
        ek = one.debug_export(sk, 1, n, 0)
        np.testing.assert_array_equal(dbg["zkeys"][k * n:(k + 1) * n], ek["zkeys"])
        np.testing.assert_array_equal(dbg["rects"][k * n:(k + 1) * n], ek["rects"])
        seen += int(ek["vis_off"][1])
    assert 0.03 * n * n_views < seen < 0.9 * n * n_views


# views that see none, one or thousands of the pairs, blocks that end on a view's
# last pair, more blocks than the kernels over visible pairs have workgroups
@pytest.mark.parametrize("n,n_views,chunk", [(2048, 9, 64), (2049, 64, 0), (65537, 33, 64)])
def test_blocks_of_visible_pairs(n, n_views, chunk):
    """Views that see everything, some or nothing, in one call and one call each:
    the same depth order and per-tile lists."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"visible blocks {n} {n_views}")
    W, H = 64, 48
    scene, views = _case(n, n_views, W, H)
    # in front of every third view lies the whole scene, behind every other third
    # nothing: the camera is moved out of the room, looking in or away
    for k in range(n_views):
        if k % 3 != 1:
            views.viewmats[k, :, :3] = np.diag([1.0, 1.0, 1.0 if k % 3 == 0 else -1.0])
            views.viewmats[k, :, 3] = (0.0, 0.0, 12.0 if k % 3 == 0 else -12.0)
    scene.opacity_logits[:] = np.maximum(scene.opacity_logits, -1.0)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views, chunk=chunk)
    c, *_, state = big.forward(st, vt)
    dbg = big.debug_export(state, n_views, n_views * n, 0)
    one = Rasterizer(W, H, n, 1, chunk=chunk)
    for k in (0, 1, 2, 4, 5, n_views - 1):
        ck, *_, sk = one.forward(st, vt.select([k]))
        ek = one.debug_export(sk, 1, n, 0)
        lo, hi = int(dbg["vis_off"][k]), int(dbg["vis_off"][k + 1])
        assert hi - lo == int(ek["vis_off"][1])
        assert hi - lo == (n if k % 3 == 0 else hi - lo if k % 3 == 1 else 0)
        np.testing.assert_array_equal(dbg["order"][lo:hi].astype(np.int64) - k * n,
                                      ek["order"].astype(np.int64))
        np.testing.assert_array_equal(c[k].cpu().numpy(), ck[0].cpu().numpy())


# metres from the origin: a centimetre is 2 (at 50 km), 10 and 80 FP32 steps
@pytest.mark.parametrize("far", [5e4, 1e4, 1e3])
def test_key_pass_far_from_the_origin(far):
    """Small splats across the edges of views far from the origin, where the
    rotation and the translation of a mean cancel: the queued key pass (five views
    or more of a set) sees the same pairs as one call per view, bit for bit."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"key pass far {far}")
    W, H, n_views, n, f = 72, 40, 6, 60000, 600.0
    rng = np.random.default_rng(int(far))
    intr = np.array([f, f, W / 2.0, H / 2.0])
    vm, means = [], []
    for k in range(n_views):
        c = far * rng.uniform(0.3, 1.0, 3) * rng.choice([-1.0, 1.0], 3)
        T = look_at(c, c + rng.normal(size=3), 0.3, 0.4)
        vm.append(T)
        # this view's share of the splats, on its image's edges
        m = n // n_views
        z = rng.uniform(0.25, 1.0, m)
        u, v = rng.uniform(0, W, m), rng.uniform(0, H, m)
        e = rng.integers(0, 4, m)
        near = rng.uniform(-2.5, 2.5, m)
        u = np.where(e == 0, near, np.where(e == 1, W + 8 + near, u))  # 72 = 4.5 tiles
        v = np.where(e == 2, near, np.where(e == 3, H + 8 + near, v))
        p = np.stack([(u - intr[2]) / f * z, (v - intr[3]) / f * z, z], 1)
        means.append((p - T[:, 3]) @ T[:, :3])
    scene = Scene(*draw_gaussians(rng, n, ROOM_LO, ROOM_HI), set_offsets=np.array([0, n], np.int64))
    scene.means[:] = np.concatenate(means)
    scene.log_scales[:] = rng.normal(-8.5, 0.3, (n, 3))
    scene.opacity_logits[:] = 1.0
    views = Views(np.array(vm, np.float32), np.array([intr] * n_views, np.float32),
                  np.zeros(n_views, np.int32), W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views)
    *_, state = big.forward(st, vt)
    dbg = big.debug_export(state, n_views, n_views * n, 0)
    one = Rasterizer(W, H, n, 1)
    seen = 0
    for k in range(n_views):
        *_, sk = one.forward(st, vt.select([k]))
        ek = one.debug_export(sk, 1, n, 0)
        np.testing.assert_array_equal(dbg["zkeys"][k * n:(k + 1) * n], ek["zkeys"])
        np.testing.assert_array_equal(dbg["rects"][k * n:(k + 1) * n], ek["rects"])
        seen += int(ek["vis_off"][1])
    assert 0.2 * n < seen < 0.95 * n


@pytest.mark.parametrize("z_near", [-8.0, 0.0])
def test_key_pass_with_any_near_plane(z_near):
    """A near plane at or behind the camera: the queued key pass keeps the pairs
    that one call per view keeps, those of negative depth among them."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"key pass near plane {z_near}")
    W, H, n_views, n = 72, 40, 6, 3000
    scene, views = _case(n, n_views, W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views)
    *_, state = big.forward(st, vt, z_near=z_near)
    dbg = big.debug_export(state, n_views, n_views * n, 0)
    one = Rasterizer(W, H, n, 1)
    behind = 0
    for k in range(n_views):
        *_, sk = one.forward(st, vt.select([k]), z_near=z_near)
        ek = one.debug_export(sk, 1, n, 0)
        np.testing.assert_array_equal(dbg["zkeys"][k * n:(k + 1) * n], ek["zkeys"])
        np.testing.assert_array_equal(dbg["rects"][k * n:(k + 1) * n], ek["rects"])
        vis = ek["zkeys"] != 0xFFFFFFFF
        behind += int((ek["zkeys"][vis].view(np.float32) < 0).sum())
    assert (behind > 0) == (z_near < 0)


# one view of the most blocks whose sort goes without scan kernels, and of one more
@pytest.mark.parametrize("n", [1000 * 2048, 1000 * 2048 + 1])
def test_sort_of_one_large_view(n):
    """A large view that sees everything: its depth order is the stable order of its
    depth keys, with and without scan kernels."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"sort one view {n}")
    W, H = 64, 48
    rng = np.random.default_rng(n)
    means = np.stack([rng.uniform(-1, 1, n), rng.uniform(-1, 1, n), rng.uniform(3, 9, n)], 1)
    scene = Scene(means, np.full((n, 3), -6.0), np.tile([1.0, 0.0, 0.0, 0.0], (n, 1)),
                  np.ones(n), rng.random((n, 3)), set_offsets=np.array([0, n], np.int64))
    vm = np.concatenate([np.eye(3), np.zeros((3, 1))], 1)[None]
    views = Views(vm.astype(np.float32), np.array([pinhole(W, H, W / 2.0)], np.float32),
                  np.zeros(1, np.int32), W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    r = Rasterizer(W, H, n, 1, max_instances=3 * n)
    *_, state = r.forward(st, vt)
    e = r.debug_export(state, 1, n, 0)
    assert int(e["vis_off"][1]) == n
    np.testing.assert_array_equal(e["order"], np.argsort(e["zkeys"], kind="stable"))


# the other tile shapes, and the two of eight blocks with views of 1,225 tiles, up
# to which their backward takes a workgroup per tile
@pytest.mark.parametrize("tile,cols,W,H,n_views", [
    ((32, 16), 1, 1113, 555, 9), ((16, 32), 1, 555, 1111, 9), ((16, 8), 2, 779, 400, 5),
    ((8, 16), 2, 397, 783, 5), ((32, 8), 1, 1561, 397, 5)])
def test_forms_of_every_tile_shape(tile, cols, W, H, n_views):
    test_wave_and_workgroup_forms(tile, cols, W, H, n_views)


# entries per lane of the forward and the backward, tiles per backward wave
@pytest.mark.parametrize("fb,bb,cols", [(1, 1, 1), (2, 2, 1), (2, 4, 1), (1, 1, 2), (1, 2, 2),
                                        (2, 4, 2)])
def test_one_wave_options_against_oracle(fb, bb, cols):
    """A call of more tiles than go to workgroups, so that the plan's options
    choose the one-wave kernels of either direction: images, entry counts and the
    gradients of two views against the oracle."""
    import torch
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"one-wave options fb={fb} bb={bb} cols={cols}")
    W, H, n_views, n = 203, 205, 64, 20000
    assert n_views * 13 * 13 * 4 > 40000  # 8x8 blocks of the call
    scene, views = _case(n, n_views, W, H)
    scene.opacity_logits -= 2.0  # pixels walk up to 540 entries: several rounds
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    r = Rasterizer(W, H, n_views * n, n_views, fwd_batch=fb, bwd_batch=bb, bwd_cols=cols)
    c, d, a, state, ne = r.forward(st, vt, n_eval=True)
    c2, d2, a2, _ = r.forward(st, vt)
    assert torch.equal(c, c2) and torch.equal(d, d2) and torch.equal(a, a2)
    ids = (7, 40)
    g = {k: {q: x[k].cpu().numpy() for q, x in (("color", c), ("depth", d), ("alpha", a),
                                                ("n_eval", ne))} for k in ids}
    rng = np.random.default_rng(12)
    up = [np.zeros((n_views,) + s, np.float32) for s in ((3, H, W), (H, W), (H, W))]
    for k in ids:
        o = render_view(scene, views, k, Settings())
        ok = ~o["ambiguous"]
        assert o["last"].max() > 256
        zmax = max(1.0, float(np.max(o["setup"]["pr"]["z"], initial=0.0)))
        assert np.abs(g[k]["color"] - o["color"])[:, ok].max() <= IMG_TOL
        assert np.abs(g[k]["alpha"] - o["alpha"])[ok].max() <= IMG_TOL
        assert np.abs(g[k]["depth"] - o["depth"])[ok].max() <= IMG_TOL * zmax
        np.testing.assert_array_equal(g[k]["n_eval"][ok], o["n_eval"][ok])
        per_view = {q: {k: g[k][q]} for q in g[k]}
        check_ambiguous_pixels(per_view, k, o, views, Settings(), zmax)
        for u in up:
            u[k] = rng.normal(size=u[k].shape) * ok
    got = r.backward(st, vt, state, *[torch.from_numpy(u).cuda() for u in up])
    ref = render_backward(scene, views, *up, view_ids=ids)
    for k_gpu, k_ref in GMAP.items():
        e_inf, e_2 = grad_rel_err(got[k_gpu].cpu().numpy(), ref[k_ref])
        assert e_inf <= GRAD_TOL and e_2 <= GRAD_TOL, (k_gpu, e_inf, e_2)


# as test_blocks_of_visible_pairs: chunks that end on a view's last pair, views that
# see none of their pairs
@pytest.mark.parametrize("n,n_views,chunk", [(2048, 9, 64), (2049, 64, 0), (20011, 33, 100)])
def test_tile_lists_of_visible_pairs(n, n_views, chunk):
    """Views that see everything, some or nothing, in one call and one call each:
    the same rectangles, tile ranges and lists."""
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"visible lists {n} {n_views} {chunk}")
    W, H = 70, 53
    scene, views = _case(n, n_views, W, H)
    for k in range(n_views):
        if k % 3 != 1:
            views.viewmats[k, :, :3] = np.diag([1.0, 1.0, 1.0 if k % 3 == 0 else -1.0])
            views.viewmats[k, :, 3] = (0.0, 0.0, 12.0 if k % 3 == 0 else -12.0)
    scene.opacity_logits[:] = np.maximum(scene.opacity_logits, -1.0)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    big = Rasterizer(W, H, n_views * n, n_views, chunk=chunk)
    *_, state = big.forward(st, vt)
    counts = big.poll(state)
    dbg = big.debug_export(state, n_views, n_views * n, counts["instances"])
    T = dbg["TX"] * dbg["TY"]
    one = Rasterizer(W, H, n, 1, chunk=chunk)
    total = 0
    for k in range(n_views):
        *_, sk = one.forward(st, vt.select([k]))
        ck = one.poll(sk)
        total += ck["instances"]
        if k >= 7 and k != n_views - 1:
            continue
        ek = one.debug_export(sk, 1, n, ck["instances"])
        np.testing.assert_array_equal(dbg["rects"][k * n:(k + 1) * n], ek["rects"])
        lens = lambda r: (r[:, 1] - r[:, 0]).astype(np.int64)
        rg = dbg["ranges"][k * T:(k + 1) * T]
        np.testing.assert_array_equal(lens(rg), lens(ek["ranges"]))
        assert lens(rg).sum() == ck["instances"]
        for t in np.nonzero(lens(rg))[0]:
            np.testing.assert_array_equal(dbg["inst"][rg[t, 0]:rg[t, 1]].astype(np.int64) - k * n,
                                          ek["inst"][ek["ranges"][t, 0]:ek["ranges"][t, 1]])
        if k % 3 != 1:
            assert (ck["instances"] > n) == (k % 3 == 0) and ck["instances"] >= 0
    assert total == counts["instances"]


def test_autotune_of_a_small_call():
    """Options of the one-wave kernels are not chosen for a call whose tiles go to
    workgroups, where they change nothing but the noise of a timing."""
    from paper_2605_10760_amd import SceneTensors, ViewTensors, autotune
    announce("autotune small call")
    scene, views = _case(3000, 2, 150, 90)
    best = autotune(SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views))
    assert (best["fwd_batch"], best["bwd_batch"], best["bwd_cols"]) == (1, 1, 1)
    assert best["ms"] > 0
