"""The projection backward's two ways through a set's views against each other:
one call with views in all directions, where a lane takes the views that see
its own Gaussian, and one call per view, where a wave takes the views in
turn.  Gradients agree to the rounding of their sums (RERUN_TOL of the
tensor's largest value), and a second backward of the same call finds the
per-pair rows and the pose sums cleared."""
import numpy as np
import pytest

from gpu_harness import RERUN_TOL, announce
from synth.scenes import ROOM_HI, ROOM_LO, Scene, Views, draw_gaussians, look_at, pinhole

pytestmark = pytest.mark.gpu

PARAMS = ("d_means", "d_log_scales", "d_quats", "d_opacity_logits", "d_colors")


# one Gaussian, a partial and a full wave and workgroup, several workgroups of
# two sets; up to the largest number of views
@pytest.mark.parametrize("sizes,n_views,sh", [
    ((1,), 3, 0), ((63, 64), 64, 3), ((257,), 33, 1), ((256, 1), 20, 2), ((700, 300), 64, 0)])
def test_views_in_turn_and_own_views(sizes, n_views, sh):
    import torch
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce(f"backward views {sizes} {n_views} sh {sh}")
    rng = np.random.default_rng(sum(sizes) + n_views)
    n, W, H = sum(sizes), 64, 48
    scene = Scene(*draw_gaussians(rng, n, ROOM_LO, ROOM_HI, sh_degree=sh),
                  set_offsets=np.cumsum((0,) + sizes).astype(np.int64), sh_degree=sh)
    vm = [look_at(rng.uniform(-0.5, 0.5, 3), rng.uniform(-1, 1, 3) * [3.0, 1.5, 2.0], 0.2)
          for _ in range(n_views)]
    # the last set sees two views of three
    vs = np.where(np.arange(n_views) % 3 == 0, 0, len(sizes) - 1).astype(np.int32)
    views = Views(np.array(vm, np.float32),
                  np.array([pinhole(W, H, W / 2.0)] * n_views, np.float32), vs, W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    up = [torch.from_numpy(rng.choice([-1.0, 1.0], s).astype(np.float32)).cuda()
          for s in ((n_views, 3, H, W), (n_views, H, W), (n_views, H, W))]
    big = Rasterizer(W, H, n_views * n, n_views)
    *_, state = big.forward(st, vt)
    runs = [{k: v.clone() for k, v in big.backward(st, vt, state, *up).items()} for _ in range(2)]
    one = Rasterizer(W, H, n, 1)
    total = {k: torch.zeros_like(runs[0][k]) for k in PARAMS + ("d_pose",)}
    for k in range(n_views):
        vk = vt.select([k])
        *_, sk = one.forward(st, vk)
        gk = one.backward(st, vk, sk, *[x[k:k + 1].contiguous() for x in up])
        for q in PARAMS:
            total[q] += gk[q]
        total["d_pose"][k] = gk["d_pose"][0]
    for g in runs:
        for q in PARAMS + ("d_pose",):
            err = float((total[q] - g[q]).abs().max())
            assert err <= RERUN_TOL * float(total[q].abs().max()), (q, err)


def test_pose_sums_of_own_views():
    """Two views side by side, each seeing every other Gaussian of one workgroup: a
    lane takes its own view, and the views' translation gradients are the sums of
    their Gaussians' mean gradients (unit rotations: the very same numbers) to the
    one rounding of the result."""
    import torch
    from paper_2605_10760_amd import Rasterizer, SceneTensors, ViewTensors
    announce("backward pose sums of own views")
    rng = np.random.default_rng(77)
    n, W, H = 256, 64, 48
    scene = Scene(*draw_gaussians(rng, n, (-0.9, -0.6, 2.0), (0.9, 0.6, 3.0)),
                  set_offsets=np.array([0, n], np.int64))
    scene.log_scales[:] = rng.normal(-3.5, 0.2, (n, 3))
    scene.opacity_logits[:] = 1.0
    scene.means[1::2, 0] += 50.0
    vm = np.zeros((2, 3, 4), np.float32)
    vm[:, [0, 1, 2], [0, 1, 2]] = 1.0
    vm[1, 0, 3] = -50.0
    views = Views(vm, np.array([pinhole(W, H, W / 2.0)] * 2, np.float32), np.zeros(2, np.int32),
                  W, H)
    st, vt = SceneTensors.from_numpy(scene), ViewTensors.from_numpy(views)
    gc = torch.linspace(-1.0, 1.0, W, device="cuda").expand(2, 3, H, W).contiguous()
    gd = torch.full((2, H, W), 3.0, device="cuda")
    r = Rasterizer(W, H, 2 * n, 2)
    *_, state = r.forward(st, vt)
    assert r.poll(state)["visible_pairs"] == n
    g = r.backward(st, vt, state, gc, gd)
    for v in range(2):
        want = g["d_means"][v::2].double().sum(0)
        err = (g["d_pose"][v, :3].double() - want).abs() / want.abs()
        assert float(err.max()) <= 1.001 * 2.0 ** -24, (v, err.tolist())


# the degrees and numbers of views on either side of the line between one loop for
# both ways and a loop for each
@pytest.mark.parametrize("sizes,n_views,sh", [
    ((300,), 1, 3), ((257,), 12, 3), ((257,), 13, 3), ((320,), 4, 2), ((320,), 5, 2),
    ((63, 64), 64, 1)])
def test_one_loop_and_two(sizes, n_views, sh):
    test_views_in_turn_and_own_views(sizes, n_views, sh)
