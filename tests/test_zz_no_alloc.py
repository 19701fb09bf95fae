"""The allocation-free seeding entry point (gsr_seed_noalloc) against
gsr_seed through the C ABI: identical rows and count on two calls in a row,
the second on a smaller keyframe (the library-held block counts keep the
first call's contents), plus its size and argument checks."""
import ctypes as C

import numpy as np
import pytest

from gpu_harness import announce
from synth.scenes import look_at, slanted_depth

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rows(cap):
    import torch
    return dict(means=torch.full((cap, 3), -7.0, device="cuda"),
                log_scales=torch.full((cap, 3), -7.0, device="cuda"),
                quats=torch.full((cap, 4), -7.0, device="cuda"),
                opacity_logits=torch.full((cap,), -7.0, device="cuda"),
                colors=torch.full((cap, 3), -7.0, device="cuda"))


@pytest.mark.parametrize("shape", [((680, 1200), 1, (97, 131), 1), ((480, 640), 2, (37, 53), 3)])
def test_seed_noalloc_matches_seed(shape):
    (H1, W1), s1, (H2, W2), s2 = shape
    import torch
    from paper_2605_10760_amd import seed, seed_noalloc
    rng = np.random.default_rng(70 + s1)
    n_dev = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    for k, (H, W, stride) in enumerate(((H1, W1, s1), (H2, W2, s2))):
        announce(f"seed_noalloc call {k}: {H}x{W} stride {stride}")
        depth, _, intr = slanted_depth(rng, 1, W, H, f=0.5 * W, hole_frac=0.03)
        col = rng.random((3, H, W)).astype(np.float32)
        vm = look_at(np.array([0.4, -0.1, -1.5]), (0.0, 0.0, 1.0), 0.1).astype(np.float32)
        dt, ct, vt, it = _t(depth[0]), _t(col), _t(vm), _t(intr[0])
        ref = seed(dt, ct, vt, it, stride=stride, opacity_logit=-0.7)
        cap = ((W + stride - 1) // stride) * ((H + stride - 1) // stride)
        rows = _rows(cap)
        seed_noalloc(dt, ct, vt, it, rows, n_dev, stride=stride, opacity_logit=-0.7)
        torch.cuda.synchronize()
        n = int(n_dev.item())
        assert n == ref["means"].shape[0] > 0
        for key in rows:
            # the same kernels on the same inputs: bit-identical rows
            assert torch.equal(rows[key][:n], ref[key]), key
            # nothing is written past the count
            assert bool((rows[key][n:] == -7.0).all()), key


def test_seed_noalloc_capacity_and_args():
    announce("seed_noalloc capacity / args")
    import torch
    from paper_2605_10760_amd import _lib
    lib = _lib.load()
    H, W = 9, 11
    d = _t(np.full((H, W), 2.0, np.float32))
    col = _t(np.zeros((3, H, W), np.float32))
    vm = _t(np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32))
    intr = _t(np.array([10.0, 10.0, 5.5, 4.5], np.float32))
    rows = _rows(4)
    n_dev = torch.zeros(1, dtype=torch.int64, device="cuda")
    p = [rows[k].data_ptr() for k in ("means", "log_scales", "quats", "opacity_logits", "colors")]
    # a capacity below the count: the count is still reported, 4 rows written
    st = lib.gsr_seed_noalloc(d.data_ptr(), col.data_ptr(), vm.data_ptr(), intr.data_ptr(), W, H,
                              1, 0.0, 4, *p, n_dev.data_ptr(), None)
    torch.cuda.synchronize()
    assert st == _lib.GSR_OK and int(n_dev.item()) == H * W
    # a grid beyond the library-held buffer is refused before any launch
    big = 1 << 13
    st = lib.gsr_seed_noalloc(d.data_ptr(), col.data_ptr(), vm.data_ptr(), intr.data_ptr(), big,
                              big // 2 + 1, 1, 0.0, 4, *p, n_dev.data_ptr(), None)
    assert st == _lib.GSR_E_CAPACITY
    st = lib.gsr_seed_noalloc(d.data_ptr(), col.data_ptr(), vm.data_ptr(), intr.data_ptr(), W, H,
                              1, 0.0, 4, *p, None, None)
    assert st == _lib.GSR_E_INVALID_ARG


@pytest.mark.parametrize("shape", [(1023, 1025, 1), (1025, 1025, 1), (33, 63, 2)])
def test_seed_counts_around_the_scan_size(shape):
    """Up to 4096 blocks of 256 grid points each block sums the counts before
    it, beyond them a scan kernel runs: the same rows in grid order on both
    sides of the line, with a hole every seventh point, from both entry
    points."""
    import torch
    from paper_2605_10760_amd import seed, seed_noalloc
    H, W, stride = shape
    announce(f"seed scan size {H}x{W} stride {stride}")
    js, is_ = np.arange(0, H, stride), np.arange(0, W, stride)
    depth = np.full((H, W), 2.0, np.float32)
    grid = np.arange(js.size * is_.size).reshape(js.size, is_.size)
    sub = depth[::stride, ::stride]
    sub[grid % 7 == 3] = 0.0
    col = np.zeros((3, H, W), np.float32)
    col[0] = np.arange(H)[:, None]
    col[1] = np.arange(W)[None]
    vm = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    intr = np.array([100.0, 100.0, W / 2.0, H / 2.0], np.float32)
    want = np.argwhere(depth[::stride, ::stride] > 0) * stride
    got = seed(_t(depth), _t(col), _t(vm), _t(intr), stride=stride)
    np.testing.assert_array_equal(got["colors"][:, :2].cpu().numpy(), want.astype(np.float32))
    rows = _rows(grid.size)
    n_dev = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    seed_noalloc(_t(depth), _t(col), _t(vm), _t(intr), rows, n_dev, stride=stride)
    torch.cuda.synchronize()
    assert int(n_dev.item()) == want.shape[0]
    for key in rows:
        assert torch.equal(rows[key][:want.shape[0]], got[key]), key


def test_calls_that_wait_are_refused_under_capture():
    """seed, prune and dedup return results to the host: on a stream under capture
    they are refused before anything is enqueued, so the capture goes on without
    them and later eager calls are whole."""
    announce("refused under capture")
    import torch
    from paper_2605_10760_amd import GsrError, SceneTensors, dedup, prune, seed
    rng = np.random.default_rng(8)
    n, H, W = 700, 37, 53
    depth, _, intr = slanted_depth(rng, 1, W, H, f=0.5 * W, hole_frac=0.03)
    col = rng.random((3, H, W)).astype(np.float32)
    vm = look_at(np.array([0.4, -0.1, -1.5]), (0.0, 0.0, 1.0), 0.1).astype(np.float32)
    dt, ct, vt, it = _t(depth[0]), _t(col), _t(vm), _t(intr[0])
    f = lambda *s: _t(rng.normal(-1.0, 1.0, s).astype(np.float32))
    scene = SceneTensors(f(n, 3), f(n, 3) - 3.0, f(n, 4), f(n) * 4.0, f(n, 3),
                         np.array([0, 300, n], np.int64))
    calls = [lambda: seed(dt, ct, vt, it, stride=2),
             lambda: prune(scene, 0.3),
             lambda: dedup(scene.means, scene.means, scene.log_scales, None, None, None, 0.05, 1.0,
                           table_slots=1 << 16)]
    want = [c() for c in calls]
    x = torch.zeros(64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for c in calls:
            with pytest.raises(GsrError) as e:
                c()
            assert "GSR_E_DEVICE" in str(e.value)
        x.add_(1.0)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((x == k + 1).all())
        got = [c() for c in calls]
        assert all(torch.equal(got[0][q], want[0][q]) for q in want[0])
        np.testing.assert_array_equal(got[1].set_offsets, want[1].set_offsets)
        assert torch.equal(got[1].means, want[1].means) and 0 < got[1].n < n
        assert torch.equal(got[2][0], want[2][0]) and got[2][1] == want[2][1] > 0
