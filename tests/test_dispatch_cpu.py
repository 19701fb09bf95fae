"""The host rules that choose between two forms of a kernel, compiled from the
library's own header for the host: on either side of each line the form that
was measured faster there (no GPU needed)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_10760_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(expression) evaluated in namespace gsr, as an int."""
    d = tmp_path_factory.mktemp("rules")

    def run(expr, setup=""):
        src, exe = str(d / "r.cpp"), str(d / "r")
        open(src, "w").write('#include <cstdio>\n#include "internal.h"\nusing namespace gsr;\n'
                             f'int main() {{ {setup} std::printf("%d", (int)({expr})); }}\n')
        subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, src, "-o", exe],
                       check=True, capture_output=True, text=True)
        return int(subprocess.run([exe], check=True, capture_output=True, text=True).stdout)

    return run


# pairs of each view; whether the sort goes without scan kernels
@pytest.mark.parametrize("views,want", [
    ([1000], 1), ([300000], 1), ([1000000], 1), ([2000000], 1), ([2300000], 0), ([3000000], 0),
    ([4000000], 0), ([1000000] * 3, 1), ([1000000] * 4, 0), ([500000] * 8, 1), ([200000] * 8, 1), ([400000] * 8, 1), ([800000] * 8, 0), ([85000] * 48, 1),
    ([170000] * 48, 0), ([278000] * 48, 0), ([3000000] * 48, 0), ([1000000] + [100] * 63, 1),
    ([3000000] + [100] * 63, 0), ([65536] * 64, 1), ([65537] * 64, 0)])
def test_sort_without_scan_kernels(rule, views, want):
    off = [0]
    for n in views:
        off.append(off[-1] + -(-n // 2048))
    setup = f"SortTab t{{}}; t.nv = {len(views)}; const int o[] = {{{','.join(map(str, off))}}};" \
            " for (int i = 0; i <= t.nv; ++i) t.sblk_off[i] = o[i];"
    assert rule("SORT_TILE == 2048") and rule("sort_folds(t)", setup) == want


# views, width, height; most steps of a march and least waves of the call
@pytest.mark.parametrize("nv,W,H,steps,waves", [
    (1, 16, 16, 4, 12), (1, 64, 64, 4, 90), (1, 320, 240, 5, 700), (16, 64, 64, 5, 700),
    (300, 32, 32, 7, 1800), (1, 40, 2000, 5, 700), (1, 640, 480, 9, 900)])
def test_ssim_marches_of_small_calls(rule, nv, W, H, steps, waves):
    setup = f"const SsimShape s = ssim_shape({nv}, {W}, {H});" \
            f" const int n = 3 * {nv} * s.strips * (({H} + s.rows - 1) / s.rows) * s.nw;"
    assert rule("s.rows / 4 + 3", setup) <= steps
    assert waves <= rule("n", setup) <= 2048
    # its columns and rows are covered, and the workspace holds its partials
    assert rule("s.strips * ss_out(s.nw)", setup) >= W
    from paper_2605_10760_amd import _lib
    import ctypes as C
    nb = C.c_size_t()
    assert _lib.load().gsr_ssim_workspace_bytes(nv, W, H, C.byref(nb)) == _lib.GSR_OK
    assert nb.value >= 12 * rule("n / s.nw", setup) + 4 * nv


# the batches whose strips the GPU tests probe: waves of a workgroup
@pytest.mark.parametrize("nv,W,H,nw", [
    (172, 40, 33, 1), (172, 41, 5, 2), (58, 104, 37, 2), (58, 105, 33, 3), (35, 168, 64, 3),
    (35, 169, 41, 4), (30, 232, 35, 4), (30, 233, 33, 3), (58, 104, 38, 2), (35, 168, 38, 3),
    (30, 232, 38, 4), (48, 640, 480, 4)])
def test_ssim_strips_of_batches(rule, nv, W, H, nw):
    assert rule("s.nw", f"const SsimShape s = ssim_shape({nv}, {W}, {H});") == nw
    assert rule("s.rows >= SS_T", f"const SsimShape s = ssim_shape({nv}, {W}, {H});")


# 8x8 blocks of a tile, tiles, whether a workgroup takes a tile: the faster form of
# the two as measured (views of 640x480 or 1200x680), and the calls that the GPU
# tests render both ways
@pytest.mark.parametrize("blocks,tiles,fwd,bwd", [
    (4, 48, 1, 1), (4, 1200, 1, 1), (4, 3225, 1, 0), (4, 9600, 1, 0), (4, 19200, 0, 0),
    (8, 150, 1, 1), (8, 1200, 1, 1), (8, 1634, 1, 0), (8, 3600, 1, 0), (8, 9600, 0, 0),
    (2, 2400, 1, 1), (2, 4800, 1, 0), (2, 14400, 0, 0), (1, 1200, 1, 1), (1, 4800, 1, 0),
    (1, 9600, 0, 0), (1, 28800, 0, 0),
    (4, 2450, 1, 1), (4, 12250, 0, 0), (8, 2145, 1, 0), (8, 10725, 0, 0), (1, 2450, 1, 1),
    (1, 12250, 0, 0), (8, 1225, 1, 1), (8, 11025, 0, 0), (2, 2450, 1, 1), (2, 12250, 0, 0),
    (4, 10816, 0, 0)])
def test_compositing_by_workgroup(rule, blocks, tiles, fwd, bwd):
    assert rule(f"fwd_by_workgroup({tiles}, {blocks})") == fwd
    assert rule(f"bwd_by_workgroup({tiles}, {blocks})") == bwd


@pytest.mark.parametrize("pairs,want", [(400000, 64), (800000, 128), (1000000, 128),
                                        (1200000, 128), (1500000, 256), (3000000, 256)])
def test_chunk_of_an_open_plan(rule, pairs, want):
    assert rule(f"auto_chunk({pairs})") == want


@pytest.mark.parametrize("sh,views,want", [(0, 1, 1), (0, 64, 1), (1, 1, 0), (1, 64, 0), (2, 1, 0),
                                           (2, 4, 0), (2, 6, 1), (2, 64, 1), (3, 1, 0), (3, 8, 0),
                                           (3, 12, 0), (3, 20, 1), (3, 64, 1)])
def test_projection_backward_loops(rule, sh, views, want):
    assert rule(f"bwd_by_two_loops({sh}, {views})") == want
