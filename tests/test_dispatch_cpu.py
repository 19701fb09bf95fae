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
    ([1000], 1), ([300000], 1), ([1000000], 1), ([1500000], 1), ([2000000], 0), ([3000000], 0),
    ([4000000], 0), ([200000] * 8, 1), ([400000] * 8, 1), ([800000] * 8, 0), ([85000] * 48, 1),
    ([170000] * 48, 0), ([278000] * 48, 0), ([3000000] * 48, 0), ([1000000] + [100] * 63, 1),
    ([3000000] + [100] * 63, 0), ([65536] * 64, 1), ([65537] * 64, 0)])
def test_sort_without_scan_kernels(rule, views, want):
    off = [0]
    for n in views:
        off.append(off[-1] + -(-n // 2048))
    setup = f"SortTab t{{}}; t.nv = {len(views)}; const int o[] = {{{','.join(map(str, off))}}};" \
            " for (int i = 0; i <= t.nv; ++i) t.sblk_off[i] = o[i];"
    assert rule("SORT_TILE == 2048") and rule("sort_folds(t)", setup) == want
