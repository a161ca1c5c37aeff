"""Rules that choose between kernels, on the host: measured points of both sides stay on the side that was faster."""
import os
import subprocess

import pytest

from paper_2405_18832_amd.build import CSRC, HIPCC, ROOT

SHAPES = ["big", "narrow", "fine"]


@pytest.fixture(scope="module")
def unit_shapes(tmp_path_factory):
    """A function over (big tiles, half tiles, N, k-steps, GeLU first product) points of a 256-CU device."""
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text('''
#include <cstdio>
#include "tile_schedule.hpp"
int main() {
    long big, half; int n, k, gelu;
    while (scanf("%ld %ld %d %d %d", &big, &half, &n, &k, &gelu) == 5)
        printf("%d\\n", static_cast<int>(moe::tiled_product_units(big, half, n, k, 256, gelu != 0)));
}''')
    subprocess.run([HIPCC, "-std=c++17", "--cuda-host-only", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    str(d / "rules.hip"), "-o", str(d / "rules")], check=True, capture_output=True)

    def ask(points):
        text = "\n".join(" ".join(str(int(v)) for v in p) for p in points)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        return [SHAPES[int(v)] for v in out.split()]
    return ask


def test_tiled_product_units(unit_shapes):
    # (row tiles of 256 and of 128 rows, columns, 32-k steps, GeLU first product), the faster side and us of the two
    points = [((8, 16, 3072, 24, 0), "narrow"),      # 39 big -> 31
              ((8, 16, 3072, 24, 1), "narrow"),      # 44 fine -> 36
              ((10, 20, 2048, 64, 0), "narrow"),     # 55 big -> 45
              ((20, 40, 1024, 96, 0), "narrow"),     # 70 big -> 61
              ((12, 24, 2048, 128, 0), "narrow"),    # 89 big -> 81
              ((6, 12, 3072, 96, 0), "big"),         # 57 big, 63 narrow (140 rows)
              ((4, 8, 4608, 72, 0), "big"),          # 62 big, 64 narrow
              ((6, 12, 3072, 96, 1), "fine"),        # 57 fine, 65 narrow
              ((8, 16, 2304, 63, 1), "fine"),        # narrow 1.14 of fine
              ((4, 8, 5632, 96, 1), "fine"),         # 78 fine, 83 narrow
              ((16, 32, 1152, 144, 1), "fine"),      # 74 fine, 79 big
              ((15, 30, 1152, 171, 1), "fine"),      # 82 fine, 95 big
              ((16, 32, 1152, 144, 0), "big"),
              ((12, 24, 1536, 131, 1), "fine"),      # 70 fine, 79 big
              ((16, 32, 2048, 256, 1), "big"),       # half a round of big units
              ((4, 8, 3072, 24, 0), "fine")]         # at most one round
    assert unit_shapes([p for p, _ in points]) == [s for _, s in points]
