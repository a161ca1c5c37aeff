"""Rules that choose between kernels, on the host: measured points of both sides stay on the side that was faster."""
import ctypes
import os
import subprocess

import pytest

import paper_2405_18832_amd as moe
from paper_2405_18832_amd.build import CSRC, HIPCC, ROOT

SHAPES = ["big", "narrow", "fine"]


@pytest.fixture(scope="module")
def schedules(tmp_path_factory):
    """A function over (big tiles, half tiles, N, k-steps, GeLU first product) points of a 256-CU device: (shape of the units, full
    rounds, units left over, parts of each)."""
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text('''
#include <cstdio>
#include "tile_schedule.hpp"
int main() {
    int big, half, n, k, gelu;
    while (scanf("%d %d %d %d %d", &big, &half, &n, &k, &gelu) == 5) {
        const moe::TileSchedule s = moe::product_schedule(big, half, n, k, 256, gelu != 0);
        printf("%d %d %d %d\\n", static_cast<int>(s.shape), s.rounds, s.R, s.split);
    }
}''')
    subprocess.run([HIPCC, "-std=c++17", "--cuda-host-only", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    str(d / "rules.hip"), "-o", str(d / "rules")], check=True, capture_output=True)

    def ask(points):
        text = "\n".join(" ".join(str(int(v)) for v in p) for p in points)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        return [(SHAPES[v[0]], *v[1:]) for v in ([int(t) for t in line.split()] for line in out.splitlines())]
    return ask


def test_tiled_product_units(schedules):
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
    assert [s[0] for s in schedules([p for p, _ in points])] == [s for _, s in points]


def test_product_units_of_the_cases(schedules):
    """The schedules that the cases of test_gpu_edges.test_product_units are there for."""
    from test_gpu_edges import PRODUCT_UNITS
    for rows, d, f, want in PRODUCT_UNITS:
        least = moe.moe_tiled_kernel_min_rows(moe.make_shape(sum(rows), d, f, len(rows), 1, "bf16", False), rows)
        large = [r for r in rows if r >= least]
        big, half = (sum(-(-r // n) for r in large) for n in (256, 128))
        got = schedules([(big, half, f, d // 32, 0), (big, half, d, f // 32, 0)]) if large else None
        assert got == want, (rows, d, f, got)


def layer_is_few(T, d, f, E, k, dtype="bf16"):
    """Whether a layer without a mask takes the three launches of few tokens (moe::layer_is_few of the library)."""
    rule = moe.load()._ZN3moe12layer_is_fewERK9moe_shape
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.POINTER(moe.moe_shape)]
    return rule(ctypes.byref(moe.make_shape(T, d, f, E, k, dtype, True)))


def test_few_token_layers():
    # (T, d_model, d_ff, E, k), us on the general path and in three launches (256 CUs)
    faster = [(1, 2048, 8192, 128, 2),       # 36.4 32.9
              (2, 2048, 8192, 128, 2),       # 56.2 54.8
              (4, 2048, 8192, 128, 2),       # 97.3 93.7
              (1, 1024, 4096, 128, 1),       # 23.7 14.8
              (8, 1024, 4096, 128, 1),       # 33.7 31.1
              (8, 768, 3072, 64, 1),         # 28.5 26.6
              (3, 1376, 5504, 8, 1),         # 36.6 24.3
              (2, 4096, 192, 128, 1),        # 23.6 15.4
              (7, 896, 2496, 63, 1),         # 30.2 25.9
              (1, 64, 256, 8, 1)]
    slower = [(8, 256, 1024, 128, 8),        # 38.0 60.7
              (7, 640, 2560, 128, 1),        # 26.2 27.0
              (5, 256, 8192, 64, 2),         # 33.5 52.2
              (4, 512, 4096, 128, 4),        # 40.7 51.5
              (6, 512, 2048, 8, 2),          # 25.4 27.5
              (7, 160, 320, 128, 8),         # 27.8 47.1
              (4, 2176, 4352, 16, 8),        # 116 140
              (2, 2560, 5120, 16, 2),        # 44.5 48.8
              (7, 4096, 8192, 16, 1),        # 169 187
              (2, 1024, 4096, 128, 8),       # 63.5 67.4
              (8, 2048, 8192, 128, 2),
              (9, 64, 256, 8, 1)]
    assert [s for s in faster if not layer_is_few(*s)] == []
    assert [s for s in slower if layer_is_few(*s)] == []
    assert not layer_is_few(1, 64, 256, 8, 1, "f32")


def f32_is_wide(rows, E, N, K):
    """Whether an fp32 product of `rows` rows on E experts, all of them 16-byte aligned, runs in units of 32 columns (moe::f32_is_wide)."""
    rule = moe.load()._ZN3moe11f32_is_wideElliiPKvS1_S1_PKf
    rule.restype = ctypes.c_bool
    rule.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_int, ctypes.c_int] + 4 * [ctypes.c_void_p]
    return rule(rows, rows // 64 + min(E, rows), N, K, 0x1000, 0x2000, 0x3000, 0x4000)


def test_f32_wide_units():
    # (rows, experts, columns, contraction) of 256 CUs, us in units of 16 and of 32 columns
    wide = [(500, 8, 3072, 768),               # 45.4 39.0
            (752, 14, 1024, 288),              # 43.2 41.0, of the layer
            ((1 << 21) - 128, 1, 16384, 256)]  # 512 units fewer than 2^24
    narrow = [(500, 8, 768, 3072),             # 46.0 60.9
              (155, 14, 2048, 544),            # 42.3 47.4, of the layer
              ((1 << 21) - 64, 1, 16384, 256), # 2^24 units of 256 threads and more: no launch holds them
              (1 << 21, 1, 16384, 256),
              (1 << 24, 8, 2048, 512),
              ((1 << 30) - 1, 1, 1024, 256)]
    assert [s for s in wide if not f32_is_wide(*s)] == []
    assert [s for s in narrow if f32_is_wide(*s)] == []


def test_f32_wide_units_of_the_cases():
    """The fp32 cases of test_gpu_edges.py that are there for wide units run in them."""
    import test_gpu_edges as g
    T, d, f, E, k = g.F32_WIDE_LAYER.values()
    assert f32_is_wide(T * k, E, f, d) and T * k > 1024          # up to 1024 assignments the first product may sort them instead
    for K, N in g.F32_WIDE_ROUNDING:
        assert f32_is_wide(sum(g.F32_WIDE_ROWS), len(g.F32_WIDE_ROWS), N, K)
