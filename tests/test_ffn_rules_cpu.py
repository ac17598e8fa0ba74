"""The rules that choose the expert FFN's kernels (csrc/ffn_rules.hpp), built by a plain C++ compiler, at both sides of their
lines and against times that were measured there."""
import shutil
import subprocess

import pytest

from paper_2602_21140_amd import build
from test_gpu_few_rows import CASES

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

DRIVER = """
#include <iostream>
#include "ffn_rules.hpp"
int main() {
  revive::FfnSizes f;
  while (std::cin >> f.P >> f.H >> f.I >> f.I_shared >> f.N >> f.T)
    if (!revive::takes_stream(f)) std::cout << "none\\n";
    else std::cout << revive::stream_form(f) << '\\n';
}
"""
TALL, FULL, HALF = "0", "1", "2"  # 128 rows x 128 columns, 64 x 64, 64 x 32


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + build.CSRC, str(d / "driver.cpp"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def run(calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        return subprocess.run([str(d / "driver")], input=text, check=True, capture_output=True, text=True).stdout.split()

    return run


# (P, H, I, I_shared, routed rows, tokens of the shared expert): us of the FFN with each form, other data in the caches
FORMS = {
    (384, 2368, 1984, 1984, 7508, 3754): (1677.6, 1779.9, 1860.0), (288, 1088, 960, 960, 5124, 732): (359.5, 379.8, 393.5),
    (384, 1280, 1152, 0, 7350, 0): (613.2, 657.1, 679.9), (240, 3456, 512, 0, 3648, 0): (406.1, 452.8, 469.6),
    (288, 2112, 576, 576, 4000, 1000): (364.3, 391.3, 410.8), (216, 576, 1088, 0, 2880, 0): (141.7, 155.6, 160.4),
    (240, 5568, 1216, 0, 4575, 0): (1618.2, 1701.1, 1780.5), (144, 1408, 1728, 1728, 1845, 615): (360.5, 394.0, 409.9),
    (192, 5696, 512, 1024, 2875, 575): (648.4, 702.3, 739.5), (320, 2176, 1408, 0, 5925, 0): (948.0, 1034.5, 1094.4),
    (216, 1856, 896, 3584, 3262, 1631): (467.3, 512.2, 541.8), (216, 2560, 1792, 7168, 3152, 788): (1041.3, 1123.3, 1180.6),
    (384, 640, 512, 2048, 5076, 1692): (181.3, 192.5, 199.9), (192, 4928, 640, 2560, 2652, 884): (701.6, 788.9, 822.5),
    (20, 6848, 128, 256, 312, 104): (136.1, 70.8, 65.7), (24, 1280, 512, 2048, 316, 316): (78.0, 54.5, 52.6),
    (80, 256, 832, 1664, 1100, 550): (61.2, 45.0, 46.6), (20, 1408, 1280, 1280, 315, 105): (71.1, 58.9, 59.3),
    (384, 576, 1344, 2688, 24, 4): (58.1, 45.0, 37.8), (36, 3328, 1088, 1088, 384, 192): (159.9, 141.1, 129.7),
    (72, 640, 640, 640, 210, 30): (45.3, 45.6, 42.9), (48, 896, 896, 0, 63, 0): (55.5, 54.0, 50.1),
    (192, 704, 1024, 1024, 56, 8): (55.3, 51.6, 48.2), (40, 1728, 1856, 0, 32, 0): (97.1, 91.9, 87.3),
    (288, 1472, 1088, 1088, 45, 9): (96.7, 85.8, 82.4), (36, 640, 1472, 1472, 33, 11): (51.0, 43.3, 38.4),
    (24, 640, 1728, 6912, 270, 270): (149.2, 90.6, 99.4), (40, 640, 1664, 3328, 660, 110): (99.3, 73.6, 77.5),
    (72, 2112, 960, 960, 1278, 213): (193.6, 170.2, 179.3), (48, 320, 256, 256, 553, 79): (31.6, 23.4, 22.8),
    (20, 448, 192, 384, 175, 175): (35.4, 23.6, 21.7), (20, 384, 1152, 4608, 218, 218): (96.2, 55.0, 53.4),
}


def test_streaming_takes_the_faster_form(ask):
    for (call, us), form in zip(FORMS.items(), ask(FORMS)):
        assert us[int(form)] <= 1.035 * min(us), call  # runs of one call differ by as much


# Both sides of each line.
LIMITS = {
    # rows per slot: few tall tiles, many of them (768 of gate/up, 512 of down), cached weights, narrow experts
    (64, 2368, 576, 0, 1280, 0): FULL, (64, 2368, 576, 0, 1281, 0): TALL,
    (96, 1536, 1024, 0, 1152, 0): FULL, (96, 1536, 1024, 0, 1153, 0): TALL, (95, 1536, 1024, 0, 1153, 0): FULL,
    (96, 1280, 1024, 0, 1153, 0): FULL, (96, 256, 1024, 0, 1153, 0): FULL,
    (512, 640, 128, 0, 4096, 0): FULL, (512, 640, 128, 0, 4097, 0): TALL, (512, 640, 384, 0, 4097, 0): TALL, (512, 640, 448, 0, 4097, 0): FULL,
    # cached weights: 192 workgroups of each launch
    (192, 256, 128, 0, 1537, 0): TALL, (191, 256, 128, 0, 1537, 0): HALF, (96, 512, 256, 0, 769, 0): TALL, (96, 256, 256, 0, 769, 0): HALF,
    # the shared expert's rows: above 128 tokens, where eight times their row-tiles outweigh the slots
    (40, 2112, 1024, 2624, 200, 128): HALF, (40, 2112, 1024, 2624, 200, 129): TALL, (40, 2112, 1024, 2560, 200, 129): HALF,
    # half the columns: below 512 workgroups, below 1024 of long products; the row-tiles of the shared expert count
    (73, 4096, 448, 0, 100, 0): HALF, (74, 4096, 448, 0, 100, 0): FULL, (63, 1024, 1024, 0, 100, 0): HALF, (64, 1024, 1024, 0, 100, 0): FULL,
    (40, 2048, 512, 0, 100, 0): HALF, (80, 2112, 512, 0, 100, 0): FULL, (80, 2048, 512, 0, 100, 0): HALF, (80, 448, 512, 0, 100, 0): FULL,
    (60, 1024, 1024, 1024, 100, 192): HALF, (60, 1024, 1024, 1024, 100, 193): FULL,
    # not streamed
    (64, 256, 128, 0, 1025, 0): "none", (64, 1024, 576, 0, 6145, 0): "none", (769, 256, 128, 0, 800, 0): "none",
}


def test_limits_of_the_forms(ask):
    assert dict(zip(LIMITS, ask(LIMITS))) == LIMITS


# The forms that the GPU tests of few rows per slot reach, without a shared expert and with one as wide.
REACHED = {
    "odd_k": (FULL, FULL), "small_tiles": (HALF, HALF), "small_tiles_narrow": (HALF, HALF), "half_columns": (HALF, HALF),
    "tiles_of_64": (HALF, TALL), "tiles_of_64_wide": (FULL, FULL), "tiles_of_128": (TALL, TALL), "tiles_of_128_many": (TALL, TALL),
    "tiles_of_128_narrow": (TALL, TALL), "rows_shared": (HALF, TALL), "many_tiles_streamed": (TALL, TALL), "tiles": ("none", "none"),
}


def test_gpu_cases_reach_the_forms(ask):
    calls = [(len(CASES[n][2]), *CASES[n][:2], CASES[n][1] * shared, sum(CASES[n][2]), sum(CASES[n][2]) * shared) for n in REACHED for shared in (0, 1)]
    forms = ask(calls)
    assert {n: tuple(forms[2 * i:2 * i + 2]) for i, n in enumerate(REACHED)} == REACHED
