"""Addresses of the vector convolution kernel, enumerated on the host.

The kernel's index arithmetic (csrc/cnn_rows.h) is compiled for the CPU with the
sanitizers and every slice it would read is compared with the convolution's definition
(tests/sanitize/conv_rows_driver.cpp).  What is read beyond an operand meets zero
filters, so no result shows it.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

SHAPES = [  # n, h, w, c, k, r, stride, pad
    (61, 19, 23, 24, 40, 3, 2, 1),     # rows and slices both with a remainder
    (7, 61, 59, 8, 68, 3, 1, 1),
    (61, 19, 23, 8, 40, 3, 1, 1),
    (3, 5, 5, 24, 24, 3, 1, 1),
    (1, 3, 8001, 8, 8, 3, 1, 1),       # a row far longer than the image is high
    (1, 8001, 3, 8, 8, 3, 1, 2),
    (17, 1, 1, 512, 104, 1, 1, 0),     # a fully connected head: 104 of 128 k backwards
    (24, 4, 4, 16, 104, 1, 1, 0),
    (100, 2, 2, 16, 104, 3, 1, 1),
    (2, 20, 21, 16, 8, 3, 4, 1),       # classes without a tap
    (3, 9, 7, 72, 40, 3, 1, 1),
    (6, 13, 12, 24, 72, 1, 2, 0),
    (5, 7, 9, 16, 24, 3, 3, 2),
    (1, 1, 1, 8, 8, 1, 1, 0),
    (2, 4, 6, 32, 32, 3, 2, 0),
    (2, 5, 5, 8, 4, 3, 1, 1),          # 4 output channels in a block: 4, 16 + 4, 64 + 4
    (2, 5, 5, 8, 20, 1, 1, 0),
]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("conv_rows") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-Wno-unused-function",
                    os.path.join(ROOT, "tests", "sanitize", "conv_rows_driver.cpp"),
                    "-I", os.path.join(ROOT, "paper_2503_16424_amd", "csrc"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)
    return exe


@pytest.mark.parametrize("shape", SHAPES)
def test_every_read_lies_inside_its_operand(driver, shape):
    r = subprocess.run([driver, *map(str, shape)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
