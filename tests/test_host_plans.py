"""The library's host-side decisions that need no GPU, compiled on their own
from its headers with the host compiler: the gradient's lines per block at
every accepted side, against the same rule in Python's integers."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1603_09180_amd", "csrc")


def compiled(tmp_path, name, source, *flags):
    """A shared library of `source`, which may include the library's headers."""
    src, lib = tmp_path / f"{name}.cpp", tmp_path / f"lib{name}.so"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-fPIC", "-shared", *flags,
                    "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


def lines_per_block(lines, floats, num_cus, waves):
    most = min(16, (160 * 1024 - 1024) // 4 // floats)
    if most <= 0 or most * num_cus * waves < lines:
        return 0
    return min(-(-lines // num_cus), most)


def chain_floats(n):
    return 4 * ((n + 3) // 4 | 1)


SIDES = [1, 2, 5, 64, 1024, 1025, 1283, 2500, 2501, 9900, 9936, 9937, 10160, 10161, 40000, 2 ** 20,
         2 ** 28 - 3, 2 ** 28, 2 ** 29 - 3, 2 ** 29, 2 ** 29 + 1, 2 ** 30 - 8, 2 ** 30 - 4,
         2 ** 30 - 3, 2 ** 30 - 1, 2 ** 30]


def test_gradient_lines_per_block(tmp_path):
    """A line that does not fit LDS is never given to the LDS passes, at sides
    where four lines of it pass 2^31 and 2^32 too."""
    lib = compiled(tmp_path, "gradient_plan", """
#include "gradient_plan.h"
extern "C" int cols(int h, int w, int cus) { return thin::columns_per_block(h, w, cus); }
extern "C" int rows(int h, int w, int cus) { return thin::rows_per_block(h, w, cus); }
""")
    fits = 0
    for long in SIDES:
        for short in (1, 3, 255, 256, 257, 768, 769, 4096):
            for cus in (1, 32, 256):
                want_c = lines_per_block(short, 4 * chain_floats(long) + 4, cus, 1)
                want_r = lines_per_block(short, 4 * chain_floats(long), cus, 3)
                assert lib.cols(long, short, cus) == want_c, (long, short, cus)
                assert lib.rows(short, long, cus) == want_r, (long, short, cus)
                if 4 * 4 * long > 160 * 1024:
                    assert want_c == want_r == 0
                fits += want_c > 0
    assert fits > 50
