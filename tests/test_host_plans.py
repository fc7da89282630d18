"""The library's host-side decisions that need no GPU, compiled on their own
from its headers with the host compiler: the gradient's lines per block at
every accepted side, against the same rule in Python's integers, and the
admission to a device of kernels whose blocks wait for each other."""
import ctypes
import os
import subprocess
import time

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
extern "C" int rows(int h, int w, int cus, int halves) { return thin::rows_per_block(h, w, cus, halves != 0); }
""")
    fits = 0
    for long in SIDES:
        for short in (1, 3, 255, 256, 257, 768, 769, 4096):
            for cus in (1, 32, 256):
                want_c = lines_per_block(short, 4 * chain_floats(long) + 4, cus, 1)
                floats = 4 * chain_floats(long)
                few = (160 * 1024 - 1024) // 4 // floats <= 4
                want_r = lines_per_block(short, floats, cus, 2 if few else 1)
                sums_r = lines_per_block(short, floats, cus, 3)
                assert lib.cols(long, short, cus) == want_c, (long, short, cus)
                assert lib.rows(short, long, cus, 1) == want_r, (long, short, cus)
                assert lib.rows(short, long, cus, 0) == sums_r, (long, short, cus)
                if 4 * 4 * long > 160 * 1024:
                    assert want_c == want_r == sums_r == 0
                fits += want_c > 0
    assert fits > 50


@pytest.fixture(scope="module")
def room(tmp_path_factory):
    """enter(device, which, blocks, holds) starts a thread that asks for room on
    a device of 256 units, patient(..., microseconds) one that does so for a
    while; inside(i, should) says whether thread i has room (1), waits (0) or
    went without (2), waiting up to 20 s for `should`; leave(i) lets it go."""
    lib = compiled(tmp_path_factory.mktemp("room"), "room", """
#include "room.h"
#include <atomic>
#include <chrono>
#include <thread>
namespace {
struct Job {
    std::thread th;
    std::atomic<int> state{0}, go{0};
};
Job jobs[512];
int n = 0;
}
extern "C" int patient(int device, int which, int blocks, int holds, int patience)
{
    Job& j = jobs[n];
    j.th = std::thread([=, &j] {
        const thin::Room room(device, which, blocks, holds, 256, patience);
        j.state = room.held() ? 1 : 2;
        while (!j.go) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    });
    // until it has room or waits for it
    for (int k = 0; k < 50 && !j.state; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    return n++;
}
extern "C" int enter(int device, int which, int blocks, int holds)
{
    return patient(device, which, blocks, holds, -1);
}
extern "C" int inside(int i, int should)
{
    for (int k = 0; k < 20000 && should != jobs[i].state && should; ++k)
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
    return jobs[i].state;
}
extern "C" void leave(int i)
{
    jobs[i].go = 1;
    jobs[i].th.join();
}
""", "-pthread")
    return lib


@pytest.mark.parametrize("blocks,held,fit", [(85, 0, 2), (64, 0, 4), (57, 0, 4), (1, 0, 32),
                                             (170, 512, 2), (168, 512, 3), (300, 512, 1)])
def test_room_counts_the_fullest_xcd(room, blocks, held, fit):
    """As many kernels of `blocks` blocks as every XCD has units for (or, all of
    one kernel, holds blocks of it: `held` in all) run together, and one more
    waits for one of them to end."""
    device = 1 + (blocks * 7 + held) % 60
    holds = held or 256
    # the fullest XCD takes a block of every turn a kernel deals
    assert fit * -(-blocks // 8) <= holds // 8 < (fit + 1) * -(-blocks // 8)
    ids = [room.enter(device, 1, blocks, holds) for _ in range(fit + 1)]
    assert [room.inside(i, 1) for i in ids[:-1]] == [1] * fit
    assert room.inside(ids[-1], 0) == 0
    room.leave(ids[0])
    assert room.inside(ids[-1], 1) == 1
    for i in ids[1:]:
        room.leave(i)


def test_room_lets_what_fits_past_what_waits(room):
    """A kernel of 242 blocks waits for one of 64; eight that fit beside that one
    go past it, the ninth waits behind it, and all get their turn."""
    first = room.enter(61, 0, 64, 2048)
    big = room.enter(61, 1, 242, 512)
    assert (room.inside(first, 1), room.inside(big, 0)) == (1, 0)
    for _ in range(8):
        i = room.enter(61, 2, 8, 512)
        assert room.inside(i, 1) == 1
        room.leave(i)
    ninth = room.enter(61, 2, 16, 512)
    assert room.inside(ninth, 0) == 0
    room.leave(first)
    assert room.inside(big, 1) == 1
    assert room.inside(ninth, 0) == 0     # 248 + 16 blocks are more than 256
    room.leave(big)
    assert room.inside(ninth, 1) == 1
    room.leave(ninth)


def test_room_is_waited_for_while_it_is_given_back(room):
    """A kernel that could run another way leaves when no room has been given
    back for its patience, counted anew each time some has; one that waits
    behind it then has its turn."""
    first = room.enter(62, 0, 64, 2048)
    big = room.patient(62, 1, 242, 512, 3_000_000)
    for _ in range(8):
        i = room.enter(62, 2, 8, 512)
        assert (room.inside(i, 1), room.inside(big, 0)) == (1, 0)
        time.sleep(0.2)
        room.leave(i)
    ninth = room.enter(62, 2, 8, 512)
    assert (room.inside(ninth, 0), room.inside(big, 0)) == (0, 0)
    assert (room.inside(big, 2), room.inside(ninth, 1)) == (2, 1)
    for i in (first, big, ninth):
        room.leave(i)
    alone = room.patient(62, 1, 242, 512, 0)
    assert room.inside(alone, 1) == 1
    room.leave(alone)
