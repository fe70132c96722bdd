"""Launch shapes (pic_launch.h) over the accepted sizes: a HIP launch has less
than 2^32 threads on an axis.  The header is plain C++: compiled here with
g++ and called through ctypes."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_14795_amd", "csrc")
LIMIT = 1 << 32

SOURCE = """
#include "pic_launch.h"
extern "C" int settle_threads(int64_t n, int64_t n_tiles, int most) { return pic::settle_threads(n, n_tiles, most); }
extern "C" void block_grid(int64_t blocks, int threads, unsigned *out)
{
    const pic::BlockGrid g = pic::block_grid(blocks, threads);
    out[0] = g.x;
    out[1] = g.y;
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("shapes")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, str(d / "s.cpp"), "-o",
                    str(d / "s.so")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))
    lib.block_grid.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_uint)]
    lib.settle_threads.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return lib


# the largest accepted grid (32,767 cells an axis) is 4,095^2 tiles of 8 x 8
TILES = [1, 3, 15, 256, 4096, 65536, 4194304, 8388608, 4095 * 4095]
PARTICLES = [0, 1, 64, 4095, 1 << 20, (1 << 28) + 1, (1 << 31) - 1]


def test_settle_threads(shapes):
    for tiles in TILES:
        for n in PARTICLES:
            nt = shapes.settle_threads(n, tiles, 1024)
            assert nt in (16, 32, 64, 128, 256, 512, 1024)
            assert nt == 1024 or 16 * nt * tiles >= n     # four passes of four per thread
            # half as many would not do, or the device holds these at once and they have work
            assert nt == 16 or 8 * nt * tiles < n or (nt * tiles <= 256 * 2048 and 2 * nt * tiles < n)
            block = max(nt, 256)
            assert -(-tiles // (block // nt)) * block < LIMIT, (tiles, n)
            # a batch: items of four tiles, each by one block or (on the second axis) several
            assert -(-tiles // 4) * min(block, 4 * nt) < LIMIT, (tiles, n)


def test_block_grid(shapes):
    out = (ctypes.c_uint * 2)()
    for threads in (256, 640, 1024):
        most = (LIMIT - 1) // threads
        # four species' plan blocks on the largest grid beside its field blocks, and about the border
        for blocks in [1, 5, 4096, most - 1, most, most + 1, 2 * most + 1, 4095 * 4095 + 32760 * 32760 // 512]:
            shapes.block_grid(blocks, threads, out)
            x, y = out
            assert x * threads < LIMIT and 1 <= y <= 65535
            assert (x - 1) * y < blocks <= x * y < 1 << 31
            assert y == 1 or blocks > most
