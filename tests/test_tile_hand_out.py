"""The hand-out of a traversal launch's tiles to its waves (csrc/st_tiles.h, the code the
kernels run), built for the CPU: every tile goes to exactly one wave, whatever the number
of waves and the order in which they come to the counters."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "st_tiles.h"
#include <atomic>
#include <thread>
#include <vector>
using namespace st;
// how often each tile was taken; serial: one wave after the other, first or last wave
// first; else every wave a thread
extern "C" void hand_out(uint32_t waves, uint32_t tiles, int order, uint32_t* taken) {
    std::vector<std::atomic<uint32_t>> count(TAKE_NC), got(tiles);
    auto wave = [&](uint32_t w) {
        hand_out_tiles(w, waves, tiles, [&](uint32_t c) { return count.at(c)++; }, [&](uint32_t t) { ++got.at(t); });
    };
    if (order == 2) {
        std::vector<std::thread> th;
        for (uint32_t w = 0; w < waves; ++w) th.emplace_back(wave, w);
        for (auto& t : th) t.join();
    } else {
        for (uint32_t i = 0; i < waves; ++i) wave(order == 0 ? i : waves - 1 - i);
    }
    for (uint32_t t = 0; t < tiles; ++t) taken[t] = got[t];
}
"""


@pytest.fixture(scope="module")
def hand_out(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    src, lib = d / "t.cpp", d / "t.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-I",
                    os.path.join(ROOT, "paper_2012_03939_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).hand_out
    fn.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_void_p]
    return fn


@pytest.mark.parametrize("waves", [1, 2, 3, 4, 8, 12, 15, 16, 17, 20, 32, 2048])
def test_every_tile_is_taken_once(hand_out, waves):
    # around the number of waves, and what 256 paths a block make at 1 to 17 shadow entries
    counts = {0, 1, waves - 1, waves, waves + 1, 2 * waves, 3 * waves + 1, 5 * waves - 1, 18 * waves, 18 * waves + 5}
    for tiles in sorted(counts):
        for order in (0, 1, 2) if waves <= 32 else (0, 1):
            taken = np.zeros(max(tiles, 1), np.uint32)
            hand_out(waves, tiles, order, taken.ctypes.data)
            assert (taken[:tiles] == 1).all(), (waves, tiles, order, np.flatnonzero(taken[:tiles] != 1)[:20])
