"""The work queues' index arithmetic (csrc/queue.h, the header that the
counting kernels' unit loop is written with) built for the host: whatever the
number of units and waves, the grab sizes, the split of the units over the
queues and the interleaving of the waves, every unit is taken exactly once."""

import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1804_09741_amd", "csrc")

SOURCE = r"""
#include "queue.h"
#include <cstddef>
#include <cstdint>
#include <vector>
using namespace mk;
// A launch of `grid` waves over [begin, begin + span): seen[u] counts how often
// unit u was taken.  A wave makes one grab a turn; a generator (SplitMix64)
// picks whose turn it is.
extern "C" int run_launch(uint32_t begin, uint32_t span, uint32_t grid, uint32_t chunk,
                          int heavy_first, int mix, uint64_t seed, const uint8_t *heavy,
                          uint32_t *seen)
{
    struct Wave { UnitQueue q; int sweep, t; bool done; };
    std::vector<Wave> w(grid);
    std::vector<uint32_t> head[2] = {std::vector<uint32_t>(kQueues), std::vector<uint32_t>(kQueues)};
    for (uint32_t i = 0; i < grid; ++i) {
        w[i].q = unit_queue(begin, begin + span, grid, i, chunk, heavy_first != 0, mix != 0);
        w[i].sweep = w[i].q.two ? 0 : 1;
        w[i].t = 0;
    }
    std::vector<uint32_t> live(grid);
    for (uint32_t i = 0; i < grid; ++i) live[i] = i;
    uint64_t s = seed;
    uint64_t turns = 0;
    while (!live.empty()) {
        if (++turns > 64ull * (span + 1) + 64ull * grid) return 1;  // waves that never end
        s += 0x9E3779B97F4A7C15ull;
        uint64_t z = s;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        const size_t at = (size_t)((z ^ (z >> 31)) % live.size());
        Wave &v = w[live[at]];
        const int x = queue_range(v.q, v.t);
        if (x < 0 || x >= kQueues) return 2;
        uint32_t &h = head[v.sweep][x], first, stop;
        const uint32_t taken = h;
        h += queue_chunk(v.q, v.sweep);
        if (queue_grab(v.q, x, v.sweep, taken, first, stop)) {
            if (first < begin || stop > begin + span || stop <= first) return 3;
            if (v.sweep == 0 && stop - first > 64) return 4;  // a lane a unit
            for (uint32_t u = first; u < stop; ++u)
                if (!v.q.two || (heavy[u - begin] != 0) == (v.sweep == 0)) ++seen[u - begin];
        } else if (++v.t > v.q.tries) {
            v.t = 0;
            if (++v.sweep == 2) {
                live[at] = live.back();
                live.pop_back();
            }
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def launch(tmp_path_factory):
    d = tmp_path_factory.mktemp("queue")
    src, lib = d / "queue.cpp", d / "queue.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-D__host__=",
                    "-D__device__=", "-D__forceinline__=inline", "-I" + CSRC, str(src), "-o",
                    str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).run_launch
    fn.argtypes = [ctypes.c_uint32] * 4 + [ctypes.c_int] * 2 + [ctypes.c_uint64,
                                                               ctypes.c_char_p, ctypes.c_void_p]
    return fn


@pytest.mark.parametrize("grid", [1, 2, 7, 8, 9, 63, 64, 65, 100, 640])
@pytest.mark.parametrize("mix", [0, 1])
@pytest.mark.parametrize("heavy_first", [0, 1])
def test_every_unit_once(launch, grid, mix, heavy_first):
    rng = random.Random(grid * 4 + mix * 2 + heavy_first)
    spans = [0, 1, 7, 8, 9, 64, 65, 15 * grid, 16 * grid - 1, 16 * grid, 32 * grid - 1, 32 * grid,
             33 * grid + 5, rng.randint(0, 6000)]
    for span in spans:
        for chunk in (0, 1, 3, 16, 64, 300):
            begin = rng.choice([0, 5, 100000])
            heavy = bytes(rng.random() < 0.4 for _ in range(span))
            seen = (ctypes.c_uint32 * max(span, 1))()
            rc = launch(begin, span, grid, chunk, heavy_first, mix, rng.getrandbits(64), heavy,
                        ctypes.byref(seen))
            assert rc == 0, (rc, span, chunk)
            assert list(seen)[:span] == [1] * span, (span, chunk)


def test_end_of_the_index_range(launch):
    """Units up to 2^32 - 1: sums of a range's start and a grab stay in 32 bits."""
    for mix in (0, 1):
        begin, span = 2**32 - 1 - 5000, 5000
        seen = (ctypes.c_uint32 * span)()
        assert launch(begin, span, 64, 0, 0, mix, 7, bytes(span), ctypes.byref(seen)) == 0
        assert list(seen) == [1] * span
