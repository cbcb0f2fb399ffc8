"""The planner's launch shape (csrc/plan_shape.h, built for the host): every
slot has a thread and every node a team, and the launch stays within the 2^32
threads a dimension holds, up to the largest graph the library accepts."""

import ctypes
import os
import subprocess

import pytest

from paper_1804_09741_amd import motifs as M

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1804_09741_amd", "csrc")
SOURCE = r"""
#include "plan_shape.h"
extern "C" uint64_t blocks(int64_t nnz) { return mk::plan_blocks(nnz); }
extern "C" uint32_t threads(int k, uint64_t b, uint64_t ng) { return mk::plan_threads(k, b, ng); }
"""


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I" + CSRC, str(d / "s.cpp"),
                    "-o", str(d / "s.so")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))
    lib.blocks.restype = ctypes.c_uint64
    lib.blocks.argtypes = [ctypes.c_int64]
    lib.threads.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64]
    return lib


@pytest.mark.parametrize("k", [2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("ng", [1, 101, 14337])
def test_shape(shape, k, ng):
    # adjacency entries of a batch stay below 2^32 (its last 64 fill the dimension)
    most = M.MK_MAX_VERTICES * M.MK_MAX_DEGREE - 65
    for nnz in (0, 1, 64, 65, 32768, 32769, 2**20, 2**24 + 1, 2**30 - 64, 2**30, 2**30 + 1, most):
        b = shape.blocks(nnz)
        t = shape.threads(k, b, ng)
        assert b >= 1 and b * 64 >= nnz and (b - 1) * 64 < max(nnz, 1)
        assert t % 64 == 0 and 64 <= t <= 1024
        assert b * t < 2**32, (nnz, t)
        if k > 3 and nnz < 2**30 - 64:
            assert t == (1024 if b * ng <= 512 else 256)
