"""How many chunks Seg-Sum cuts a call into (csrc/segsum_plan.hpp), compiled for
the host: the counts follow the compute units that the call's stream may use."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_10045_amd", "csrc")

SOURCE = r"""
#include "segsum_plan.hpp"
extern "C" void rounds(int64_t K, int R, int part_vec, int tiles, int nchunks, int max_chunks,
                       int64_t room, int cus, int* n, int* enough) {
  const lmz::ChunkCount c =
      lmz::whole_rounds(K, R, part_vec != 0, tiles, nchunks, max_chunks, room, cus);
  *n = c.n;
  *enough = c.enough;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    so = str(d / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                    str(d / "plan.cpp")], check=True)
    f = ctypes.CDLL(so).rounds
    f.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 5 + [ctypes.c_int64, ctypes.c_int,
                                                          ctypes.c_void_p, ctypes.c_void_p]

    def rounds(K, R, part_vec, tiles, nchunks, max_chunks, blocks, cus):
        """`blocks` workgroups of 4 waves fit on a compute unit."""
        n, enough = ctypes.c_int(), ctypes.c_int()
        f(K, R, part_vec, tiles, nchunks, max_chunks, 4 * blocks * cus, cus, ctypes.byref(n),
          ctypes.byref(enough))
        return n.value, enough.value
    return rounds


# fp32 calls on 256 compute units: (K, R, part vector, tiles, chunks needed) -> chunks
@pytest.mark.parametrize("K,R,part,tiles,need,want", [
    (19_200, 32, 0, 2, 604, 1024), (40_000, 64, 0, 1, 627, 2048), (106_496, 128, 0, 1, 1664, 2048),
    (30_011, 32, 0, 1, 1876, 1876), (20_000, 32, 0, 1, 629, 1250), (60_000, 64, 1, 1, 946, 946),
    (21_386, 32, 1, 1, 669, 1024), (640, 16, 0, 1, 63, 63)])
def test_short_chunks_fill_the_device(plan, K, R, part, tiles, need, want):
    assert plan(K, R, part, tiles, need, 5 * K // R + 1, 4, 256) == \
        (want, need if R >= 256 else -(-2560 // tiles))


@pytest.mark.parametrize("cus", [32, 64, 128, 224, 256])
@pytest.mark.parametrize("part", [0, 1])
def test_waves_follow_the_compute_units_of_the_stream(plan, cus, part):
    """Never filled above 8 waves (4 where partial rows are written a column at
    a time) for each compute unit of the stream; as many as are needed stay."""
    K, R = 40_000, 64
    top = cus * (4 if part else 8)
    for need in (16, top // 2, top - top // 8 - 1, top - top // 8, top, 3 * top // 2):
        n, enough = plan(K, R, part, 1, need, 5 * K // R + 1, 4, cus)
        assert n == (min(top, K // 16) if need < top - top // 8 else need), need
        assert enough == 10 * cus


def test_long_chunks_fill_whole_rounds(plan):
    assert plan(524_288, 512, 0, 1, 1063, 5121, 2, 256)[0] == 2048
    assert plan(524_288, 512, 0, 1, 1063, 5121, 2, 32)[0] == 1280  # a last round 39 of 256 full
    assert plan(1_048_576, 512, 0, 2, 2088, 10241, 2, 256)[0] == 3072


def test_an_unknown_device_keeps_the_chunks_it_needs(plan):
    assert plan(40_000, 64, 0, 1, 627, 3126, 0, 256)[0] == 627
    assert plan(40_000, 64, 0, 1, 627, 3126, 4, 0)[0] == 627
