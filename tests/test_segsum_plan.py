"""How many chunks Seg-Sum cuts a call into (csrc/segsum_plan.hpp), compiled for
the host: the counts follow the compute units that the call's stream may use,
and calls with few types are not cut for more waves than those can start at once."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_10045_amd", "csrc")

SOURCE = r"""
#include "segsum_plan.hpp"
extern "C" void rounds(int64_t K, int64_t D, int64_t u_cap, int R, int bf16, int tiles,
                       int nchunks, int max_chunks, int64_t room, int cus, int* n, int* enough) {
  const lmz::ChunkCount c = lmz::whole_rounds(K, D, u_cap, R, bf16 != 0, tiles, nchunks,
                                              max_chunks, room, cus);
  *n = c.n;
  *enough = c.enough;
}
extern "C" int by_column(uintptr_t grad, int64_t ld, int64_t D, int bf16) {
  return lmz::column_per_lane(grad, ld, D, bf16 != 0);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    so = str(d / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                    str(d / "plan.cpp")], check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def plan(lib):
    f = lib.rounds
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 5 + [ctypes.c_int64, ctypes.c_int,
                                                             ctypes.c_void_p, ctypes.c_void_p]

    def rounds(K, u_cap, R, need, tiles=1, bf16=0, D=512, blocks=4, cus=256, most=None):
        """`need` chunks; `blocks` workgroups of 4 waves fit on a compute unit."""
        n, enough = ctypes.c_int(), ctypes.c_int()
        f(K, D, min(K, u_cap), R, bf16, tiles, need, most or 5 * K // R + 1, 4 * blocks * cus,
          cus, ctypes.byref(n), ctypes.byref(enough))
        return n.value, enough.value
    return rounds


# Calls on 256 compute units: chunks needed (one round at most) -> chunks.
MANY = [(40_000, 2_000, 64, 627, 2048, {}), (106_496, 800_000, 128, 1664, 2048, {}),
        (30_011, 50_000, 32, 1876, 1876, {}), (21_386, 2_865, 32, 669, 1024, dict(D=358)),
        (20_000, 5_000, 32, 629, 1250, {}), (640, 10_000, 16, 63, 63, {}),
        (100_000, 5_000, 128, 938, 2048, dict(bf16=1)),
        (524_288, 20_000, 512, 1063, 2048, dict(blocks=2)),
        (200_000, 20_000, 256, 860, 3907, dict(blocks=6))]  # the workspace's room
FEW = [(30_000, 98, 32, 950, 950, dict(bf16=1)), (60_000, 500, 64, 945, 945, {}),
       (100_000, 500, 128, 786, 1024, dict(bf16=1)), (19_200, 98, 32, 604, 604, {}),
       (19_200, 98, 32, 604, 1024, dict(tiles=2)), (19_200, 98, 32, 604, 604, dict(tiles=2, D=1791)),
       (200_000, 98, 256, 782, 1024, dict(blocks=6)), (262_144, 98, 256, 1025, 1025, {}),
       (905_469, 221, 512, 1769, 2048, dict(bf16=1)),
       (16_000, 98, 16, 900, 900, {}),
       (300_000, 221, 512, 586, 2048, dict(bf16=1, D=14)), (300_000, 221, 512, 586, 2048, dict(D=91)),
       (300_000, 221, 512, 586, 1024, dict(D=357)), (60_000, 221, 64, 941, 941, dict(D=64)),
       (200_000, 98, 256, 782, 2048, dict(D=255)), (200_000, 98, 256, 782, 1024, dict(D=256))]


@pytest.mark.parametrize("K,V,R,need,want,how", MANY + FEW)
def test_less_than_one_round(plan, K, V, R, need, want, how):
    """Long segments are cut for whole workgroups of the compute units only."""
    assert (K >= 32 * V) == ((K, V, R, need, want, how) in FEW)
    assert plan(K, V, R, need, **how)[0] == want


@pytest.mark.parametrize("cus", [32, 64, 128, 224, 256])
@pytest.mark.parametrize("D", [512, 513])
@pytest.mark.parametrize("V", [100, 4000])
def test_waves_follow_the_compute_units_of_the_stream(plan, cus, D, V):
    """Never filled above 8 waves (4 where partial rows are written a column at
    a time) for each compute unit of the stream; as many as are needed stay."""
    K, R = 100_000, 64
    for need in (16, cus, 3 * cus, 4 * cus, 5 * cus, 7 * cus, 8 * cus, 12 * cus):
        n, enough = plan(K, V, R, need, D=D, cus=cus)
        assert need <= n <= max(need, cus * (8 if D == 512 else 4)) and enough == n
        assert n in (need, 4 * cus, 8 * cus)
        assert plan(K, V, R, need, D=D, cus=cus, bf16=1) == (n, 10 * cus)


def test_whole_rounds(plan):
    assert plan(1_048_576, 98, 512, 2088, tiles=2, blocks=2)[0] == 3072
    assert plan(1_048_576, 98, 512, 2049, blocks=2)[0] == 4096
    assert plan(524_288, 20_000, 512, 1063, blocks=2, cus=32)[0] == 1280  # 39 of 256 in the last
    assert plan(524_288, 20_000, 512, 1200, blocks=2, cus=32)[0] == 1200  # 176 of 256
    assert plan(524_288, 20_000, 512, 1063, blocks=2, cus=32, most=1100)[0] == 1100


def test_the_chunk_length_stays_with_fp32_rows(plan):
    """Only bf16 calls lower the count where few types turn up."""
    assert plan(120_000, 800_000, 128, 1875, tiles=2) == (1875, 1875)
    assert plan(30_011, 50_000, 32, 4690, tiles=2, bf16=1)[1] == 1280
    assert plan(400_000, 300_000, 512, 3125, bf16=1) == (3907, 3907)  # the workspace's room


def test_an_unknown_device_keeps_the_chunks_it_needs(plan):
    assert plan(40_000, 2_000, 64, 627, blocks=0) == (627, 627)
    assert plan(40_000, 2_000, 64, 627, cus=0) == (627, 627)


def test_bf16_rows_between_words_take_a_column_per_lane(lib):
    f = lib.by_column
    f.argtypes = [ctypes.c_size_t, ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    base = 0x7f0000001000
    for D, ld, at, want in ((7, 7, 0, 1), (8, 8, 0, 0), (8, 8, 2, 1), (8, 9, 0, 1), (9, 10, 0, 1),
                            (10, 10, 0, 0), (10, 10, 4, 0), (255, 255, 0, 1), (256, 256, 0, 0),
                            (256, 257, 0, 1), (257, 257, 0, 0), (1031, 1031, 2, 0)):
        assert f(base + at, ld, D, 1) == want, (D, ld, at)
    assert [f(base + 4, D + 1, D, 0) for D in (1, 3, 4, 5, 255)] == [1, 1, 0, 0, 0]
