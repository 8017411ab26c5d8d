"""Which kernel an fp32 product gets: the planner is plain C++ and is asked on the host.  The GPU tests of the products on two fp16
pieces name the kernel of every shape; here these names are held against the plan, so that none of them tests another kernel."""
import ctypes
import os
import subprocess

import pytest

from test_gpu_fp16_pairs import FIMS, SCORES, STEPS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_18976_amd", "csrc")
TILES = {0: "256", 1: "128", 2: "64x512", 3: "128x256"}
SOURCE = """
#include "gemm_f32_plan.h"
using namespace grass;
extern "C" void plan(int a_kn, int b_kn, uint64_t M, uint64_t N, uint64_t K, uint64_t ld, int lower, uint32_t most, uint32_t* out) {
    const GemmPlan p = gemm_f32_plan(a_kn, b_kn, M, N, K, ld, lower, most);
    out[0] = p.pair; out[1] = p.tile; out[2] = p.splits;
}
extern "C" uint64_t cut(uint64_t M, uint64_t N, uint64_t K, uint32_t most, uint32_t* out) {
    const GemmCut c = gemm_f32_cut(M, N, K, 0, most);
    out[0] = c.head.pair; out[1] = c.head.tile; out[2] = c.head.splits;
    out[3] = c.tail.pair; out[4] = c.tail.tile; out[5] = c.tail.splits;
    return c.head_n;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")], check=True)
    so = ctypes.CDLL(str(d / "plan.so"))
    so.plan.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_uint64] * 4 + [ctypes.c_int, ctypes.c_uint32, ctypes.c_void_p]
    so.cut.argtypes, so.cut.restype = [ctypes.c_uint64] * 3 + [ctypes.c_uint32, ctypes.c_void_p], ctypes.c_uint64
    return so


def _name(pair, tile):
    return TILES[tile] if pair else "-"


def _plan(lib, a_kn, b_kn, M, N, K, ld, lower, most):
    out = (ctypes.c_uint32 * 3)()
    lib.plan(a_kn, b_kn, M, N, K, ld, lower, most, out)
    return _name(out[0], out[1]), out[2]


def _cut(lib, M, N, K, most):
    out = (ctypes.c_uint32 * 6)()
    head = lib.cut(M, N, K, most, out)
    return (_name(out[0], out[1]) + "+" if head else "") + _name(out[3], out[4])


@pytest.mark.parametrize("shape", SCORES)
def test_scores(lib, shape):
    assert (_cut(lib, *shape, 64), _cut(lib, *shape, 1)) == SCORES[shape]


@pytest.mark.parametrize("shape", FIMS)
def test_projected_fim(lib, shape):
    N, k = shape
    assert _plan(lib, 1, 1, k, k, N, k, 1, 32)[0] == FIMS[shape]


@pytest.mark.parametrize("shape", STEPS)
def test_selective_mask_step(lib, shape):
    m, n, p = shape
    forward, backward = _plan(lib, 0, 0, m, n, p, 0, 0, 64)[0], _plan(lib, 0, 1, m, p, n, p, 0, 1)[0]
    assert (forward, "grad" if m <= 128 and backward != "-" else backward) == STEPS[shape]


def test_gaussian_projection_in_chunks(lib):
    assert _plan(lib, 0, 0, 20, 40, 512, 0, 0, 8)[0] == "-"
    assert _plan(lib, 0, 0, 20, 40, 4_096, 0, 0, 8) == ("128", 8)


def test_every_tile_is_reached():
    assert {t for names in SCORES.values() for n in names for t in n.split("+")} == {"256", "128", "128x256", "-"}
    assert set(FIMS.values()) == {"256", "128"} and {b for _, b in STEPS.values()} == {"grad", "256", "128"}


def test_plans_stay_within_their_limits(lib):
    """K ranges of two fp16 pieces have 256 k and more, of anything at most one per 32 k; 64 x 512 is for at most 64 row-major rows
    and three bf16 pieces, 128 x 256 for two fp16 ones; rows too far apart for 32-bit offsets get 128 x 128 and three bf16 pieces."""
    sizes = (1, 3, 64, 65, 128, 129, 1_000, 70_001)
    for M in sizes:
        for N in sizes:
            for K in (1, 31, 255, 256, 257, 511, 512, 4_097, 1_863_690):
                for a_kn, b_kn, most in ((0, 0, 64), (0, 1, 1), (1, 1, 32)):
                    name, splits = _plan(lib, a_kn, b_kn, M, N, K, 0, 0, most)
                    assert 1 <= splits <= min(most, -(-K // 32))
                    assert name == "-" or K // splits >= 256
                    assert name != "64x512" and (name != "128x256" or not a_kn)
                    assert _plan(lib, a_kn, b_kn, M, N, K, 1 << 26, 0, most)[0] == "-"


@pytest.mark.parametrize("shape", [(85, 1_684, 16_224), (1_035, 5_703, 411), (969, 763, 3_181), (38, 21_102, 2_253)])
def test_the_later_start_counts_once(lib, shape):
    """Two fp16 pieces take 8 us more to start and win here (63.5 -> 51.7, 46.4 -> 38.4, 56.8 -> 45.8 and 60.0 -> 55.9 us); 13 us, the
    whole of their start, kept these on three bf16 ones."""
    assert _cut(lib, *shape, 64) != "-"
