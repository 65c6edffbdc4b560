"""LDS of the lookup launches, on the host: every configuration that slide_query_memory and slide_init accept has to
find room, with a sampling budget for the whole bitmap of a sample in one segment."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS = 160 * 1024
SHIM = """
#include "lookup_plan.h"
extern "C" size_t accepted(int L, int H, int NT, int NH, int words) { return slide::lookup_accepted_lds(L, H, NT, NH, words); }
extern "C" void plan(int L, int H, int NH, int NWpad, int budgeted, int rounds, size_t limit, long long* out) {
  const slide::LookupPlan p = slide::lookup_plan(L, H, NH, NWpad, budgeted != 0, rounds != 0, limit);
  out[0] = p.segw; out[1] = p.lcw; out[2] = (long long)p.bytes;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("lookup_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2201_12667_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.accepted.restype = C.c_size_t
    lib.plan.argtypes = [C.c_int] * 6 + [C.c_size_t, C.c_void_p]
    return lib


def _plan(lib, L, H, NH, words, budgeted, rounds):
    out = (C.c_longlong * 3)()
    lib.plan(L, H, NH, words, int(budgeted), int(rounds), LDS, out)
    return tuple(out)


def _shapes():
    rng = random.Random(3)
    shapes = [(400, 128, 2400), (50, 128, 450), (200, 1024, 1600), (4, 16, 24), (1, 4, 1), (3000, 2048, 9000)]
    shapes += [(L := int(2 ** rng.uniform(0, 12)), 4 * int(2 ** rng.uniform(0, 9)), L * rng.randint(1, 9)) for _ in range(60)]
    return shapes


def _largest(lib, L, H, NH, TW):
    """Bitmap words (a multiple of 32) of the largest layer whose bitmap is accepted in one piece."""
    words = 0
    while lib.accepted(L, H, (words + 32) // TW, NH, words + 32) <= LDS:
        words += 32
    return words


@pytest.mark.parametrize("TW", [4, 8, 16, 32])
def test_a_sampling_budget_has_the_whole_bitmap(lib, TW):
    for L, H, NH in _shapes():
        most = _largest(lib, L, H, NH, TW)
        for words in sorted({32, most // 64 * 32, most - 32, most}):
            if words <= 0:
                continue
            segw, lcw, used = _plan(lib, L, H, NH, words, True, False)
            assert segw == words and 2 <= lcw <= 5 and used <= LDS, (L, H, NH, words, segw, used)
            assert segw % (1 << lcw) == 0                     # (a thread's words do not reach past the segment)


def test_limit_of_the_classes_with_a_sampling_budget(lib):
    """About 1.2 million classes, as the header says."""
    assert _largest(lib, 400, 128, 2400, 32) * 32 == 1214464
    assert _largest(lib, 4, 16, 24, 32) * 32 == 1260544


@pytest.mark.parametrize("TW", [4, 8, 16, 32])
@pytest.mark.parametrize("rounds", [False, True])
def test_every_accepted_layer_has_a_segment(lib, TW, rounds):
    for L, H, NH in _shapes():
        for words in (32, 1024, 20960, 39392, 39424, 60000 // 32 * 32, 1 << 17):
            if lib.accepted(L, H, words // TW, NH, 1024) > LDS:
                continue                                       # (refused)
            segw, lcw, used = _plan(lib, L, H, NH, words, False, rounds)
            assert segw % 32 == 0 and segw >= min(words, 32 if rounds else 1024), (L, H, NH, words, segw)
            assert used <= LDS and 2 <= lcw <= 5


@pytest.mark.parametrize("rounds_of", [1, 2, 3, 4])
def test_two_workgroups_share_a_compute_unit(lib, rounds_of):
    """Batches of more than one round: up to four segments of half of the LDS, ranks of their words and all."""
    for L, H, NH in _shapes():
        half = next((w for w in range(LDS // 8, 0, -32) if _plan(lib, L, H, NH, 4 * w, False, True)[0] <= w), 0) // 32 * 32
        for per_segment in range(max(32, half - 1024), half + 1, 32):
            words = per_segment * rounds_of
            if lib.accepted(L, H, words // 32, NH, 1024) > LDS:
                continue                                       # (refused)
            segw, lcw, used = _plan(lib, L, H, NH, words, False, True)
            assert segw <= half and used <= LDS // 2, (L, H, NH, words, segw, lcw, used)
