"""Rules that size launches, on the host."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "launch_rules.h"
extern "C" int workers(int nworkers, int items, int ntiles, int nxcd) { return slide::logit_workers(nworkers, items, ntiles, nxcd); }
extern "C" int tables_of_wave(int L, int C, int lg, int nlong, int entries) { 
  return slide::tables_of_wave(slide::long_rule(L, C, lg), lg, nlong, entries);
}
extern "C" int streams_weights(double rows, int H, int aligned) { return slide::streams_weights(rows, H, aligned != 0); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_rules")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2201_12667_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.streams_weights.argtypes = [C.c_double, C.c_int, C.c_int]
    return lib


@pytest.mark.parametrize("cus", [256, 32, 304, 80])
def test_logit_workers_fill_the_dies_evenly(lib, cus):
    nxcd = cus // 32 if cus % 32 == 0 else 1
    for nworkers in (3 * cus, 2 * cus, 3 * cus // 2):
        for ntiles in (0, 1, 100, 2272, 30000):
            for items in (1, 2 * nworkers * 8, 2 * nworkers * 8 + 1, 41000, 600000, 5000000):
                stay = lib.workers(nworkers, items, ntiles, nxcd)
                assert nworkers // 2 <= stay <= nworkers
                assert stay % nxcd == 0
                if ntiles == 0 or items <= 2 * nworkers * 8:
                    assert stay == nworkers
                else:
                    assert stay < nworkers


def _lanes(L):
    lg = 0
    while lg < 6 and L << (lg + 1) <= 1024:
        lg += 1
    return lg


@pytest.mark.parametrize("L", [1, 2, 15, 16, 17, 50, 64, 65, 68, 100, 200, 400, 512, 513, 1000, 1024, 1025, 4000])
def test_long_buckets_are_shared_out(lib, L):
    """Every table belongs to one wave, and where long buckets go by waves none has many more than its share of them."""
    lg = _lanes(L)
    for C in (9 << lg, 16 << lg, 256, 1024):
        for nlong in sorted({1, min(L, 5), min(L, 64), min(L, 65), max(1, L // 2), L}):
            for mean in {(8 << lg) + 1, (C + (8 << lg)) // 2, C}:
                if not (8 << lg) < mean <= C:
                    continue                                   # (no long buckets)
                per = lib.tables_of_wave(L, C, lg, nlong, min(nlong * mean, 2 ** 31 - 1))
                assert 0 <= per <= 64 and (per > 0 or nlong > 64)
                if per == 0:
                    continue
                assert 16 * per >= min(L, 1024)
                spread = [t * L // nlong for t in range(nlong)]
                waves = [0] * 16
                for t in spread:
                    waves[t // per % 16] += 1
                assert max(waves) <= max(8, 2 * (nlong // 16 + 1))


# tables, capacity, long buckets, entries of a sample; what was measured to be the faster
@pytest.mark.parametrize("L,C,nlong,entries,waves", [
    (68, 256, 68, 68 * 146, True), (68, 256, 60, 60 * 200, True), (50, 256, 50, 50 * 195, True), (100, 512, 100, 100 * 390, True),
    (150, 64, 150, 150 * 48, False), (200, 64, 200, 200 * 48, False), (200, 256, 200, 200 * 195, True), (214, 64, 200, 214 * 36, False),
    (300, 32, 250, 300 * 19, False), (300, 128, 300, 300 * 97, True), (400, 32, 300, 400 * 19, False), (400, 64, 400, 400 * 48, False),
    (400, 256, 400, 400 * 195, True), (600, 32, 600, 600 * 19, False), (600, 128, 600, 600 * 97, True), (1000, 16, 800, 1000 * 10, False),
    (1000, 64, 1000, 1000 * 43, True), (1000, 200, 1000, 1000 * 175, True), (2000, 64, 2000, 2000 * 43, True)])
def test_long_buckets_go_the_faster_way(lib, L, C, nlong, entries, waves):
    assert (lib.tables_of_wave(L, C, _lanes(L), nlong, entries) > 0) == waves


# rows, their length; whether streaming them was measured to be faster
@pytest.mark.parametrize("rows,H,faster", [
    (642_000, 128, True), (540_000, 160, True), (358_000, 256, True), (635_000, 256, True), (539_000, 320, True), (579_000, 192, True),
    (331_000, 352, True), (331_000, 480, True), (582_000, 512, True), (270_000, 512, True), (208_000, 1024, True),
    (255_000, 128, False), (178_000, 384, False), (100_000, 1024, False),                         # the cache holds them
    (170_000, 356, False), (220_000, 300, False), (480_000, 200, False), (668_000, 120, False),   # parts of lines
    (208_000, 544, False), (208_000, 640, False), (208_000, 672, False), (208_000, 768, False), (208_000, 928, False)])
def test_weights_are_streamed_where_that_pays(lib, rows, H, faster):
    assert bool(lib.streams_weights(rows, H, 1)) == faster
    assert not lib.streams_weights(rows, H, 0)
