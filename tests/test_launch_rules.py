"""Rules that size launches, on the host."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "launch_rules.h"
extern "C" int workers(int nworkers, int items, int ntiles, int nxcd) { return slide::logit_workers(nworkers, items, ntiles, nxcd); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_rules")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2201_12667_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    return C.CDLL(str(d / "shim.so"))


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
