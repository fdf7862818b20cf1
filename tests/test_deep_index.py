"""Every load of the two-step kernel lies inside the population buffer, and every
one that a result needs is the pull's: the kernel's own index expressions
(csrc/fslbm_deep_index.hpp), evaluated on the CPU for lattices of one to three
planes, rows from one cell to past two tiles, periodic and walled, with rows up
to the last that the kernel may take."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def loads(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("deep") / "deep_index")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_1409_5645_amd", "csrc"),
                    os.path.join(ROOT, "tests", "deep_index.cpp"), "-o", exe], check=True)

    def run(*args):
        return [int(v) for v in subprocess.run([exe] + [str(v) for v in args], check=True, capture_output=True,
                                               text=True).stdout.split()]
    return run


@pytest.mark.parametrize("s", [8, 4])
@pytest.mark.parametrize("px,pz", list(itertools.product((0, 1), (0, 1))))
def test_loads_stay_inside_and_are_the_pulls(loads, s, px, pz):
    tx = 32 if s == 8 else 64
    for nx in (1, 2, 3, 4, 8, tx // 2 - 1, tx // 2, tx - 1, tx, tx + 1, 2 * tx - 1, 2 * tx, 2 * tx + 1):
        for nz in (1, 2, 3, 17):
            for ny, yd in ((26, 24), (40, 38), (41, 25), (90, 24)):
                out, wrong = loads(s, nx, ny, nz, px, pz, yd)
                assert (out, wrong) == (0, 0), (nx, ny, nz, yd)
