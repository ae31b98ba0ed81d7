"""The tile arithmetic that the kernels and the host share, built for the CPU (tests/host_rules.cpp)."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "paper_1708_07525_amd", "csrc"),
                    os.path.join(HERE, "host_rules.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.first_wrong_tile.restype = ctypes.c_longlong
    lib.divides_exactly.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return lib


def test_frame_tiles_at_every_width(rules):
    """The frame between node walls has every tile of its rows and columns, up to the widest lattice
    that a population buffer of 4 GiB holds (865504 x 64 nodes in FP32: 54094 tiles of 16)."""
    for ntx in list(range(8, 400)) + list(range(46000, 54100, 7)) + [46508, 54094]:
        assert rules.first_wrong_tile(ntx, 4, 1, 0, 0) == -1, ntx
    for ntx, nty in ((8, 4), (9, 63), (54094, 4), (8, 54094)):
        for perx, pery in ((0, 0), (1, 0), (0, 1)):
            assert rules.first_wrong_tile(ntx, nty, 1, pery, perx) == -1, (ntx, nty, perx, pery)


def test_region_tiles_where_the_quotient_is_exact(rules):
    """A whole region launch: right for every tile count that the launcher takes, and the launcher
    refuses counts for which the multiplication is not exact."""
    for ntx in list(range(1, 300)) + [511, 2526, 4445, 13334]:
        for nty in (1, 2, 7, 20):
            assert rules.divides_exactly(ntx * nty, ntx)
            assert rules.first_wrong_tile(ntx, nty, 0, 0, 0) == -1, (ntx, nty)
    assert rules.divides_exactly(46340 * 2, 46340) and not rules.divides_exactly(2 * 54094, 54094)
