"""How the tiles of packed table rows are dealt to waves (dash_pack_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    lib = C.CDLL(so)

    def call(tiles, nseg, pack):
        blocks = C.c_uint32()
        return lib.cc_pack_shape(C.c_uint64(tiles), nseg, int(pack), C.byref(blocks)), blocks.value
    return call


@pytest.mark.parametrize("pack", [True, False])
def test_few_tiles_side_by_side_and_no_waves_for_the_walk_alone(shape, pack):
    """up to 8 192 tiles no wave does two in a row while places are left; below 2^16 no more waves than are resident at a time"""
    resident = 1024 if pack else 1792
    for nseg in (5, 20, 28, 60, 96):
        if not pack and nseg <= 27:
            continue
        for tiles in (1, 3, 700, 4096, 8191):
            assert shape(tiles, nseg, pack) == (0, resident)
        for tiles in (8192, 16383):
            assert shape(tiles, nseg, pack) == (1, resident)
        for tiles in (16384, (1 << 16) - 1):
            assert shape(tiles, nseg, pack) == (2, resident)
        assert shape(1 << 40, nseg, pack) == (2, 4096 if pack else 1792)
    # more blocks than are resident only where a wave has tiles enough for its walk
    for nseg in (20, 60, 96):
        for tiles in (1 << 16, 100000, 1 << 18, (1 << 20) - 1, 1 << 20):
            run, blocks = shape(tiles, nseg, True)
            assert run == 2 and (blocks <= 1536 or tiles >= 3072 * nseg)


def test_a_short_walk_is_paid_for_every_tile(shape):
    for nseg in (1, 5, 27):
        for tiles in (1, 8192, 1 << 16, 1 << 30):
            assert shape(tiles, nseg, False) == (0, 32768 if nseg <= 15 else 4096)
