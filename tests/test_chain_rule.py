"""How the tiles of carry gates are dealt to waves (dash_chain_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
QUANTA = {96: 3, 26: 13, 204: 51, 46: 23, 91: 91, 10: 5, 90: 45, 22: 11}      # modulus -> tiles after which a lane comes back to its value


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    return C.CDLL(so)


def test_few_candidates_find_what_all_of_them_would(lib):
    rng = random.Random(4)
    sizes = [1, 2, 3, 44, 45, 46, 8191, 8192, 8193, 30600, 112896] + [int(2 ** (26 * rng.random())) for _ in range(60)]
    most = 0
    for quantum in QUANTA.values():
        for units in (1, 2, 5, 6, 7, 9, 16, 24, 60, 160, 256):
            for resident in (8192, 64):
                for tiles in sizes:
                    tried = C.c_uint32()
                    got = lib.cc_chain_waves(C.c_uint64(tiles), units, quantum, resident, C.byref(tried))
                    assert got == lib.cc_chain_waves_all(C.c_uint64(tiles), units, quantum, resident), (tiles, units, quantum, resident)
                    assert got % quantum == 0 and got > 0
                    if resident == 8192 and tiles * units < 2 ** 20:      # 64 M rows in a launch
                        most = max(most, tried.value)
    assert most <= 100
