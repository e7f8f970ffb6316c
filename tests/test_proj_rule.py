"""Which launches the evaluator's independent projection gates take (dash_proj_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
BANKED = 1 << 20


@pytest.fixture(scope="module")
def own(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    lib = C.CDLL(so)
    return lambda q, gates, calls=1, bits_only=False, alone=True, banked=BANKED: bool(
        lib.cc_proj_own(q, C.c_uint64(calls), C.c_uint64(gates), int(bits_only), int(alone), C.c_uint64(banked)))


def test_one_pair_of_moduli_takes_the_faster_kernel(own):
    """batches of one pair, where the shared kernel measured slower by more than a few per cent have launches of their own"""
    for n in (1, 10 ** 4, 10 ** 5, 4 * 10 ** 5, 1 << 20, 1 << 22):
        assert own(2, n) and own(2, n, bits_only=True)
    for q in (3, 5, 7, 17, 37):
        assert own(q, 1) and own(q, 10 ** 5)
    for q in (7, 17, 37):
        assert own(q, 1 << 22) and own(q, 1 << 21) and not own(q, 1 << 20) and own(q, 1 << 20, bits_only=True)
        assert not own(q, 4 * 10 ** 5)
    for q in (3, 5):
        assert not own(q, 1 << 18) and not own(q, 1 << 22)


def test_mixed_moduli_share_launches_unless_a_modulus_fills_the_chip(own):
    for q in (2, 3, 5, 7, 37):
        assert not own(q, 1000, alone=False) and not own(q, 10 ** 4, calls=12, alone=False)
    assert own(2, 1 << 18, calls=12, alone=False) and not own(2, (1 << 18) - 1, calls=12, alone=False)
    assert own(37, 1 << 22, calls=12, alone=False) and not own(37, 350000, calls=12, alone=False)
    # many small calls: 16 to a launch of its own, 64 to a shared one
    assert not own(2, 10 ** 6, calls=1000, alone=False) and not own(2, 10 ** 6, calls=1000) and not own(3, 1000, calls=17)
    assert own(37, 1 << 22, calls=32, alone=False) and not own(37, 1 << 22, calls=33, alone=False)


def test_the_banked_threshold_moves_the_line(own):
    assert own(7, 2, alone=False, banked=1) and not own(7, 1, alone=False, banked=1) and own(7, 1, bits_only=True, alone=False, banked=1)
    assert not own(7, 1 << 40, alone=False, banked=1 << 60)
