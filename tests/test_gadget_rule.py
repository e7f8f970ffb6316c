"""Which kernels garble the gates of a sign gadget (dash_gadget_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MAX_JOBS = 16


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    return C.CDLL(so)


def test_one_copy_of_the_tables_for_different_digits_of_few_primes(lib):
    for k in range(2, 16):
        assert lib.cc_digits_banked(1, 1, k) and lib.cc_digits_banked(1, 0, k) and lib.cc_digits_banked(0, 1, k)
        assert bool(lib.cc_digits_banked(0, 0, k)) == (k > 5)


def test_gates_on_a_bit_wire_have_a_launch_of_their_own_where_it_is_no_launch_more(lib):
    def own(bits, others, rows, few):
        return bool(lib.cc_bits_own(bits, others, C.c_uint64(rows), int(few), MAX_JOBS))
    # ReLU of k primes: 2 k of them beside k others; scaling: k - 1 casts
    for k in range(2, 16):
        more = -(-2 * k // MAX_JOBS) + -(-k // MAX_JOBS) > -(-3 * k // MAX_JOBS)
        assert own(2 * k, k, 1000, True) == own(2 * k, k, 599999, True) == (not more)
        assert own(2 * k, k, 600000, True) and own(2 * k, k, 1 << 21, False)
        assert own(k - 1, 0, 1000, True) == own(k - 1, 0, 1 << 20, True) == (k >= 5) and own(k - 1, 0, 1 << 21, False)
    assert [k for k in range(2, 13) if own(2 * k, k, 1000, True)] == [6, 7, 8, 11, 12]
    assert not own(0, 5, 1000, True) and not own(0, 5, 1 << 21, False)
