"""Which kernels garble the gates of a sign gadget (dash_gadget_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    return C.CDLL(so)


def test_one_copy_of_the_tables_for_different_digits_of_few_primes(lib):
    for k in range(2, 16):
        assert lib.cc_digits_banked(1, 1, k) and lib.cc_digits_banked(1, 0, k) and lib.cc_digits_banked(0, 1, k)
        assert bool(lib.cc_digits_banked(0, 0, k)) == (k > 5)
