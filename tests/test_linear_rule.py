"""The choice of the kernel of a dense or convolution layer (dash_linear_rule.h), compiled for the host.  No GPU involved."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
TILE4, TILE8, SPLIT, MFMA, TILE1, ROW1, ROW2, ROW4 = 1, 2, 3, 4, 5, 6, 7, 8
CHANNELS = {SPLIT: 8, ROW1: 1, ROW2: 2, ROW4: 4}
LANES = {SPLIT: 64, ROW1: 16, ROW2: 16, ROW4: 16}
CHUNKS = {7: 29, 8: 31, 9: 33, 12: 39}      # 16-digit chunks of the labels of the first k primes


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "core_check.cpp")])
    lib = C.CDLL(so)

    def f(npx, out_c, K, k=8, mfma=False, forced=0, in_c=16):
        return lib.cc_linear_form(forced, C.c_int64(npx), C.c_int64(CHUNKS[k]), 8, out_c, K, in_c, int(mfma))
    f.lib = lib
    return f


def lanes(f, npx, out_c):
    return npx * ((out_c + CHANNELS[f] - 1) // CHANNELS[f]) * 8 * LANES[f]


def test_split_forms_only_where_a_grid_holds_them(form):
    """a wave or a row of lanes per (pixel, chunk, block of channels): fewer than 2^32 lanes, whatever asks for the form"""
    assert form(2 ** 22 - 1, 16, 64, forced=SPLIT) == SPLIT
    assert form(2 ** 22, 16, 64, forced=SPLIT) == TILE8               # 2^22 * 2 * 8 waves = 2^32 lanes
    assert form(2 ** 25 - 1, 1, 64, forced=ROW1) == ROW1 and form(2 ** 25, 1, 64, forced=ROW1) == TILE8
    for e in range(31):
        for out_c in (1, 2, 3, 4, 5, 9, 257, 4097):
            for K in (1, 64, 257, 70000):
                for forced in (0, SPLIT, ROW1, ROW2, ROW4):
                    for mfma in (False, True):
                        for in_c in (1, 9):
                            f = form(2 ** e, out_c, K, mfma=mfma, forced=forced, in_c=in_c) if 2 ** e * out_c < 2 ** 31 else 0
                            assert f not in LANES or lanes(f, 2 ** e, out_c) < 2 ** 32, (2 ** e, out_c, K, mfma, forced)


def test_few_channels_take_a_form_for_few_channels(form):
    """up to four channels: a row of lanes, or a lane per pixel where neighbouring pixels share cache lines; a wave for a long reduction"""
    assert form(64 * 784, 1, 25, in_c=1) == TILE1 and form(64 * 784, 2, 25, in_c=1) == TILE4
    assert form(784, 1, 288, in_c=32) == ROW1 and form(784, 2, 288, in_c=32) == ROW2 and form(784, 4, 288, in_c=32) == ROW4
    assert form(2048, 1, 100, in_c=100) == ROW1
    assert form(1, 1, 4096, k=12, in_c=4096) == SPLIT                 # (a chain of 64 loads by a row of lanes, of 16 by a wave)


# (batch or pixels, out_c, K, primes) of the MFMA tests on the GPU
MFMA_SHAPES = [(5, 300, 500, 12), (7, 257, 128, 8), (3, 70, 1030, 12), (2, 96, 4096, 12), (1, 70, 13000, 12), (2, 40, 13000, 12), (3, 130, 250, 8),
               (3, 130, 192, 8), (108, 70, 100, 8), (25, 64, 64, 8), (256, 48, 108, 12), (40, 40, 108, 12), (40, 100, 192, 8)]


def test_mfma_form_can_be_forced_where_its_tiles_fit(form):
    """several of the MFMA tests' layers are small enough for k_linear_split to be the faster one: they need the hook"""
    chosen = [form(npx, out_c, K, k, mfma=True) for npx, out_c, K, k in MFMA_SHAPES]
    assert SPLIT in chosen and form(128, 4096, 4096, 12, mfma=True) == MFMA
    for npx, out_c, K, k in MFMA_SHAPES:
        assert form(npx, out_c, K, k, mfma=True, forced=MFMA) == MFMA
        assert form(npx, out_c, K, k, mfma=False, forced=MFMA) == form(npx, out_c, K, k, mfma=False) != MFMA
