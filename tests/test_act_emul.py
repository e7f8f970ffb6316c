"""The repacking of tables (k_rows_repack), the kernel itself compiled for the host (tests/simt: a fiber per lane) with the address
and undefined-behaviour sanitizers, against the oracle over exactly-sized buffers: every access in bounds and aligned as its type
says, every byte equal.  No GPU involved."""
import os
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import workloads
from oracle import capi

HERE = os.path.dirname(os.path.abspath(__file__))
SEED = bytes(range(31, 47))
KIND = dict(relu=4, scale=5, sign=6)
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
FLAGS = ["-x", "c++", "-std=c++17", "-O1", "-g1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", os.path.join(HERE, "simt"),
         "-include", "hip/hip_runtime.h", "-Wno-unknown-pragmas", "-Wno-pass-failed", "-c", os.path.join(HERE, "act_emul.cpp")]


@pytest.fixture(scope="module")
def emul(tmp_path_factory):
    """the program, its parts compiled side by side"""
    d = str(tmp_path_factory.mktemp("act_emul"))
    units = {"main": []}
    for rule, flag in ((0, []), (1, ["-DDASH_RULE_FLOOR"])):
        units["gates%d" % rule] = ["-DPART_GATES"] + flag
        for k in (7, 8, 9, 12):
            units["act%d_%d" % (k, rule)] = ["-DPART_ACT", "-DDASH_SET=%d" % k] + flag

    def compile_unit(item):
        return subprocess.run([CLANG] + FLAGS + item[1] + ["-o", os.path.join(d, item[0] + ".o")], capture_output=True, text=True)
    with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as ex:
        for r in ex.map(compile_unit, units.items()):
            assert r.returncode == 0, r.stderr[-3000:]
    exe = os.path.join(d, "act_emul")
    subprocess.check_call([CLANG, "-fsanitize=address,undefined", "-o", exe] + [os.path.join(d, u + ".o") for u in units])
    return exe


def run(emul, tmp_path, mode, k, rule, kind, n, repeat=1, layer=5, in_place=False, elem_base=0, env=None):
    """-> (output bytes, oracle, its labels before and after, its tables)"""
    primes, digits = workloads.PRIMES[:k], workloads.DIGITS[k]
    orc = capi.Oracle(primes, digits, SEED, rule)
    x = np.random.default_rng(n * 100 + k).integers(0, orc.P, n)
    zero = [orc.input_labels(9, n, i) for i in range(k)]
    act = [orc.encode(i, x, zero[i]) for i in range(k)]
    if kind == "relu":
        _, rt = orc.relu_garble(layer, zero, elem_base)
        want = orc.relu_eval(layer, act, rt, elem_base)
    else:
        _, rt = orc.scale_garble(layer, zero, repeat, elem_base)
        want = orc.scale_eval(layer, act, rt, repeat, elem_base)
    blob = struct.pack("<8iQ", k, rule, KIND[kind], n, repeat, layer, int(in_place), len(digits), elem_base)
    blob += np.array(primes, np.uint16).tobytes() + np.array(digits, np.uint16).tobytes() + SEED
    blob += b"".join(a.tobytes() for a in act) + rt.tobytes()
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    open(fin, "wb").write(blob)
    e = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0", **(env or {}))
    r = subprocess.run([emul, mode, fin, fout], capture_output=True, text=True, env=e)
    assert r.returncode == 0, r.stderr[-3000:]
    return np.fromfile(fout, np.uint8), orc, want, rt


@pytest.mark.parametrize("k,kind,n,repeat", [(8, "relu", 3, 1), (8, "scale", 67, 2), (12, "relu", 65, 1), (7, "scale", 17, 1)])
def test_tables_repacked_from_a_4_byte_address(emul, tmp_path, k, kind, n, repeat):
    """tables are 4-byte aligned, and with an odd number of values so is the segment of every modulus"""
    got, orc, _, rt = run(emul, tmp_path, "pack", k, 1, kind, n, repeat=repeat)
    want = orc.tables_pack(kind, n, rt, repeat)
    assert got.size == want.size + rt.size
    assert (got[:want.size] == want).all(), "packed bytes"
    assert (got[want.size:] == rt).all(), "unpacked tables"
