"""The evaluator's one-launch activation layers (k_act_eval), the repacking of tables (k_rows_repack) and the linear layers, the kernels themselves
compiled for the host (tests/simt: a fiber per lane) with the address and undefined-behaviour sanitizers, against the oracle over
exactly-sized buffers: every access in bounds and aligned as its type says, every byte equal, in both orders of the lanes.  No GPU
involved."""
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
         "-Wno-unknown-pragmas", "-Wno-pass-failed", "-c", os.path.join(HERE, "act_emul.cpp")]
BIG = "1000000000"
LINEAR_FORMS = ["1", "2", "3", "5", "6", "7", "8"]


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
    run.stderr = r.stderr
    return np.fromfile(fout, np.uint8), orc, want, rt


@pytest.mark.parametrize("form", ["tiny", "shallow", "deep"])
@pytest.mark.parametrize("k", [7, 8, 9, 12])
@pytest.mark.parametrize("rule", [0, 1])
def test_one_launch_activation_layers(emul, tmp_path, k, rule, form):
    env = {"DASH_ACT_SHALLOW_MIN_ELEMS": BIG if form == "tiny" else "0", "DASH_ACT_DEEP_MIN_ELEMS": "0" if form == "deep" else BIG}
    per_block = dict(tiny=2 if k < 9 else 1, shallow=16, deep=64)[form]
    for kind, n, in_place in (("relu", per_block + 1, False), ("scale", per_block + 1, True), ("relu", 1, True)):
        for order in ({}, {"SIMT_REVERSE": "1"}):
            got, orc, want, _ = run(emul, tmp_path, "act", k, rule, kind, n, repeat=2 if kind == "scale" else 1, in_place=in_place,
                                    elem_base=2 ** 32 - 2, env=dict(env, **order))
            ref = np.concatenate([a.reshape(-1) for a in want])
            bad = np.flatnonzero(got != ref)
            assert got.size == ref.size and bad.size == 0, (kind, n, order, bad[:1])


@pytest.mark.parametrize("k,n_digits", [(8, 13), (8, 14), (7, 16), (12, 16)])
def test_deep_layers_whose_digit_sums_exceed_the_table_span(emul, tmp_path, monkeypatch, k, n_digits):
    """the same moduli with more digits: 67 to 85 dwords of sums, 64 lie beside the deep form's tables; large layers keep that form"""
    monkeypatch.setitem(workloads.DIGITS, k, workloads.DIGITS[k][:2] + workloads.DIGITS[k][1:2] * (n_digits - 2))
    rows = {13: 67, 14: 72, 16: 75 if k == 7 else 74}[n_digits]       # (16 digits: 85 and 81 dwords, the last ten in the free half of rows 64 to 73)
    env = {"DASH_ACT_SHALLOW_MIN_ELEMS": "0", "DASH_ACT_DEEP_MIN_ELEMS": "0", "SIMT_TRACE": "1"}
    for kind, n in (("relu", 65), ("scale", 17)):
        got, orc, want, _ = run(emul, tmp_path, "act", k, 0, kind, n, env=env)
        assert (got == np.concatenate([a.reshape(-1) for a in want])).all(), kind
        assert "grid %d 1 1 block %d lds %d" % ((n + 63) // 64, 64 * (k if kind == "relu" else k - 1), rows * 1024) in run.stderr


@pytest.mark.parametrize("k,kind,n,repeat", [(8, "relu", 3, 1), (8, "scale", 67, 2), (12, "relu", 65, 1), (7, "scale", 17, 1)])
def test_tables_repacked_from_a_4_byte_address(emul, tmp_path, k, kind, n, repeat):
    """tables are 4-byte aligned, and with an odd number of values so is the segment of every modulus"""
    got, orc, _, rt = run(emul, tmp_path, "pack", k, 1, kind, n, repeat=repeat)
    want = orc.tables_pack(kind, n, rt, repeat)
    assert got.size == want.size + rt.size
    assert (got[:want.size] == want).all(), "packed bytes"
    assert (got[want.size:] == rt).all(), "unpacked tables"


def test_deep_form_with_another_static_lds_is_refused(emul, tmp_path):
    """its table would lie elsewhere than where the kernel reads it; the other forms don't mind"""
    env = {"SIMT_STATIC_LDS": "1040", "DASH_ACT_SHALLOW_MIN_ELEMS": "0", "DASH_ACT_DEEP_MIN_ELEMS": "0"}
    for kind in ("relu", "scale"):
        with pytest.raises(AssertionError, match="not implemented"):
            run(emul, tmp_path, "act", 7, 0, kind, 65, env=env)
        run(emul, tmp_path, "act", 7, 0, kind, 65, env=dict(env, DASH_ACT_DEEP_MIN_ELEMS=BIG))


@pytest.mark.parametrize("run_log2,kind,n", [(0, "scale", 240), (1, "relu", 5), (2, "scale", 67), (2, "relu", 3), (3, "scale", 67), (3, "relu", 5)])
def test_tables_repacked_in_runs_of_tiles(emul, tmp_path, run_log2, kind, n):
    """waves that take 1, 2, 4 and 8 tiles of 64 rows at a time (by the number of tiles; here forced): segments that end within a run, within the tiles
    that are read together and within a tile; 240 values: more runs than waves"""
    got, orc, _, rt = run(emul, tmp_path, "pack", 8, 1, kind, n, env={"DASH_PACK_RUN_LOG2": str(run_log2)})
    want = orc.tables_pack(kind, n, rt, 1)
    assert got.size == want.size + rt.size
    assert (got[:want.size] == want).all(), "packed bytes"
    assert (got[want.size:] == rt).all(), "unpacked tables"


def run_linear(emul, tmp_path, form, k, batch, in_h, in_w, in_c, out_c, kh, stride, pad, bias, garble=False, shift=0, seed=1):
    primes, digits = workloads.PRIMES[:k], workloads.DIGITS[k]
    orc = capi.Oracle(primes, digits, SEED, 0)
    g = np.random.default_rng(seed)
    x = [workloads.uniform_labels(g, batch * in_h * in_w * in_c, orc.lam(p), p) for p in primes]
    W = g.integers(-64, 64, (out_c, kh, kh, in_c)).astype(np.int32)
    b = g.integers(-1000, 1000, out_c).astype(np.int32)
    ones = [orc.one0(i) if garble else orc.one(i) for i in range(k)]
    want = [orc.conv2d(i, x[i], batch, in_h, in_w, in_c, out_c, kh, kh, stride, pad, W, b if bias else None, ones[i]) for i in range(k)]
    blob = struct.pack("<14i", k, 0, batch, in_h, in_w, in_c, out_c, kh, stride, pad, int(bias), int(garble), shift, len(digits))
    blob += np.array(primes, np.uint16).tobytes() + np.array(digits, np.uint16).tobytes() + SEED
    blob += b"".join(a.tobytes() for a in x) + W.tobytes() + b.tobytes()
    fin, fout = str(tmp_path / "lin.bin"), str(tmp_path / "lout.bin")
    open(fin, "wb").write(blob)
    e = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0", DASH_LINEAR_FORM=form)
    r = subprocess.run([emul, "linear", fin, fout], capture_output=True, text=True, env=e)
    assert r.returncode == 0, r.stderr[-3000:]
    ref = np.concatenate([a.reshape(-1) for a in want])
    got = np.fromfile(fout, np.uint8)
    bad = np.flatnonzero(got != ref)
    assert got.size == ref.size and bad.size == 0, bad[:1]


@pytest.mark.parametrize("form", LINEAR_FORMS)
def test_linear_layers(emul, tmp_path, form):
    """every kernel but the MFMA one at the edges of its blocks: channels and taps that do not fill them, taps in the padding, weights
    at odd addresses"""
    for i, (K, out_c) in enumerate(((1, 1), (3, 2), (5, 3), (16, 4), (17, 5), (255, 8), (257, 9), (33, 33))):
        run_linear(emul, tmp_path, form, 3, 3, 1, 1, K, out_c, 1, 1, 0, bias=i % 2 == 0, garble=i % 3 == 0, shift=i % 2, seed=50 + i)
    run_linear(emul, tmp_path, form, 4, 2, 6, 7, 3, 3, 3, 2, 1, True)
    run_linear(emul, tmp_path, form, 4, 1, 5, 5, 7, 2, 5, 1, 2, True, garble=True)
    run_linear(emul, tmp_path, form, 4, 1, 4, 4, 65, 7, 2, 2, 0, False, shift=2)
