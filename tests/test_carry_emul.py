"""The garbler's kernels for large batches of carry gates, the kernels themselves compiled for the host (tests/simt: a fiber per lane) with the
address and undefined-behaviour sanitizers, against garble_body: every access in bounds, every table byte equal, in both orders of the
lanes, for every pair of moduli that they are compiled for.  No GPU involved."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


@pytest.fixture(scope="module")
def emul(tmp_path_factory):
    """the program, once per label-length rule"""
    d = str(tmp_path_factory.mktemp("carry_emul"))
    exes = [os.path.join(d, name) for name in ("carry_emul", "carry_emul_floor")]
    procs = [subprocess.Popen([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                               os.path.join(HERE, "simt"), "-Wno-unknown-pragmas", "-Wno-pass-failed"] + flags +
                              [os.path.join(HERE, "carry_emul.cpp"), "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
             for exe, flags in zip(exes, ([], ["-DDASH_RULE_FLOOR"]))]
    for pr in procs:
        out, _ = pr.communicate()
        assert pr.returncode == 0, out[-3000:]
    return exes


@pytest.mark.parametrize("gates,quanta,blocks,jobs,reps", [
    (1, 1, 1, 1, 1),        # fewer rows than a tile
    (64, 1, 2, 1, 1),       # waves without a tile beside waves with one
    (130, 1, 1, 2, 2),      # several tiles a wave, several units a wave, a last tile that ends inside a gate
    (201, 2, 3, 1, 3),
    (300, 1, 1, 1, 1),      # up to 147 tiles over 3 waves
    (70, 0, 0, 2, 2),       # as launch_chain_garble splits it
])
def test_carry_gate_kernels(emul, gates, quanta, blocks, jobs, reps):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    for exe in emul:
        for order in ({}, {"SIMT_REVERSE": "1"}):
            r = subprocess.run([exe] + [str(v) for v in (gates, quanta, blocks, jobs, reps, gates + quanta)], capture_output=True, text=True, env=dict(env, **order))
            assert r.returncode == 0 and r.stdout.strip() == "ok", (order, r.stderr[-3000:])
