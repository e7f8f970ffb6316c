"""The garbler's kernel for gates on one wire of modulus 2 (casts; evaluator's halves and known inputs of the half gates), the kernel itself compiled
for the host (tests/simt: a fiber per lane) with the address and undefined-behaviour sanitizers, against garble_body: every access in
bounds, every table byte equal, in both orders of the lanes, for every prime with a compile-time description.  No GPU involved."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


@pytest.fixture(scope="module")
def emul(tmp_path_factory):
    """the program, once per label-length rule"""
    d = str(tmp_path_factory.mktemp("bit_emul"))
    exes = [os.path.join(d, name) for name in ("bit_emul", "bit_emul_floor")]
    procs = [subprocess.Popen([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                               os.path.join(HERE, "simt"), "-Wno-unknown-pragmas", "-Wno-pass-failed"] + flags +
                              [os.path.join(HERE, "bit_emul.cpp"), "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
             for exe, flags in zip(exes, ([], ["-DDASH_RULE_FLOOR"]))]
    for pr in procs:
        out, _ = pr.communicate()
        assert pr.returncode == 0, out[-3000:]
    return exes


@pytest.mark.parametrize("gates,jobs,reps,slot", [
    (1, 1, 1, 0),           # two rows
    (128, 12, 1, 60),       # a whole tile; every prime
    (129, 11, 2, 250),      # a second tile of two rows; slots whose upper 24 bits change between the jobs; repetitions
    (300, 16, 1, 70),       # as many jobs as a launch carries
])
def test_gates_on_a_bit_wire(emul, gates, jobs, reps, slot):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    for exe in emul:
        for order in ({}, {"SIMT_REVERSE": "1"}):
            r = subprocess.run([exe] + [str(v) for v in (gates, jobs, reps, slot, gates + jobs)], capture_output=True, text=True, env=dict(env, **order))
            assert r.returncode == 0 and r.stdout.strip() == "ok", (order, r.stderr[-3000:])


@pytest.mark.parametrize("gates,jobs,reps,slot,groups,blocks", [
    (9000, 16, 1, 249, 0, 0),     # dealt out by the launcher: two jobs per lane, a lane whose slots change their upper 24 bits
    (129, 11, 2, 250, 1, 3),      # all jobs in one lane, such slots among them and in a repetition of its own
    (300, 16, 2, 245, 1, 1),      # a second tile, and a second round of tiles, for every wave
    (257, 11, 1, 250, 3, 2),       # groups of four jobs, a last one of three
    (130, 12, 1, 254, 4, 1),
])
def test_several_jobs_per_lane(emul, gates, jobs, reps, slot, groups, blocks):
    """a lane's jobs share the first rounds of their hashes; both kinds of half-gate jobs with every prime, masks of all its digits"""
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    for exe in emul:
        for order in ({}, {"SIMT_REVERSE": "1"}) if groups else ({},):
            r = subprocess.run([exe] + [str(v) for v in (gates, jobs, reps, slot, gates + jobs, groups, blocks)], capture_output=True, text=True, env=dict(env, **order))
            assert r.returncode == 0 and r.stdout.strip() == "ok", (order, r.stderr[-3000:])
