"""The kernels' assembly.  Wait states: a vector instruction that writes VCC or another scalar register has to stand two wait states
before a vector instruction that reads it (gfx950); the compiler sees to that in its own code, but not inside inline assembly.  The base
conversions of every modulus with a compile-time description, compiled for gfx950 as the library's are.  No GPU involved."""
import os
import re
import subprocess

import pytest

from paper_2302_06361_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PROBE = """
#include "%s/dash_tabs.h"
using namespace dash;
#define KERNEL(MOD, LAM) \\
    __global__ void convert_##MOD##_##LAM(const U128* h, uint32_t* out) { \\
        const uint32_t i = threadIdx.x; \\
        decompress(CMod<MOD, LAM>{nullptr}, h[i], [&](int d, uint32_t w) { out[d * 64 + i] = w; }); \\
    }
DASH_HOT_MODS(KERNEL)
""" % build.CSRC


def scalars(operand):
    """indices of the scalar registers that an operand names (VCC as 106 and 107)"""
    operand = operand.strip()
    if operand == "vcc":
        return {106, 107}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


def violations(assembly):
    """(line, text) of vector instructions that read a scalar register too soon after a vector instruction wrote it; straight-line code"""
    bad, age = [], {}                                # scalar register -> wait states since a vector instruction wrote it
    for number, line in enumerate(assembly.splitlines(), 1):
        text = line.split(";")[0].strip()
        if re.match(r"[\w.$]+:", text):
            age = {}
            continue
        if not text or text.startswith("."):
            continue
        op, _, rest = text.partition(" ")
        operands = [o for o in re.split(r",(?![^\[]*\])", rest)]
        steps, written = 1, set()
        if op == "s_nop":
            steps = int(operands[0]) + 1
        elif op.startswith("v_"):
            dests = 2 if "_co_" in op or op.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale")) else 1
            read = set().union(*[scalars(o) for o in operands[dests:]])
            written = set().union(*[scalars(o) for o in operands[:dests]])
            if any(age.get(r, 2) < 2 for r in read):
                bad.append((number, text))
        age = {r: a + steps for r, a in age.items() if a + steps < 2}
        age.update({r: 0 for r in written})
    return bad


def test_the_check_itself():
    pair = "v_mad_u64_u32 v[0:1], vcc, v2, s3, v[0:1]\n%sv_addc_co_u32_e32 v4, vcc, 0, v4, vcc"
    assert violations(pair % "") and violations(pair % "s_nop 0\n") and not violations(pair % "s_nop 1\n")
    assert not violations(pair % "v_mov_b32_e32 v7, 0\nv_mov_b32_e32 v8, 0\n")
    other = "v_mad_u64_u32 v[0:1], s[10:11], v2, s3, v[0:1]\nv_addc_co_u32_e64 v4, s[%s], 0, v4, s[%s]"
    assert violations(other % ("10:11", "10:11")) and not violations(other % ("12:13", "12:13"))


@pytest.mark.parametrize("rule", ["", "-DDASH_RULE_FLOOR"])
def test_scalar_results_of_vector_instructions_in_the_base_conversions(tmp_path, rule):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    r = subprocess.run([HIPCC] + build.FLAGS + ([rule] if rule else []) + ["--cuda-device-only", "-S", str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    text = out.read_text()
    assert text.count("v_mad_u64_u32") > 300         # (the conversions are there)
    assert violations(text) == []


def test_the_run_time_garbler_keeps_its_scalars(tmp_path):
    """k_proj_garble for any modulus holds a modulus record and the launch's arguments in scalar registers; what these do not hold comes back from
    vector registers one instruction at a time, in the loop over the tiles (826 of them with the round keys held as well)"""
    src, out = tmp_path / "garble.hip", tmp_path / "garble.s"
    src.write_text('#include "%s/dash_tabs.h"\n#undef DASH_HOT_MODS\n#define DASH_HOT_MODS(X) X(2, 128)\n#include "%s/dash_gates.hip"\n' % (build.CSRC, build.CSRC))
    r = subprocess.run([HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    kernels = dict(re.findall(r"^(_Z\S*k_proj_garble\S*):(.*?)s_endpgm", out.read_text(), re.S | re.M))
    bodies = [v for k, v in kernels.items() if "7ModInfoELb1E" in k]
    assert len(bodies) == 1 and bodies[0].count("v_readlane_b32") < 200


def test_static_lds_of_the_deep_evaluator(tmp_path):
    """the table of the evaluator's deep form is read behind HalfTab::base bytes of static LDS: its kernels have as many"""
    out = str(tmp_path / "act.s")
    subprocess.run([HIPCC] + build.FLAGS + ["-DDASH_SET=7", "--cuda-device-only", "-S", os.path.join(build.CSRC, "dash_act_eval.hip"), "-o", out], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    kernels = re.findall(r"\.amdhsa_kernel (\S+)\s+\.amdhsa_group_segment_fixed_size (\d+)", open(out).read())
    deep = {name: int(size) for name, size in kernels if re.search(r"k_act_evalILb[01]ELi64ELi1E", name)}
    base = int(re.search(r"static constexpr uint32_t base = (\d+);", open(os.path.join(build.CSRC, "dash_tabs.h")).read()).group(1))
    assert len(deep) == 2 and set(deep.values()) == {base}, kernels
