"""Build libdash.so (HIP, gfx950) in-tree.  `python -m paper_2302_06361_amd.build`"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
SO = os.path.join(HERE, "libdash.so")
GATE_SOURCES = ["dash_gates_cast.hip", "dash_gates_bit.hip", "dash_gates_chain.hip", "dash_gates.hip", "dash_gates_eval.hip", "dash_gates_digits_eval.hip", "dash_gates_digits.hip"]
SOURCES = ["dash_ctx.hip", "dash_layers.hip", "dash_linear.hip", "dash_gemm.hip", "dash_aesprof.hip"]
# (source, extra flags, object): the gate kernels once per label-length rule, the evaluator's whole layers also once per digit set
UNITS = []
for _rule, _flags in (("", []), ("_floor", ["-DDASH_RULE_FLOOR"])):
    UNITS += [(s, _flags, s.replace(".hip", _rule + ".o")) for s in GATE_SOURCES]
    UNITS += [("dash_act_eval.hip", _flags + ["-DDASH_SET=%d" % k], "dash_act_eval_%d%s.o" % (k, _rule)) for k in (12, 9, 8, 7)]
UNITS += [(s, [], s.replace(".hip", ".o")) for s in SOURCES]
HEADERS = ["dash_chain_rule.h", "dash_core.h", "dash_launch.h", "dash_bodies.h", "dash_gadget_rule.h", "dash_hostconst.h", "dash_internal.h", "dash_linear_rule.h", "dash_pack_rule.h", "dash_proj_rule.h", "dash_tabs.h", "dash_aes_sliced.h", "dash_sbox_circuit.h", os.path.join("..", "..", "include", "dash.h"),
           os.path.join("..", "..", "include", "dash_profile.h")]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function", "-Wno-pass-failed",
         # packed FP32 instructions are kept out of every code object of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build(force=True, verbose=False):
    """Compile every HIP source for gfx950 and link libdash.so.  Objects are rebuilt when a source
    or header is newer (or always with force)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    hdr_time = max(os.path.getmtime(os.path.join(CSRC, h)) for h in HEADERS)
    objs, todo = [], []
    for src, flags, obj in UNITS:
        s, o = os.path.join(CSRC, src), os.path.join(CSRC, obj)
        objs.append(o)
        if force or not os.path.exists(o) or os.path.getmtime(o) < max(os.path.getmtime(s), hdr_time):
            todo.append((obj, [hipcc] + FLAGS + flags + ["-c", s, "-o", o]))

    def compile_unit(item):
        if verbose:
            print(" ".join(item[1]))
        return item[0], subprocess.run(item[1], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)

    failed = False
    with ThreadPoolExecutor(min(16, os.cpu_count() or 1)) as ex:
        for obj, p in ex.map(compile_unit, todo):
            # the host pass does not know the packed-fp32 feature and says so: harmless
            out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
            if out.strip():
                print(out)
            if p.returncode != 0:
                failed = True
                print("FAILED:", obj)
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", SO] + objs)
    return SO


if __name__ == "__main__":
    build(force="--incremental" not in sys.argv, verbose=True)
    print("built", SO)
