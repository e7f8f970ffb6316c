"""The evaluator's deep form reads its AES table at a literal address behind HalfTab::base bytes of static LDS: every build of its kernels (digit sets and
label-length rules) has as many.  No GPU involved."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2302_06361_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_static_lds_of_every_deep_kernel(tmp_path):
    base = int(re.search(r"static constexpr uint32_t base = (\d+);", open(os.path.join(build.CSRC, "dash_tabs.h")).read()).group(1))
    units = [u for u in build.UNITS if u[0] == "dash_act_eval.hip"]
    assert len(units) == 8

    def sizes(unit):
        out = str(tmp_path / unit[2].replace(".o", ".s"))
        subprocess.run([HIPCC] + build.FLAGS + unit[1] + ["--cuda-device-only", "-S", os.path.join(build.CSRC, unit[0]), "-o", out], check=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        kernels = re.findall(r"\.amdhsa_kernel (\S+)\s+\.amdhsa_group_segment_fixed_size (\d+)", open(out).read())
        return [int(size) for name, size in kernels if re.search(r"k_act_evalILb[01]ELi64ELi1E", name)]
    with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as ex:
        assert list(ex.map(sizes, units)) == [[base, base]] * 8
