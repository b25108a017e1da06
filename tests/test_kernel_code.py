"""What the compiler made of the kernels whose time hangs on it, read from the assembly of our own sources (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2206_01288_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")

    def of(source):
        out = str(tmp_path_factory.mktemp("asm") / "out.asm")
        subprocess.run([HIPCC] + build.FLAGS + build.FILE_FLAGS.get(source, []) +
                       ["-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
        return open(out).read()

    return of


def body(text, kernel):
    m = re.search(r"^(_Z\S*%s\S*):.*?^\.Lfunc_end" % kernel, text, re.M | re.S)
    assert m is not None, kernel
    return m.group(0)


def test_gathers_of_a_block_are_in_flight_together(assembly):
    # the lane's sixteen codes: at least eight loads before the first wait for one of them
    text = assembly("dtfm_eval.hip")
    for kernel in ("7k_match", "12k_eval_small"):
        code = re.findall(r"^\s+(global_load_ushort|s_waitcnt vmcnt\(\d+\)|s_waitcnt vmcnt\(\d+\) lgkmcnt\(\d+\))",
                          body(text, kernel), re.M)
        runs, run = [], 0
        for i in code:
            if i == "global_load_ushort":
                run += 1
            else:
                runs.append(run)
                run = 0
        assert max(runs) >= 8, (kernel, runs)
