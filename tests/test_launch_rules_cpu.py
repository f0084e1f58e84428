"""The rules that choose launches of several steps (mdf_internal.h), asked on
the CPU through a small program built from that header."""
import os
import shutil
import subprocess

import pytest

from paper_2108_08591_amd import mdf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"
STRIPS, SMALL, LARGE = 0, 1, 2
STORAGES = [mdf.F64, mdf.F32, mdf.F16DEV, mdf.BF16DEV]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(f"{ROCM}/include/hip"),
                                reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", f"{ROCM}/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2108_08591_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "native", "launch_rules.cpp")], check=True)

    def run(*questions):
        text = "\n".join(" ".join(str(int(w)) if not isinstance(w, str) else w for w in q) for q in questions)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [[float(v) for v in line.split()] for line in r.stdout.splitlines()]
    return run


def test_five_steps_only_where_the_kernel_keeps_its_registers(ask):
    """Five steps per launch in FP32 strips of plain cases; four with obstacles,
    a force field or Scheme II, whose five-step kernels spill, and elsewhere."""
    qs = [(c, s, m, g) for c in (STRIPS, SMALL, LARGE) for s in STORAGES for m in (0, 1) for g in (0, 1)]
    got = ask(*[("most",) + q for q in qs])
    for (c, s, m, g), (most,) in zip(qs, got):
        assert most == (5 if (c, s, m, g) == (STRIPS, mdf.F32, 0, 0) else 4), (c, s, m, g)
