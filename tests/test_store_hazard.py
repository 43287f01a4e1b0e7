"""The four-float partial store (csrc/pa_device.h: store_partial4) is inline
assembly, for which the compiler's hazard recognizer adds no wait states: after
a vector store of more than 64 bits this GPU needs two before a VALU
instruction overwrites the stored registers (the compiler puts two after its
own stores).  A kernel that overwrites them at once is compiled for gfx950 and
the wait states in the store's own block are counted; no GPU is used."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
WAIT_STATES = 2

SOURCE = """
#include "pa_device.h"
extern "C" __global__ void stores(float* dst, float x) {
  float v[4] = {x, x + 1.f, x + 2.f, x + 3.f};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    pa::store_partial4(dst + 4 * (threadIdx.x + 64 * i), v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = v[j] * 1.5f + 1.f;
  }
}
"""


def wait_states_after_stores(lines):
    """For every 128-bit vector store: the wait states that follow it whatever
    the compiler schedules next."""
    found = []
    for at, line in enumerate(lines):
        if line.startswith("global_store_dwordx4"):
            states = 0
            for nxt in lines[at + 1:]:
                m = re.fullmatch(r"s_nop (\d+)", nxt)
                if not m:
                    break
                states += int(m[1]) + 1
            found.append(states)
    return found


def test_two_wait_states_after_the_partial_store(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    (tmp_path / "stores.hip").write_text(SOURCE)
    cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2510_14126_amd", "csrc"), "-S", "--cuda-device-only",
           "stores.hip", "-o", "stores.s"]
    r = subprocess.run(cmd, cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = [x.split(";")[0].strip().replace("\t", " ") for x in (tmp_path / "stores.s").read_text().splitlines()]
    found = wait_states_after_stores([x for x in lines if x and x[0] not in ".#" and not x.endswith(":")])
    assert len(found) == 8 and min(found) >= WAIT_STATES, found
