"""Even shares of long launches: both parts of a cut wave never in one launch
(the partition on the CPU, under the rules that launches use), and the same
bits as in launches too short for shares."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM_INC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def test_cut_waves_run_in_different_slices(tmp_path):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM_INC, "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or HIP headers not available")
    exe = str(tmp_path / "even_share_cuts_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INC,
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2307_05683_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "even_share_cuts_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "even share cuts ok" in r.stdout, r.stdout


# eight-planet ensembles whose bins' ends fall next to a step's: 1079 waves in
# 20 slices of 1024 bins, and 2171 waves in two bins per SIMD
@pytest.mark.gpu
@pytest.mark.parametrize("S", [8632, 17368])
def test_long_shares_keep_the_bits(S):
    from paper_2307_05683_amd import inputs
    from paper_2307_05683_amd.ensemble import Ensemble
    s = inputs.make_systems(500, 42, n_planets=8).subset(np.arange(S) % 500)
    out = []
    for parts in ((4096,), (50,) * 81 + (46,)):
        e = Ensemble.from_systems(s)
        for n in parts:
            e.step(n)
        out.append([x.cpu().numpy() for x in (*e.state(), e.flags())])
        e.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
