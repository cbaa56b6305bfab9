"""Even shares of a launch: the partition on the CPU, and that a run cut this
way ends in the bits of the same run in launches too short for it."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM_INC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def test_partition(tmp_path):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM_INC, "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or HIP headers not available")
    exe = str(tmp_path / "even_shares_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INC,
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2307_05683_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "even_shares_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "even shares ok" in r.stdout, r.stdout


# one bin per SIMD (two waves on the busiest), two bins with three and with four
@pytest.mark.gpu
@pytest.mark.parametrize("S,lo,hi", [(10000, 8, 8), (20011, 1, 8), (20000, 8, 8), (40011, 1, 8)])
@pytest.mark.parametrize("scheme,gr_c", [("dkd", 0.0), ("kdk", 40.0), ("saba2", 0.0)])
def test_shares_keep_the_bits(S, lo, hi, scheme, gr_c):
    from paper_2307_05683_amd import inputs
    from paper_2307_05683_amd.ensemble import Ensemble
    s = inputs.make_systems(500, 41, n_planets=None, n_range=(lo, hi), dt_mode="u15_30").subset(np.arange(S) % 500)
    out = []
    for parts in ((500, 411), (50,) * 18 + (11,)):
        e = Ensemble.from_systems(s, scheme=scheme, gr_c=gr_c)
        for n in parts:
            e.step(n)
        out.append([x.cpu().numpy() for x in (*e.state(), e.flags())])
        e.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
