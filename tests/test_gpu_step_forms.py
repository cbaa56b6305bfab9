"""The forms of a large ensemble's step against one another, bit for bit.

Even shares are taken by balanced and by unbalanced runs, so the reference
side here steps in calls too short for them (fewer than 128 kicks), each one
launch of the packing's own kernel; which form a call takes comes from the
library's rule (native/step_form.cpp) and is asserted.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2307_05683_amd import inputs
from paper_2307_05683_amd.ensemble import PACKINGS, SCHEMES, Ensemble

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM_INC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM_INC, "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or HIP headers not available")
    so = str(tmp_path_factory.mktemp("form") / "step_form.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INC,
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2307_05683_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "step_form.cpp"), "-o", so], check=True)
    f = ctypes.CDLL(so).step_form_launches

    def query(s, packing, scheme, gr_c, n_steps):
        n = np.ascontiguousarray(s.n_planets, dtype=np.int32)
        return f(s.S, n.ctypes.data_as(ctypes.c_void_p), PACKINGS[packing], SCHEMES[scheme], int(gr_c > 0),
                 4 * torch.cuda.get_device_properties(0).multi_processor_count, n_steps)
    return query


def run(s, parts, **kw):
    e = Ensemble.from_systems(s, **kw)
    windows = e.launch_windows
    for n in parts:
        e.step(n)
    out = [x.cpu().numpy() for x in (*e.state(), e.flags(), e.energy())]
    e.close()
    return out, windows


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def batch(S, lo, hi, seed):
    return inputs.make_systems(500, seed, n_planets=None, n_range=(lo, hi), dt_mode="u15_30").subset(np.arange(S) % 500)


CHUNK, N, SHORT = 1024, 1024 + 333, 50     # SHORT: below 128 kicks for SABA_2 too


@pytest.mark.parametrize("packing,scheme,gr_c", [("pow2", "dkd", 0.0), ("pow2", "dkd", 40.0), ("pow2", "kdk", 0.0),
                                                 ("pow2", "kdk", 40.0), ("pow2", "saba2", 0.0), ("mixed", "dkd", 0.0),
                                                 ("mixed", "dkd", 40.0), ("mixed", "kdk", 0.0), ("mixed", "kdk", 40.0)])
def test_even_shares_balanced_or_not_are_the_plain_step(launches, packing, scheme, gr_c):
    s = batch(16384, 2, 8, 61)
    kw = dict(packing=packing, scheme=scheme, gr_c=gr_c, chunk_steps=CHUNK)
    assert launches(s, packing, scheme, gr_c, CHUNK) > 1 and launches(s, packing, scheme, gr_c, SHORT) == 1
    plain, w = run(s, [SHORT] * (N // SHORT) + [N % SHORT], **kw)
    assert w == (1, 0)
    shares, w = run(s, [N], **kw)
    assert w == (1, 0)
    same(shares, plain)
    balanced, w = run(s, [N], balance=1, **kw)
    assert w[0] > 1 and w[1] >= 1024
    same(balanced, plain)


# several waves of shared groups on a SIMD: balanced launches stay windows
@pytest.mark.parametrize("scheme,gr_c", [("dkd", 0.0), ("kdk", 40.0)])
def test_windows_of_shared_groups_are_the_plain_step(scheme, gr_c):
    s = batch(35000, 2, 6, 62)
    kw = dict(packing="mixed", scheme=scheme, gr_c=gr_c, chunk_steps=CHUNK)
    plain, _ = run(s, [SHORT] * (N // SHORT) + [N % SHORT], **kw)
    windows, w = run(s, [N], balance=1, block_waves=4, **kw)
    assert w[0] > 1 and w[1] >= 2048
    same(windows, plain)


# Tiled past the four-lane form, an ensemble's gradients come from the kernels
# with a lane per planet: the same forward bits, and gradients that differ by
# the order of their sums.  A step's adjoint is about 500 dependent roundings
# of 1.1e-16 and the growth of 60 steps' products is within a factor of ten of
# the result's norm: 60 * 500 * 1.1e-16 * 10 = 3e-11 of the system's norm.
@pytest.mark.parametrize("scheme,gr_c", [("dkd", 0.0), ("kdk", 40.0), ("saba2", 0.0)])
@pytest.mark.parametrize("packing,lo,hi,big", [("pow2", 5, 8, 2100), ("pow2", 3, 4, 4200), ("pow2", 2, 2, 8300),
                                               ("pow2", 1, 1, 16500), ("g8", 2, 8, 2100), ("split", 2, 8, 2100)])
def test_large_gradients_are_the_small_ones(packing, lo, hi, big, scheme, gr_c):
    small = inputs.make_systems(30, 63, n_planets=None, n_range=(lo, hi), dt_mode="u15_30")
    idx = np.arange(big) % 30
    live = np.arange(8)[None, :, None] < small.n_planets[:, None, None]
    w = np.random.default_rng(64).normal(size=(2, 30, 8, 3)) * live
    out = []
    for s, k in ((small, np.arange(30)), (small.subset(idx), idx)):
        e = Ensemble.from_systems(s, packing=packing, scheme=scheme, gr_c=gr_c)
        e.forward_ckpt(60, 25)
        Q, V = e.state()
        out.append([x.cpu().numpy() for x in (Q, V, e.flags(), *e.adjoint(w[0][k], w[1][k]))])
        e.close()
    a, b = out
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x[idx], y)
    for name, x, y in zip(("gQ", "gV", "gm", "gm0"), a[3:], b[3:]):
        x = x.reshape(30, -1)
        d = np.abs(x[idx] - y.reshape(big, -1)).max(axis=1)
        n = np.abs(x).max(axis=1)[idx]
        print("%s: largest difference %.2e of the system's norm" % (name, (d / n).max()), flush=True)
        assert np.all(d <= 3e-11 * n)


def test_balanced_shares_fit_the_kernel_that_runs_them():
    """Kick-drift-kick with GR in the mixed packing: the kernel of even shares
    holds three wavefronts per SIMD (157 registers), the packing's own kernel
    four; a plan of 5001 wavefronts over four would run in two rounds."""
    s = batch(40008, 8, 8, 65)
    kw = dict(packing="mixed", scheme="kdk", gr_c=40.0, chunk_steps=CHUNK)
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    shares, w = run(s, [N], balance=1, **kw)
    assert w[0] > 1 and w[1] == 3 * simds
    plain, _ = run(s, [SHORT] * (N // SHORT) + [N % SHORT], **kw)
    same(shares, plain)
