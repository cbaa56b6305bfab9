"""Four lanes per planet (the step of small ensembles, wh_wide.h).

Its results equal the packing's own form bit for bit: a small batch stepped
alone must end where the same systems end inside a batch that is too large for
it.  The reverse pass of such a batch records in the same form, and the
forward run of wh_forward_ckpt records its last segment on the way.
"""
import numpy as np
import pytest
import torch

from paper_2307_05683_amd import inputs
from paper_2307_05683_amd.ensemble import Ensemble

pytestmark = pytest.mark.gpu

SCHEMES = [("dkd", 0.0, 0), ("dkd", 40.0, 0), ("kdk", 40.0, 0), ("kdk", 0.0, 1), ("saba3", 0.0, 0)]


def final(s, **kw):
    e = Ensemble.from_systems(s, **kw)
    e.step(1)
    e.step(40)
    out = [x.cpu().numpy() for x in (*e.state(), e.flags())]
    e.close()
    return out


def tiled(s, S):
    return s.subset(np.arange(S) % s.S)


# group sizes 8, 4, 2 and 1 lanes; one system, a partly filled wavefront and
# one group more than a wavefront holds
@pytest.mark.parametrize("scheme,gr_c,counts", SCHEMES)
@pytest.mark.parametrize("packing", ["pow2", "g8", "split"])
@pytest.mark.parametrize("S,lo,hi", [(1, 8, 8), (3, 5, 7), (9, 3, 4), (33, 2, 2), (65, 1, 1), (70, 1, 8)])
def test_small_batch_is_bitwise_the_large_one(packing, scheme, gr_c, counts, S, lo, hi):
    s = inputs.make_systems(S, 31, n_planets=None, n_range=(lo, hi), dt_mode="u15_30")
    kw = dict(packing=packing, scheme=scheme, gr_c=gr_c, kepler_counts=counts)
    big = {8: 4104, 4: 8200, 2: 16400, 1: 32800}[8 if hi > 4 or packing != "pow2" else 4 if hi > 2 else hi] * 2
    for a, b in zip(final(s, **kw), final(tiled(s, big), **kw)):
        assert np.array_equal(a, b[:S])


# and in Jacobi coordinates, whose scans cross the rows of a group
@pytest.mark.parametrize("scheme,gr_c", [("dkd", 0.0), ("kdk", 40.0), ("saba3", 40.0)])
@pytest.mark.parametrize("packing", ["pow2", "g8"])
@pytest.mark.parametrize("S,lo,hi", [(1, 8, 8), (3, 5, 7), (9, 3, 4), (33, 2, 2), (65, 1, 1)])
def test_small_jacobi_batch_is_bitwise_the_large_one(packing, scheme, gr_c, S, lo, hi):
    s = inputs.make_systems(S, 34, n_planets=None, n_range=(lo, hi), dt_mode="u15_30")
    kw = dict(packing=packing, scheme=scheme, gr_c=gr_c, coords="jacobi")
    big = {8: 4104, 4: 8200, 2: 16400, 1: 32800}[8 if hi > 4 or packing != "pow2" else 4 if hi > 2 else hi] * 2
    for a, b in zip(final(s, **kw), final(tiled(s, big), **kw)):
        assert np.array_equal(a, b[:S])


def test_trouble_stays_in_its_system():
    """Unbound, non-finite and coincident planets: flags and states as in the
    large batch, the neighbours' among them."""
    s = inputs.make_systems(24, 14, n_planets=None, n_range=(2, 8))
    s.V[3, 0] *= 3.0
    s.V[7, 1, 0] = np.nan
    s.Q[11, 1] = s.Q[11, 0]
    s.Q[15, 0, 2] = np.inf
    for packing in ("pow2", "split"):
        for a, b in zip(final(s, packing=packing), final(tiled(s, 9000), packing=packing)):
            assert np.array_equal(a, b[:24], equal_nan=a.dtype.kind == "f")


@pytest.mark.parametrize("packing", ["pow2", "split", "pair", "serial"])
@pytest.mark.parametrize("scheme,gr_c", [("dkd", 0.0), ("kdk", 40.0), ("saba2", 0.0)])
@pytest.mark.parametrize("n_steps,every", [(1, 1), (30, 30), (50, 20), (130, 40), (0, 5)])
def test_recorded_forward_run_is_the_stepped_one(packing, scheme, gr_c, n_steps, every):
    """wh_forward_ckpt ends bitwise where wh_step_n ends, and a second reverse
    pass of the tape (whose segment buffers the first has used) gives the
    first one's gradients."""
    s = inputs.make_systems(20, 32, n_planets=None, n_range=(2, 8))
    a = Ensemble.from_systems(s, packing=packing, scheme=scheme, gr_c=gr_c)
    b = Ensemble.from_systems(s, packing=packing, scheme=scheme, gr_c=gr_c)
    a.forward_ckpt(n_steps, every)
    b.step(n_steps)
    for x, y in zip((*a.state(), a.flags()), (*b.state(), b.flags())):
        assert torch.equal(x, y)
    Q, V = a.state()
    first = a.adjoint(2 * Q, V)
    for x, y in zip(first, a.adjoint(2 * Q, V)):
        assert torch.equal(x, y)
    a.step(7)
    b.step(7)
    assert torch.equal(a.state()[0], b.state()[0])
    a.close(); b.close()


def test_recorded_forward_run_in_jacobi_coordinates():
    s = inputs.make_systems(20, 33, n_planets=None, n_range=(1, 8))
    for scheme in ("dkd", "kdk", "saba2"):
        a = Ensemble.from_systems(s, coords="jacobi", scheme=scheme, gr_c=40.0)
        b = Ensemble.from_systems(s, coords="jacobi", scheme=scheme, gr_c=40.0)
        a.forward_ckpt(50, 20)
        b.step(50)
        for x, y in zip((*a.state(), a.flags()), (*b.state(), b.flags())):
            assert torch.equal(x, y)
        a.close(); b.close()
