"""The forward run of reverse mode: it ends where stepping ends, whatever the
exchange, and leaves no recording behind a run that no gradient can follow."""
import numpy as np
import pytest
import torch

from paper_2307_05683_amd import ensemble, inputs
from paper_2307_05683_amd.ensemble import Ensemble

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("packing", ["pow2", "g8"])
@pytest.mark.parametrize("scheme,gr_c,coords", [("dkd", 0.0, "dhc"), ("kdk", 40.0, "dhc"), ("saba2", 0.0, "dhc"),
                                                ("dkd", 40.0, "jacobi")])
@pytest.mark.parametrize("n_steps,every", [(30, 30), (50, 20)])
def test_lds_exchange_ends_where_stepping_ends(packing, scheme, gr_c, coords, n_steps, every):
    s = inputs.make_systems(40, 51, n_planets=None, n_range=(3, 8))
    kw = dict(packing=packing, scheme=scheme, gr_c=gr_c, coords=coords, exchange="lds")
    a, b = Ensemble.from_systems(s, **kw), Ensemble.from_systems(s, **kw)
    a.forward_ckpt(n_steps, every)
    b.step(n_steps)
    for x, y in zip((*a.state(), a.flags()), (*b.state(), b.flags())):
        assert torch.equal(x, y)
    Q, V = a.state()
    for x, y in zip(a.adjoint(2 * Q, V), a.adjoint(2 * Q, V)):
        assert torch.equal(x, y)
    a.close(); b.close()


@pytest.mark.parametrize("scheme", ["dkd", "saba2"])
def test_integrate_records_only_for_gradients(monkeypatch, scheme):
    """Without a gradient to follow, integrate() writes no step of a tape
    (10 rows per slot and step; checkpoints are 12 per slot) and returns the
    same state; what it refuses, it refuses either way."""
    s = inputs.make_systems(24, 52, n_planets=8)
    t = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")  # noqa: E731
    x = [t(s.Q), t(s.V), t(s.m), t(s.m0)]
    bufs = []
    empty = torch.empty

    def zeros(*a, **kw):       # memory that shows what was written
        b = empty(*a, **kw).zero_()
        bufs.append(b)
        return b

    def written(*args, **kw):
        bufs.clear()
        with monkeypatch.context() as mp:
            mp.setattr(ensemble.torch, "empty", zeros)
            out = ensemble.integrate(*args, t(s.dt), s.n_planets, 200, ckpt_every=100, scheme=scheme, packing="g8", **kw)
        torch.cuda.synchronize()
        return out, sum(int(torch.count_nonzero(b)) for b in bufs if b.dtype == torch.uint8)

    leaf = [y.clone().requires_grad_(True) for y in x]
    ref, recorded = written(*leaf)
    plain, n_plain = written(*x)
    with torch.no_grad():
        off, n_off = written(*leaf)
    rows = 24 * 8 * 10 * 8     # bytes of one recorded step
    assert recorded > 50 * rows
    assert n_plain < 20 * rows and n_off < 20 * rows
    for a, b, c in zip(ref, plain, off):
        assert torch.equal(a.detach(), b) and torch.equal(b, c) and a.requires_grad and not c.requires_grad
    for kw, n, every in ((dict(packing="mixed"), 10, 5), (dict(kepler_counts=1), 10, 5), ({}, 10, 0), ({}, -1, 5),
                         ({}, (1 << 62) + 3, 1)):
        for v in (x, leaf):
            with pytest.raises(ensemble._lib.WHError):
                ensemble.integrate(*v, t(s.dt), s.n_planets, n, ckpt_every=every, **kw)
