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
