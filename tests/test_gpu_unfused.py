"""FIRAL_UNFUSED=1 selects the row-tiled product and gradient on every shape, also those beyond the
fused kernels: the results are those of FIRAL_NT=0 to the bit, for probes cut into windows too, where
the packed products take their sums in another order.
"""
import numpy as np
import pytest
import torch

from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("d,c", [(132, 129), (200, 300), (392, 136)])
def test_unfused_is_row_tiled(d, c, prec, monkeypatch):
    p = make_small(n=900, n_lab=7, d=d, c=c, s=3, seed=d)
    X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
    r = np.random.default_rng(d)
    B = torch.as_tensor(r.standard_normal((d, 3, c)), dtype=torch.float32, device="cuda")
    om = torch.as_tensor(r.uniform(0.0, 2.0, p.N), device="cuda")
    out = []
    for var, val in (("FIRAL_UNFUSED", "1"), ("FIRAL_NT", "0"), (None, None)):
        with monkeypatch.context() as m:
            if var:
                m.setenv(var, val)
            ctx = RelaxContext(X, H, p.n_pool, 3, prec)
        out.append((ctx.hvp(B, om, 0.25), ctx.grad_z(B, torch.sign(B))))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    if d % (8 if prec == "bf16x3" else 4) == 0:   # windows: the packed products differ
        assert not torch.equal(out[0][0], out[2][0])
