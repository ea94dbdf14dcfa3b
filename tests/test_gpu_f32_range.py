"""firal_hvp in FP32 contexts beyond the fused kernels holds FP32's whole range: values near its
smallest and its largest, with the other factors chosen so that no product or sum leaves the range.
An output sums its terms in two FP32 contractions of K = d and K = r roundings of 2^-24 for splits of
r rows: 2^-24 (sqrt(d) + sqrt(r)) is below 2.4e-6 for d <= 200, r <= 705; the bar is 4e-6 normwise
against the FP64 oracle.
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", ["1", "0"])                        # packed, row-tiled
@pytest.mark.parametrize("d,c", [(200, 40), (132, 129)])          # one form of the row step each
@pytest.mark.parametrize("x,b,w", [(1e-36, 1e10, 1e30), (1e38, 1e-20, 1e-25)])
def test_product_over_the_fp32_range(x, b, w, d, c, nt, monkeypatch):
    monkeypatch.setenv("FIRAL_NT", nt)
    p = make_small(n=700, n_lab=5, d=d, c=c, s=4, seed=52)
    r = np.random.default_rng(d)
    X = r.uniform(1.0, 2.0, p.X.shape) * r.choice([-1.0, 1.0], p.X.shape) * x
    if x > 1.0:   # the largest values that FP32 has
        X[r.random(X.shape) < 0.02] = np.finfo(np.float32).max
    X, H = X.astype(np.float32), p.H.astype(np.float32)
    B = (r.standard_normal((d, 4, c)) * b).astype(np.float32)
    om = r.uniform(0.5, 2.0, p.N) * w
    dev = lambda a, dt=torch.float32: torch.as_tensor(a, dtype=dt, device="cuda")
    ctx = RelaxContext(dev(X), dev(H), p.n_pool, 4, "f32")
    got = ctx.hvp(dev(B), dev(om, torch.float64)).cpu().numpy().astype(np.float64)
    want = orc.hvp(X.astype(np.float64), H.astype(np.float64), om, 0.0, B.astype(np.float64))
    assert np.isfinite(want).all() and np.abs(want).max() < np.finfo(np.float32).max
    assert np.linalg.norm(got - want) <= 4e-6 * np.linalg.norm(want)
