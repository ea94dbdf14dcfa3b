"""Products on both sides of the lines between their kernels, against the FP64 oracle: the packed and
the row-tiled FP32 form for wide probes at d <= 128 (2048 rows), and the one-pass and the row-tiled
FP64 form for c > 64 (rows times probes of 50,000).  Normwise; FP32 1e-5 and FP64 1e-12, the bars of
the same kernels' other tests.
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


def check(n, d, c, s, rows, prec, bar):
    p = make_small(n=n, n_lab=3, d=d, c=c, s=s, seed=d + c)
    dt = torch.float64 if prec == "f64" else torch.float32
    X, H = (torch.as_tensor(a, dtype=dt, device="cuda") for a in (p.X, p.H))
    r = np.random.default_rng(c)
    B = r.standard_normal((d, s, c)).astype(np.float32)
    om = r.uniform(0.0, 2.0, p.N)
    ctx = RelaxContext(X, H, p.n_pool, s, prec)
    Xo, Ho = X.cpu().numpy().astype(np.float64), H.cpu().numpy().astype(np.float64)
    for k in rows:
        out = ctx.hvp(torch.as_tensor(B, dtype=dt, device="cuda"),
                      torch.as_tensor(om[:k], device="cuda"), 0.25, n_rows=k).cpu().numpy()
        ref = orc.hvp(Xo[:k], Ho[:k], om[:k], 0.25, B.astype(np.float64))
        assert np.linalg.norm(out - ref) <= bar * np.linalg.norm(ref), k


@pytest.mark.parametrize("d,c,s", [(40, 300, 2), (128, 129, 3), (7, 513, 1)])
def test_wide_probes_at_the_row_line(d, c, s):
    check(2200, d, c, s, (1, 2047, 2048, 2049, 2203), "f32", 1e-5)


@pytest.mark.parametrize("d,c,s", [(22, 128, 25), (30, 65, 20), (9, 64, 30)])
def test_fp64_probes_beyond_half_a_tile_at_the_row_line(d, c, s):
    k = 50000 // s
    check(k + 50, d, c, s, (k - 1, k, k + 1, k + 53), "f64", 1e-12)
