"""The pipelined fused product (one column block a wave) at its edges: chunks that end early, one to
three chunks a row range (the pipeline's fill and drain), every padding of d in a 16-block, one and
eight column blocks, c at the lines between the compiled Gamma steps and staging sizes (16, 17, 32,
33, 128), rows without weights, a prefix of the rows; in FP64 also shapes past its LDS (the row-tiled
kernels).  Against the FP64 oracle, normwise: FP32 the bar of the fused kernels, 1e-5; FP64 1e-12
(sums of at most a few thousand terms per partial, each rounded at 1.1e-16).
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("shape", [
    (31, 0, 1, 2, 3), (33, 0, 16, 2, 64), (8100, 3, 17, 16, 8), (16500, 0, 100, 10, 12),
    (9000, 5, 33, 17, 7), (500, 2, 97, 32, 4), (700, 1, 128, 33, 3), (300, 7, 127, 128, 2),
    (24700, 1, 64, 5, 25),
])
def test_fused_pipe_matches_oracle(shape, prec):
    n, nl, d, c, s = shape
    p = make_small(n=n, n_lab=nl, d=d, c=c, s=s, seed=d + c)
    dt, bar = (torch.float32, 1e-5) if prec == "f32" else (torch.float64, 1e-12)
    X, H = (torch.as_tensor(a, dtype=dt, device="cuda") for a in (p.X, p.H))
    r = np.random.default_rng(c)
    B = r.standard_normal((d, s, c)).astype(np.float32)
    om = r.uniform(0.0, 2.0, p.N)
    ctx = RelaxContext(X, H, p.n_pool, s, prec)
    Bd = torch.as_tensor(B, dtype=dt, device="cuda")
    for rows in (p.N, p.N - p.N // 3):
        for w in (None, om[:rows]):
            wd = None if w is None else torch.as_tensor(w, device="cuda")
            out = ctx.hvp(Bd, omega=wd, shift=0.25, n_rows=rows).cpu().numpy()
            ref = orc.hvp(X.cpu().numpy()[:rows].astype(np.float64),
                          H.cpu().numpy()[:rows].astype(np.float64), w, 0.25,
                          B.astype(np.float64))
            assert np.linalg.norm(out - ref) <= bar * np.linalg.norm(ref), (rows, w is None)
