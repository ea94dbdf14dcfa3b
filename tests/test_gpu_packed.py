"""The packed-operand products (gemm_pk.hip) at the edges of their tiles.

Shapes: d around the 16- and 32-wide operand blocks and the output tiles (128 / 256 / 384 rows),
c from 2 to several 128-column tiles (probes narrower than, equal to and wider than a tile, the
64-class line of the row sums), row counts around the 32-row stages and 128-row tiles, row chunks
that no tile divides, FP32 and bf16x3, pool rows only.

Tolerances.  firal_hvp in FP32 takes six bf16-plane products per FP32 product: each operand is
exact in its planes, the dropped products are below 3 x 2^-25 of a product, and an output sums its
terms in FP32 in two contractions, K = 6 d / 32 and K = 6 r / 32 roundings of 2^-24 for splits of r
rows: 2^-24 (3 + sqrt(6 d / 32) + sqrt(6 r / 32)) is below 1.5e-6 for d <= 520, r <= 600; the bar is
4e-6 normwise.  bf16x3 drops 2^-16 relative: 1e-4, as elsewhere.
Inside a solve the products keep the rounding of the row-tiled kernels (FIRAL_NT=0) for probes cut
without windows; the two differ only in the order of FP64 sums: 1e-9.
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu

TOL = {"f32": 4e-6, "bf16x3": 1e-4}

SHAPES = [  # n_pool, n_lab, d, c, s, chunk rows
    (1000, 3, 129, 2, 3, None),      # one feature beyond the fused kernels, narrowest probes
    (129, 0, 144, 5, 1, None),       # one row beyond a row tile, one ragged column tile
    (31, 1, 130, 63, 3, None),       # less than one 32-row stage of pool rows
    (700, 5, 203, 64, 5, "300"),     # the 64-class line, chunks no tile divides
    (641, 2, 256, 127, 2, "129"),
    (600, 33, 257, 128, 3, None),    # probes equal to a tile; first shape of three-block waves
    (533, 9, 383, 129, 2, "200"),    # probes one column wider than a tile
    (777, 4, 385, 37, 7, None),      # more than one output row tile
    (900, 7, 132, 129, 3, None),     # windows: a one-column last window
    (650, 6, 392, 300, 2, "333"),    # windows, two output row tiles, chunks
    (500, 5, 40, 300, 2, None),      # d <= 128 with probes wider than a fused tile
]


def dev(a, dt=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def problem(shape, seed):
    n, nl, d, c, s, _ = shape
    p = make_small(n=n, n_lab=nl, d=d, c=c, s=s, seed=seed, whiten_x=True, probs="maxprob")
    r = np.random.default_rng(seed)
    X, H = p.X.astype(np.float32), p.H.astype(np.float32)
    B = r.standard_normal((d, s, c)).astype(np.float32)
    om = r.uniform(0.0, 2.0, p.N)
    return p, X, H, B, om


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("shape", SHAPES)
def test_product_matches_oracle(shape, prec, monkeypatch):
    if shape[5]:
        monkeypatch.setenv("FIRAL_CHUNK_ROWS", shape[5])
    p, X, H, B, om = problem(shape, 51)
    n = p.n_pool
    ctx = RelaxContext(dev(X), dev(H), n, p.s, prec)
    X, H, B64 = X.astype(np.float64), H.astype(np.float64), B.astype(np.float64)
    got = ctx.hvp(dev(B), dev(om, torch.float64), 0.25).cpu().numpy()
    assert relerr(got, orc.hvp(X, H, om, 0.25, B64)) <= TOL[prec]
    got = ctx.hvp(dev(B), n_rows=n).cpu().numpy()
    assert relerr(got, orc.hvp(X[:n], H[:n], None, 0.0, B64)) <= TOL[prec]
    again = ctx.hvp(dev(B), n_rows=n).cpu().numpy()
    assert np.array_equal(got, again)
    # no rows at all: the shift alone
    got = ctx.hvp(dev(B), n_rows=0, shift=2.0).cpu().numpy()
    assert np.array_equal(got, 2.0 * B)


@pytest.mark.parametrize("scale", [1e-18, 1e15])
def test_three_planes_hold_the_fp32_range(scale):
    # operands far from 1: the planes of an FP32 value keep its 24 bits at any exponent in use
    p, X, H, B, om = problem((700, 5, 200, 40, 4, None), 52)
    X, B = (X * np.float32(scale)), (B * np.float32(scale ** -0.5))
    ctx = RelaxContext(dev(X), dev(H), p.n_pool, p.s, "f32")
    got = ctx.hvp(dev(B), dev(om, torch.float64)).cpu().numpy().astype(np.float64)
    want = orc.hvp(X.astype(np.float64), H.astype(np.float64), om, 0.0, B.astype(np.float64))
    assert relerr(got, want) <= TOL["f32"]


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("shape", SHAPES)
def test_solves_and_gradient_keep_the_row_tiled_rounding(shape, prec, monkeypatch):
    if shape[5]:
        monkeypatch.setenv("FIRAL_CHUNK_ROWS", shape[5])
    p, X, H, B, om = problem(shape, 53)
    d, c = shape[2], shape[3]
    windows = d > 128 and c > 128 and d % (8 if prec == "bf16x3" else 4) == 0
    out = []
    for nt in ("0", "1"):
        monkeypatch.setenv("FIRAL_NT", nt)
        ctx = RelaxContext(dev(X), dev(H), p.n_pool, p.s, prec)
        w = torch.full((p.n_pool,), 1.0 / p.n_pool, dtype=torch.float64, device="cuda")
        g = torch.empty_like(w)
        ctx.relax_step(w, 20.0, 1e-2, 0.5, 7, 1, p.s, 0.0, 2, project=True, g_out=g)
        out.append((ctx.grad_z(dev(np.sign(B)), dev(B)).cpu().numpy(), g.cpu().numpy()))
    assert relerr(out[1][0], out[0][0]) <= 1e-9
    # with windows the row sums are taken in another order than the row-tiled kernels'
    assert relerr(out[1][1], out[0][1]) <= (2e-4 if windows else 1e-9)
