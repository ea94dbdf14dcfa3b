"""The tuner on bf16x3 contexts whose own tiling does not cover the shape (d <= 128, 128 < c <= 256
with one column block a wave): it may still choose two blocks a wave, by timing or from a choice that
another context of the bucket made, and the planes which that kernel reads are there.  Products
against the FP64 oracle at the bar of the bf16x3 products, 1e-4.
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxBatch, RelaxContext, default_beta0
from synthdata import make_small

pytestmark = pytest.mark.gpu


def setup(d, c, seed):
    p = make_small(n=700, n_lab=5, d=d, c=c, s=3, seed=seed)
    X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
    B = np.random.default_rng(seed).standard_normal((d, 3, c)).astype(np.float32)
    ref = orc.hvp(X.cpu().numpy().astype(np.float64), H.cpu().numpy().astype(np.float64), None, 0.25,
                  B.astype(np.float64))
    return p, X, H, torch.as_tensor(B, device="cuda"), ref


def check(ctx, B, ref):
    out = ctx.hvp(B, shift=0.25).cpu().numpy()
    assert np.linalg.norm(out - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("first", ["narrow", "wide"])
@pytest.mark.parametrize("d,c", [(40, 200), (128, 256), (33, 129)])
def test_tuned_narrow_context(d, c, first, monkeypatch):
    # "wide": a context of the default tiling has already left its choice for the bucket
    p, X, H, B, ref = setup(d + (first == "wide"), c, d + c) if d < 128 else setup(d, c, d + c)
    if first == "wide":
        wide = RelaxContext(X, H, p.n_pool, 3, "bf16x3")
        wide.autotune(3)
        check(wide, B, ref)
    monkeypatch.setenv("FIRAL_FUSED_MAX_NCB", "1")
    ctx = RelaxContext(X, H, p.n_pool, 3, "bf16x3")
    check(ctx, B, ref)
    ctx.autotune(3)
    check(ctx, B, ref)


def test_batch_of_narrow_context(monkeypatch):
    monkeypatch.setenv("FIRAL_FUSED_MAX_NCB", "1")
    p, X, H, B, ref = setup(48, 150, 9)
    ctx = RelaxContext(X, H, p.n_pool, 3, "bf16x3")
    w = torch.full((p.n_pool,), 1.0 / p.n_pool, dtype=torch.float64, device="cuda")
    batch = RelaxBatch([dict(ctx=ctx, w=w, b=20.0, lam=1e-2, beta0=default_beta0(p.n_pool, 3), seed=1,
                             tol=1e-4, max_iter=40)])
    batch.run(2)
    assert batch.info(0)["bad_block"] == -1
    assert abs(float(w.sum()) - 1.0) <= 1e-12
    check(ctx, B, ref)
