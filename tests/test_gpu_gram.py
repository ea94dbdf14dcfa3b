"""The Gram blocks from packed operands at the edges of their tiles: one to eight class blocks, one
and several class tiles, pair tiles cut by d, both row orders, splits that end inside a stage, units
cut between workgroups, and operands packed a range of stages at a time.

A small row chunk leaves the operands little scratch, so that the sums go through memory between
ranges: the same sums in the same order, equal to the bit.  Against the oracle: the FP32 bar of the
other forms (1e-5 on the blocks, through L L^T).
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("shape", [
    (33000, 5, 20, 5), (40001, 0, 33, 37), (20000, 3, 47, 64),
    (9000, 7, 100, 100),      # 7 class blocks, wide order
    (17000, 3, 129, 129),     # two class tiles of 5 blocks, units cut between workgroups
    (9100, 2, 132, 300),      # three class tiles of 7 blocks
    (8300, 9, 129, 128),      # 8 class blocks, classic order
])
def test_gram_matches_oracle_and_its_ranges(shape, prec, monkeypatch):
    n, nl, d, c = shape
    p = make_small(n=n, n_lab=nl, d=d, c=c, s=1, seed=d + c)
    X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
    om = np.random.default_rng(c).uniform(0.0, 1.0, p.N)
    w = torch.as_tensor(om, device="cuda")
    L, Pinv, info = RelaxContext(X, H, p.n_pool, 1, prec).build_precond(w, shift=1e-3)
    assert info["bad_block"] == -1
    monkeypatch.setenv("FIRAL_CHUNK_ROWS", "128")
    L1, Pinv1, _ = RelaxContext(X, H, p.n_pool, 1, prec).build_precond(w, shift=1e-3)
    assert torch.equal(L, L1) and torch.equal(Pinv, Pinv1)
    P = orc.precond_blocks(p.X, p.H, om, 1e-3)
    LL = torch.bmm(L, L.transpose(1, 2).contiguous()).cpu().numpy()
    assert np.linalg.norm(LL - P) <= 1e-5 * np.linalg.norm(P)
