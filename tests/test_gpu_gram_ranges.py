"""The Gram blocks from packed operands in one range of stages and in several, every class-block count
of a workgroup, both row orders, with tiles cut between workgroups and without.

Each shape's splits, stages and ranges are computed here from the rules of the host code, and the test
asserts that its two contexts differ in their ranges; the blocks are equal to the bit all the same.
Against the oracle: the FP32 bar of the other forms (1e-5 on the blocks, through L L^T).
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxContext
from synthdata import make_small

pytestmark = pytest.mark.gpu


def cdiv(a, b):
    return -(-a // b)


def plan(N, d, c, s, rows):
    """Units, workgroup slots, stages of 32 rows a split and stages a range (FP32)."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    wide = c > 64 and d % 4 == 0
    if wide:
        tc, br = 128, 4 * 4
    else:
        cb, wc = (1, 1) if c <= 16 else (1, 2) if c <= 32 else (2, 2) if c <= 64 else (4, 2)
        tc, br = 16 * cb * wc, 4 * (4 // wc)
    nab = cdiv(d, 16)
    pairs = sum(1 for a in range(nab) for b in range(cdiv(d, br)) if b * br <= 16 * a + 15)
    wgs, blk = pairs * cdiv(c, tc), c * d * d * 4
    if wide and wgs >= 2 * n_cu:
        S = 1
        for t in range(2, min(8, max(1, (4 << 30) // blk)) + 1):
            if cdiv(wgs * t, 2 * n_cu) * S < cdiv(wgs * S, 2 * n_cu) * t:
                S = t
    else:
        S = max(1, min(cdiv(1024, wgs), 64, max(1, (1 << 28) // blk)))
    nct = cdiv(c, 128)
    cmw = cdiv(cdiv(c, nct), 16)
    stages = cdiv(cdiv(N, S), 32)
    stage = S * (nct * cmw + nab) * 2048
    G = max(rows * s * c * 4, 16384 + stage * min(32, stages))
    if d > 128:
        G = max(G, cdiv(s * c, 128) * 128 * cdiv(rows, 128) * 128 * 4)
    per_cu = 7 if cmw <= 1 else 5 if cmw <= 2 else 4 if cmw <= 3 else 3 if cmw <= 5 else 2
    return nct * nab * (nab + 1) // 2 * S, n_cu * per_cu, stages, min(stages, (G - 16384) // stage), cmw


@pytest.mark.parametrize("n,d,c,cmw,cut", [
    (1400, 1000, 10, 1, True), (1300, 830, 20, 2, True), (1300, 735, 40, 3, True),
    (1300, 640, 60, 4, True), (25000, 100, 20, 2, False), (17000, 130, 64, 4, False),
    (50000, 100, 70, 5, True),        # wide order, as the next and every d % 4 == 0 with c > 64
    (50000, 100, 90, 6, True), (26000, 101, 90, 6, True), (26000, 101, 100, 7, True),
    (32000, 132, 128, 8, True), (17000, 129, 128, 8, True), (11000, 132, 300, 7, True),
    (11000, 256, 90, 6, True),
])
def test_ranges_to_the_bit(n, d, c, cmw, cut, monkeypatch):
    p = make_small(n=n, n_lab=3, d=d, c=c, s=1, seed=d + c)
    one, several = plan(p.N, d, c, 128, p.N), plan(p.N, d, c, 1, 128)
    assert one[4] == cmw and (one[0] > one[1]) == cut
    assert one[3] == one[2] > 32 and several[3] == 32
    X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
    om = np.random.default_rng(c).uniform(0.0, 1.0, p.N)
    w = torch.as_tensor(om, device="cuda")
    L, Pinv, info = RelaxContext(X, H, p.n_pool, 128, "f32").build_precond(w, shift=1e-1)
    assert info["bad_block"] == -1
    monkeypatch.setenv("FIRAL_CHUNK_ROWS", "128")
    L1, Pinv1, _ = RelaxContext(X, H, p.n_pool, 1, "f32").build_precond(w, shift=1e-1)
    assert torch.equal(L, L1) and torch.equal(Pinv, Pinv1)
    P = orc.precond_blocks(p.X, p.H, om, 1e-1)
    LL = torch.bmm(L, L.transpose(1, 2).contiguous()).cpu().numpy()
    assert np.linalg.norm(LL - P) <= 1e-5 * np.linalg.norm(P)
