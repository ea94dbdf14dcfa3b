"""The Gram blocks from packed operands at the edges of their tiles: one to eight class blocks, one
and several class tiles, pair tiles cut by d, both row orders, splits that end inside a stage, units
cut between workgroups, and operands packed a range of stages at a time.

A small row chunk leaves the operands little scratch, so that the sums go through memory between
ranges: the same sums in the same order, equal to the bit.  Against the oracle: the FP32 bar of the
other forms (1e-5 on the blocks, through L L^T).
"""
import threading

import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import RelaxBatch, RelaxContext, default_beta0
from synthdata import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("shape", [
    (33000, 5, 20, 5), (40001, 0, 33, 37), (20000, 3, 47, 64),
    (9000, 7, 100, 100),      # 7 class blocks, wide order
    (17000, 3, 129, 129),     # two class tiles of 5 blocks
    (17000, 3, 256, 100),     # units cut between workgroups (1088 on 512 slots), wide order
    (17000, 3, 255, 100),     # the same (544 units), classic order
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


def test_gram_in_concurrent_streams_and_replays():
    # two contexts on two streams at once (their workgroups share the device), and the same work in a
    # captured graph replayed several times, each equal to the bit to a context on its own
    shapes = [(17000, 3, 256, 100), (17000, 3, 255, 100)]   # units cut in both
    outs, ctxs, ws = [], [], []
    for n, nl, d, c in shapes:
        p = make_small(n=n, n_lab=nl, d=d, c=c, s=1, seed=d + c)
        X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
        ctx = RelaxContext(X, H, p.n_pool, 1, "f32")
        w = torch.as_tensor(np.random.default_rng(c).uniform(0.0, 1.0, p.N), device="cuda")
        outs.append(ctx.build_precond(w, shift=1e-2, want_L=False)[1])
        ctxs.append(ctx)
        ws.append(w)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in shapes]

    def run(i, got):
        with torch.cuda.stream(streams[i]):
            for _ in range(4):
                got.append((i, ctxs[i].build_precond(ws[i], shift=1e-2, want_L=False)[1]))

    got = []
    ths = [threading.Thread(target=run, args=(i, got)) for i in range(len(shapes))]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    torch.cuda.synchronize()
    assert len(got) == 8 and all(torch.equal(P, outs[i]) for i, P in got)


def test_gram_in_a_replayed_batch():
    # the counters and flags of the cut units start anew in every replay of a captured step
    p = make_small(n=17000, n_lab=3, d=256, c=100, s=1, seed=5)
    X, H = (torch.as_tensor(a, dtype=torch.float32, device="cuda") for a in (p.X, p.H))
    a, b = (RelaxContext(X, H, p.n_pool, 1, "f32") for _ in range(2))
    wa = torch.full((p.n_pool,), 1.0 / p.n_pool, dtype=torch.float64, device="cuda")
    wb = wa.clone()
    beta0 = default_beta0(p.n_pool, 30)
    batch = RelaxBatch([dict(ctx=a, w=wa, b=50.0, lam=1e-2, beta0=beta0, seed=3, t0=1, s=1, tol=1e-4,
                             max_iter=30, project=True)])
    b.autotune(1)
    for t in range(1, 4):
        batch.run(1)
        torch.cuda.synchronize()
        b.relax_step(wb, 50.0, 1e-2, beta0, 3, t, 1, 1e-4, 30, project=True)
        assert torch.allclose(wa, wb, rtol=1e-12, atol=0.0), t
