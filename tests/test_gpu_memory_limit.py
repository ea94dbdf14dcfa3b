"""A context whose packed copies of X, X^T and H^T do not fit beside its workspace is created without
them and runs on the row-tiled kernels: the results are those of FIRAL_NT=0 to the bit, for products,
gradients and a Relax step, and a Round step still fits.
"""
import pytest
import torch

from paper_2409_07392_amd import RelaxContext, RoundSolver

pytestmark = pytest.mark.gpu

N, D, C, S = 600_000, 256, 8, 2
LEAVE = 900 << 20    # bytes left free: the packed form takes 1.2 GB of copies and more, the other 0.3


def outputs(ctx, B, om):
    w = torch.full((ctx.n_pool,), 1.0 / ctx.n_pool, dtype=torch.float64, device="cuda")
    g = torch.empty_like(w)
    ctx.relax_step(w, 20.0, 1e-2, 0.5, 7, 1, S, 0.0, 2, project=True, g_out=g)
    return [ctx.hvp(B, om, 0.25), ctx.grad_z(B, torch.sign(B)), w, g]


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_creation_without_packed_copies(prec, monkeypatch):
    gen = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(N, D, device="cuda", generator=gen)
    H = torch.softmax(torch.randn(N, C, device="cuda", generator=gen), 1)
    B = torch.randn(D, S, C, device="cuda", generator=gen)
    om = torch.rand(N, dtype=torch.float64, device="cuda", generator=gen)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    ctx = RelaxContext(X, H, N - 100, S, prec)
    packed = free0 - torch.cuda.mem_get_info()[0]
    ctx.close()
    with monkeypatch.context() as m:
        m.setenv("FIRAL_NT", "0")
        ctx = RelaxContext(X, H, N - 100, S, prec)
    tiled = free0 - torch.cuda.mem_get_info()[0]
    want = outputs(ctx, B, om)
    ctx.close()
    # bf16x3 contexts hold planes of X and X^T in either form
    leave = LEAVE if prec == "f32" else (packed + tiled) // 2
    torch.cuda.empty_cache()
    free1 = torch.cuda.mem_get_info()[0]
    assert tiled < leave < packed
    hog = torch.empty(free1 - leave, dtype=torch.uint8, device="cuda")
    try:
        ctx = RelaxContext(X, H, N - 100, S, prec)
    finally:
        del hog
        torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(outputs(ctx, B, om), want))
    rs = RoundSolver(ctx, torch.ones(N - 100, dtype=torch.float64, device="cuda"), 1e-2, 30.0, 2)
    rs.step(2)
    assert rs.result()["t"] == 2
    rs.close()
    ctx.close()
