"""The block inverse on FP64 MFMA tiles (128 < d <= 576, no factor asked for) at its edges.

Sizes: one feature into a new 16-block, full blocks, the last size of the row form (256), the first
and last of the panel form (257, 576) and the first size past it (577).  With the factor asked for,
the sweeps without MFMA give the inverse: the same products and sums in the same order, so the two
agree to the bit.  Against the oracle: 1e-10 times ten condition numbers of the block, as for the
other forms (backward error of an FP64 sweep, through the perturbation bound of the inverse).
"""
import numpy as np
import pytest
import torch

from oracle import relax as orc
from paper_2409_07392_amd import FiralError, RelaxContext, _lib
from synthdata import make_small

pytestmark = pytest.mark.gpu


def context(p, X=None):
    def dev(a):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    return RelaxContext(dev(p.X if X is None else X), dev(p.H), p.n_pool, 1, "f64")


@pytest.mark.parametrize("d", [129, 144, 145, 255, 256, 257, 272, 383, 576, 577])
def test_inverse_matches_oracle(d):
    p = make_small(n=2 * d + 100, n_lab=3, d=d, c=3, s=1, seed=d)
    om = np.random.default_rng(d).uniform(0.0, 1.0, p.N)
    ctx, omega = context(p), torch.as_tensor(om, device="cuda")
    _, Pinv, info = ctx.build_precond(omega, shift=1e-2, want_L=False)
    assert info["bad_block"] == -1
    assert torch.equal(Pinv, ctx.build_precond(omega, shift=1e-2)[1])
    P = orc.precond_blocks(p.X, p.H, om, 1e-2)
    Pinv = Pinv.cpu().numpy()
    for k in range(3):
        ref = np.linalg.inv(P[k])
        bar = 1e-10 * max(10.0, 10 * np.linalg.cond(P[k]))
        assert np.linalg.norm(Pinv[k] - ref) <= bar * np.linalg.norm(ref), k


@pytest.mark.parametrize("d", [129, 256, 257])
def test_inverse_reports_a_bad_last_pivot(d):
    # the last feature is zero in every row: with no shift every pivot but the last is positive
    p = make_small(n=2 * d + 100, n_lab=3, d=d, c=3, s=1, seed=d)
    X = p.X.copy()
    X[:, -1] = 0.0
    with pytest.raises(FiralError) as ei:
        context(p, X).build_precond(shift=0.0, want_L=False)
    assert ei.value.code == _lib.ENOTSPD
