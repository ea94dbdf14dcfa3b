"""The Round step's FP64 state to the bit: nu of every round and the objective of every pool row
equal to recorded values (golden/round_bits.json: nu as hexadecimal floats, SHA-256 of the objective's
bytes).  They were recorded with the plain form of every kernel of the chain: the triangular inverse a
column a thread, the tridiagonalisation with the sums of a step in one wave, Sturm counts by pivots
alone, the block inverse by plain sums, the scores a tile at a time, nu's sums by 64 threads (up to
2048 eigenvalues) or by 1024.  nu moves the FP32 copy of the operand, so that a sum taken in another
order, harmless by itself, shows in the FP32 objective at single rows.

Shapes: every group size of the eigenvalue search (64, 32, 16 lanes and 1), both forms of nu's sums,
blocks in registers (d <= 128) and in memory, one and several blocks of 16, few labeled rows (most
eigenvalues equal within rounding) and many, d = 1 and 2.
"""
import hashlib
import json
import os

import numpy as np
import pytest
import torch

from paper_2409_07392_amd import RelaxContext, RoundSolver
from synthdata import dirichlet_weights, make_small

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "round_bits.json")
CASES = [  # n_pool, n_lab, d, c, rounds
    (300, 5, 7, 3, 8), (200, 3, 1, 3, 4), (150, 2, 2, 2, 4), (500, 30, 20, 5, 8), (700, 10, 33, 6, 8),
    (900, 3, 64, 4, 6), (1500, 10, 100, 10, 10), (1500, 300, 100, 10, 10), (800, 40, 128, 7, 6),
    (900, 50, 50, 50, 6), (1200, 9, 97, 24, 6),      # 2048 < c d <= 4096
    (600, 12, 60, 80, 4), (700, 5, 130, 6, 4),       # 32 lanes; the block in memory
    (500, 8, 128, 260, 2), (400, 8, 127, 520, 2),    # 16 lanes, one lane an eigenvalue
]


def run_case(case, prec, fp32):
    n, nl, d, c, b = case
    p = make_small(n=n, n_lab=nl, d=d, c=c, s=1, seed=n + d + c)
    dt = torch.float64 if prec == "f64" else torch.float32
    X, H = (torch.tensor(a, dtype=dt, device="cuda") for a in (p.X, p.H))
    z = torch.tensor(dirichlet_weights(np.random.default_rng(d), n, float(b)), dtype=torch.float64,
                     device="cuda")
    ctx = RelaxContext(X, H, n, 1, prec)
    rs = RoundSolver(ctx, z, 1e-3, 8.0 * np.sqrt(d * c), b, fp32=fp32)
    rs.step(b)
    res = rs.result()
    scores = rs.scores().cpu().numpy()
    rs.close()
    ctx.close()
    return dict(nu=[float(v).hex() for v in res["nu"]], selected=[int(i) for i in res["selected"]],
                scores=hashlib.sha256(scores.tobytes()).hexdigest())


def key(case, prec, fp32):
    return "-".join(map(str, case)) + f"-{prec}-{'fp32' if fp32 else 'fp64'}"


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("case", CASES)
def test_round_state_to_the_bit(case, prec, fp32):
    with open(GOLDEN) as f:
        want = json.load(f)[key(case, prec, fp32)]
    assert run_case(case, prec, fp32) == want
