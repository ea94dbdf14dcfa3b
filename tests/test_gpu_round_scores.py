"""The scores from LDS-resident operands at the edges of their ranges: the last block of features
partial and full, an odd and an even number of blocks, one and two row blocks a wave, the first
sizes past the limits (97 in FP64, 145 in FP32: the tiled kernel), a pool of less than one row tile.
Tolerances and oracle are those of the Round step's other tests (1e-9; FP32 decisions 1e-4).
"""
import pytest

from synthdata import make_small
from test_gpu_round import check_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(260, 4, 17, 3), (331, 0, 80, 4), (270, 9, 96, 2), (270, 3, 97, 3),
                                   (401, 5, 112, 3), (401, 2, 113, 3), (345, 5, 144, 2),
                                   (345, 5, 145, 2), (11, 30, 9, 4)])
def test_scores_match_oracle(shape, prec, fp32):
    n, nl, d, c = shape
    p = make_small(n=n, n_lab=nl, d=d, c=c, s=1, seed=100 + d)
    check_run(p, prec, 2, 8.0, lam=1e-2, fp32=fp32)
