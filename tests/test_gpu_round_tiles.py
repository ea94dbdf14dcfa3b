"""The LDS-resident scores where a wave walks several row tiles (rows and classes enough for the device's
workgroups to be fewer than the tiles) and the last tile is ragged: FP64 and FP32 decisions from either
storage, one and two row blocks a wave.  Tolerances and oracle are those of the Round step's other tests
(1e-9; FP32 decisions 1e-4).
"""
import pytest
import torch

from synthdata import make_small
from test_gpu_round import check_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,c,prec,fp32", [
    (5003, 50, 50, "f64", False), (5003, 50, 50, "f32", False),    # 16-row tiles, FP64
    (6007, 96, 40, "f64", False),                                  # the widest FP64 operand
    (8005, 120, 20, "f32", True), (6001, 144, 24, "f32", True),    # 16-row tiles, FP32
    (9011, 100, 16, "f64", True), (9011, 90, 20, "f64", True),     # FP64 storage, FP32 decisions
    (12013, 100, 20, "f32", True),                                 # 32-row tiles
])
def test_scores_over_several_tiles_a_wave(n, d, c, prec, fp32):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert -(-n // 32) // 8 > 2 * n_cu // c   # tiles of eight waves, workgroups of a class
    p = make_small(n=n, n_lab=20, d=d, c=c, s=1, seed=d)
    check_run(p, prec, 2, 8.0, lam=1e-2, fp32=fp32)
