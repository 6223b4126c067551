"""Training steps of one LOD around the size where they leave the rank sort
(2,048 points), against the FP64 oracle with the bars of every gradient test."""
import numpy as np
import pytest

import oracle
from paper_2101_10994_amd import workloads as W

from cases import make_case
from test_gpu_train import compare, gpu_train, points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [2047, 2048, 2049, 4096])
def test_sizes(P):
    case = make_case(W.tiny_shape(), 4, 1, 8, 32, sigma=0.1)
    x, tgt = points(case, np.random.default_rng(P), P, 4)
    compare(gpu_train(case, x, tgt), oracle.train_fwd_bwd(case.otree, case.oracle_model(), x, tgt))
