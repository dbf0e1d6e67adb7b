"""Graphs whose elimination has many levels of few columns (a launch takes a run of
them): the smallest, ones with a wide first level, and runs longer than one
launch's limit of 64 levels, against the dense FP64 oracle."""

import numpy as np
import pytest
import torch

from oracle import pgo
from test_gpu_pgo import TOL, pose_err, run_gpu, small_graph

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")


@pytest.mark.parametrize("n, extra", [(2, 0), (3, 0), (9, 2), (40, 8), (70, 0), (200, 6)])
def test_level_runs_match_oracle(n, extra):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(100 + n)
    E, meas, _ = small_graph(rng, n, extra, 1e-3)
    T, rep = run_gpu(s3a.Handle(0), E, meas, n, iters=4)
    ref = pgo.pgo_solve(n, E, meas, iters=4)
    assert rep.status == 0 and ref["status"] == 0
    assert pose_err(T, ref["T"]) <= TOL
