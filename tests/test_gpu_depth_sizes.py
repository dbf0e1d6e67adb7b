"""Depth frames at the edges of the walks' sizes: rows about as long as a vector of
pixels or shorter, against the FP64 oracle."""

import pytest
import torch

from synth import depthmaps

from gpu_util import check_pair
from test_gpu_depth import DR_DEPTH, oracle_pair, run

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")


def handle():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return s3a.Handle(0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 7, 8, 9])
def test_narrow_frames(width, dtype):
    """One frame of many tiles, and two that share a tile."""
    b = depthmaps.make_depth_batch([(90001 // width, width, 1), (1200, width, 2), (35, width, 4)], seed=64)
    for k, rows in enumerate((90001 // width, 1200, 35)):
        for side in ("p", "q"):  # rows spread over the view as columns are
            b.pairs[k][side]["fy"], b.pairs[k][side]["cy"] = rows, rows / 2
    if dtype == "bf16":
        b = b.to_bf16()
    h = handle()
    for flags in (0, s3a.FLAG_PLAIN):
        T, info = run(h, b, flags)
        for k in range(3):
            check_pair(T[k], info[k], oracle_pair(b, k), where=f"pair {k} flags {flags}", dr=DR_DEPTH)
