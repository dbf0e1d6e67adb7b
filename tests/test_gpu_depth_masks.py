"""Depth pairs that hold pixels whose points are not finite though their depths
are (a lost frame's camera, a ray that overflows): such pixels are invalid
wherever they lie, in tiles of one frame as in tiles that span two, on every
launch path. Against the FP64 oracle."""

import numpy as np
import pytest
import torch

from synth import depthmaps

from gpu_util import check_pair
from test_gpu_depth import DR_DEPTH, oracle_pair, run

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")

HW = (200, 210)  # 42,000 pixels: tiles of at most 32,768 lie in either frame and across both


def handles():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    looping = s3a.Handle(0)  # a forced shape: finalize launches, a loop over the tiles
    for dt in (s3a.F32, s3a.BF16):
        looping.set_tuning(dt, 256, 4, 1)
    return [(s3a.Handle(0), 0), (s3a.Handle(0), s3a.FLAG_PLAIN), (looping, 0)]


def batch(dtype):
    b = depthmaps.make_depth_batch([(*HW, 2), (*HW, 2), (40, 50, 1)], seed=53)
    return b.to_bf16() if dtype == "bf16" else b


def lose(cam, kind):
    if kind == "rotation_nan":
        cam["R"][4] = np.nan
    elif kind == "rotation_inf":
        cam["R"][0] = np.inf
    elif kind == "focal_zero":
        cam["fx"] = 0.0
    else:
        cam["cy"] = np.nan


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["rotation_nan", "rotation_inf", "focal_zero", "centre_nan"])
def test_lost_frame(kind, dtype):
    """One frame of each two-frame pair is lost on one side: the other frame's pixels solve."""
    b = batch(dtype)
    lose(b.pairs[0]["p"][0], kind)
    lose(b.pairs[1]["q"][1], kind)
    with np.errstate(all="ignore"):
        refs = [oracle_pair(b, k) for k in range(3)]
    assert all(r["status"] == 0 for r in refs) and refs[0]["n_nonfinite"] == HW[0] * HW[1]
    for h, flags in handles():
        T, info = run(h, b, flags)
        for k in range(3):
            check_pair(T[k], info[k], refs[k], where=f"{kind} {dtype} pair {k} flags {flags}", dr=DR_DEPTH)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("side", ["p", "q"])
def test_lost_translation(side, dtype):
    """A camera whose rotation and intrinsics are good but whose centre is not finite."""
    b = batch(dtype)
    b.pairs[0][side][0]["t"][1] = np.nan
    b.pairs[1][side][1]["t"][2] = np.inf
    refs = [oracle_pair(b, k) for k in range(3)]
    assert all(r["status"] == 0 for r in refs) and refs[1]["n_nonfinite"] == HW[0] * HW[1]
    for h, flags in handles():
        T, info = run(h, b, flags)
        for k in range(3):
            check_pair(T[k], info[k], refs[k], where=f"{side} {dtype} pair {k} flags {flags}", dr=DR_DEPTH)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ray_that_overflows(dtype):
    """A pixel of ordinary depth for its type, 1e28, whose ray takes it past the
    FP32 range, below the confidence threshold as the rest of its frame."""
    b = batch(dtype)
    n = HW[0] * HW[1]
    b.pairs[0]["p"][1]["fx"] = 1e-12
    c, d = (0x3f00, 0x6e01) if dtype == "bf16" else (0.5, 1e28)  # 0.5 and 1.0e28
    b.c[n:2 * n] = c
    b.dp[70000] = d
    refs = [oracle_pair(b, k) for k in range(3)]
    assert refs[0]["status"] == 0
    refs[0]["n_nonfinite"] += 1  # finite in FP64, not in the FP32 that the points are given in
    for h, flags in handles():
        T, info = run(h, b, flags)
        for k in range(3):
            check_pair(T[k], info[k], refs[k], where=f"{dtype} pair {k} flags {flags}", dr=DR_DEPTH)
