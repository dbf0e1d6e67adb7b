"""Points of weight zero whose coordinates are finite but huge (a sentinel where a
depth is missing, marked by its confidence): they contribute nothing, whatever
their value, to the pose, the costs or the counts. Stored points and depth maps,
on every launch path, against the FP64 oracle."""

import numpy as np
import pytest
import torch

from oracle import depth, irls
from synth import depthmaps
from synth.pointmaps import bf16_encode

from gpu_util import check_pair, ragged_batch
from test_gpu_depth import DR_DEPTH

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")

VALUES = np.array([1e12, -3e15, 1e20, -1e20, 3e38, -3.3e38, 1e30, 5.0], np.float32)


def check(T, info, refs, dr=None):
    for k, ref in enumerate(refs):
        check_pair(T[k], info[k], ref, where=f"pair {k}", **({} if dr is None else dict(dr=dr)))
        if ref["status"] == 0:
            L = ref["final_cost"]
            assert abs(info[k]["final_cost"] - L) <= 1e-5 * abs(L) + np.sqrt(2 * abs(L)) * (dr or DR_DEPTH), k


def results(S, ib):
    torch.cuda.synchronize()
    return s3a.sim3_to_numpy(S), s3a.info_to_numpy(ib)


def new_handle(looping=False):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = s3a.Handle(0)
    if looping:
        for dt in (s3a.F32, s3a.BF16):
            h.set_tuning(dt, 256, 4, 1)
    return h


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tau,c", [(1.5, 0.25), (0.0, 0.0)])
def test_stored_sentinels(dtype, tau, c):
    b = ragged_batch([5000, 20000, 70000, 300], seed=91, tau=tau, specials={3: "nan_some"})
    if dtype == "bf16":
        b = b.to_bf16()
    enc = (lambda x: bf16_encode(np.asarray(x, np.float32))) if dtype == "bf16" else (lambda x: np.asarray(x, np.float32))
    rng = np.random.default_rng(92)
    for k in (0, 2, 3):  # pair 1 holds none
        a, e = int(b.offsets[k]), int(b.offsets[k + 1])
        idx = a + rng.choice(e - a, 64, replace=False)
        for j, name in enumerate(("px", "py", "pz", "qx", "qy", "qz")):
            b.planes[name][idx] = enc(np.roll(VALUES, j)[rng.integers(0, len(VALUES), len(idx))])
        b.planes["c"][idx] = enc(np.full(len(idx), c))
    refs = [irls.irls_align(*b.decoded_pair(k), b.tau, b.delta, b.iters) for k in range(b.n_pairs)]
    pm = s3a.Pointmaps.from_batch(b, "cuda:0")
    F = s3a.FLAG_FINAL_COST
    for h, flags in ((new_handle(), F), (new_handle(), F | s3a.FLAG_PLAIN), (new_handle(), F | s3a.FLAG_PERSISTENT),
                     (new_handle(looping=True), F)):
        check(*results(*h.align_pairs(pm, b.tau, b.delta, b.iters, flags=flags)), refs)
    check(*results(*s3a.align_pairs_noalloc(pm, b.tau, b.delta, b.iters, flags=F)), refs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_depth_sentinels(dtype):
    """In frames that hold whole tiles, in tiles that span frames, and in frames narrower than a vector."""
    b = depthmaps.make_depth_batch([(200, 210, 2), (40, 50, 1), (300, 5, 2)], seed=93)
    if dtype == "bf16":
        b = b.to_bf16()
    enc = bf16_encode if dtype == "bf16" else (lambda x: x)
    rng = np.random.default_rng(94)
    for k in (0, 2):
        a, e = int(b.offsets[k]), int(b.offsets[k + 1])
        idx = a + rng.choice(e - a, 64, replace=False)
        b.dp[idx] = enc(np.array([1e20, 1e30, 1e36, 2.0], np.float32))[rng.integers(0, 4, len(idx))]
        b.dq[idx] = enc(np.array([1e13, 1e36, -1e20, 3.0], np.float32))[rng.integers(0, 4, len(idx))]
        b.c[idx] = enc(np.full(1, 0.25, np.float32))[0]
    refs = []
    for k in range(b.n_pairs):
        dp, dq, c = b.decoded(k)
        refs.append(irls.irls_align(*depth.unproject_pair(dp, dq, b.pairs[k]), c, b.tau, b.delta, b.iters))
    dm = s3a.DepthPointmaps.from_batch(b, "cuda:0")
    F = s3a.FLAG_FINAL_COST
    for h, flags in ((new_handle(), F), (new_handle(), F | s3a.FLAG_PLAIN), (new_handle(looping=True), F)):
        check(*results(*h.align_depth_pairs(dm, b.tau, b.delta, b.iters, flags=flags)), refs, dr=DR_DEPTH)
