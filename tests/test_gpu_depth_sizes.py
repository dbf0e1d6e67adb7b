"""Depth frames at the edges of the walks' sizes, against the FP64 oracle: rows about as
long as a vector of pixels or shorter, rows of many millions, and pairs past the sizes
that 32-bit positions hold."""

import numpy as np
import pytest
import torch

from oracle import irls
from synth import depthmaps

from gpu_util import check_pair, ragged_batch
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [2 ** 25 + 8, 2 ** 26, 2 ** 31 - 1])
def test_wide_rows(width, dtype):
    """A pair that holds the first elements of one row of many millions; the pair
    before it ends inside a vector, so that its first vector has elements outside."""
    b = depthmaps.make_depth_batch([(7, 11, 1), (1, 6000, 1)], seed=61)
    for side in ("p", "q"):  # (a row's far end in view of the first two widths)
        b.pairs[1][side]["fx"] = min(max(6000, width / 1500), 50000)
    if dtype == "bf16":
        b = b.to_bf16()
    b.pairs[1]["width"] = b.pairs[1]["frame_pixels"] = width
    h = handle()
    for flags in (0, s3a.FLAG_PLAIN):
        T, info = run(h, b, flags)
        for k in range(2):
            check_pair(T[k], info[k], oracle_pair(b, k), where=f"pair {k} flags {flags}", dr=DR_DEPTH)


def test_pair_past_32_bit_positions():
    """Three whole frames of 720 M pixels below the threshold, then the first rows of a
    fourth: the elements that count lie past 2^31, around the frames' border."""
    W, HW = 30000, 30000 * 24000
    n = 3 * HW + 90000
    small = depthmaps.make_depth_batch([(6, W, 2)], seed=62).to_bf16()  # the last 3 rows of frame 2, the first 3 of frame 3
    rec = small.pairs[0].copy()
    rec["frame_pixels"], rec["n_frames"] = HW, 4
    for side in ("p", "q"):
        rec[side][2], rec[side][3] = small.pairs[0][side][0], small.pairs[0][side][1]
        rec[side][:2] = rec[side][2]
        rec[side]["fy"], rec[side]["cy"] = W, 12000.0
        rec[side]["fx"], rec[side]["cx"] = W, 15000.0
    rows = np.concatenate([np.arange(24000 - 3, 24000), np.arange(3)])
    f = np.repeat([2, 3], 3 * W)
    col, row = np.tile(np.arange(W), 6), np.repeat(rows, W)
    # depths of the pixels that count, seen by both sides
    rng = np.random.default_rng(63)
    dp = rng.uniform(1.0, 10.0, 6 * W).astype(np.float32)
    s = small.gt[0][0]
    dq = (s * dp * (1 + 0.005 * rng.normal(size=len(dp)))).astype(np.float32)
    c = np.exp(rng.normal(1.0, 0.5, len(dp))).astype(np.float32)
    t = [torch.from_numpy(x).to(torch.bfloat16) for x in (dp, dq, c)]
    dec = [x.double().numpy() for x in t]
    pts = []
    for d, side in ((dec[0], "p"), (dec[1], "q")):
        x = np.zeros((6 * W, 3))
        for fr in (2, 3):
            cam, sel = rec[side][fr], f == fr
            ray = np.stack([(col[sel] - float(cam["cx"])) / float(cam["fx"]), (row[sel] - float(cam["cy"])) / float(cam["fy"]),
                            np.ones(sel.sum())], 1)
            x[sel] = (d[sel, None] * ray) @ cam["R"].reshape(3, 3).astype(np.float64).T + cam["t"].astype(np.float64)
        pts.append(x)
    ref = irls.irls_align(pts[0], pts[1], dec[2], 1.5, 0.05, 5)
    h = handle()
    planes = [torch.ones(n, dtype=torch.bfloat16, device="cuda:0") for _ in range(3)]
    for p, x in zip(planes, t):
        p[3 * HW - 3 * W:] = x.to("cuda:0")
    off = torch.tensor([0, n], dtype=torch.int64, device="cuda:0")
    pairs = torch.from_numpy(np.array([rec]).view(np.uint8).copy()).to("cuda:0")
    dm = s3a.DepthPointmaps([p.view(torch.int16) for p in planes], off, pairs, s3a.BF16)
    S, ib = h.align_depth_pairs(dm, 1.5, 0.05, 5)
    torch.cuda.synchronize()
    T, info = s3a.sim3_to_numpy(S), s3a.info_to_numpy(ib)
    assert ref["status"] == 0
    check_pair(T[0], info[0], ref, where="past 2^31", dr=DR_DEPTH)


def test_stored_pair_past_32_bit_positions():
    """The same for stored points: alignment, cost and the implicit derivative of a pair
    whose points that count are its last."""
    b = ragged_batch([50000], seed=65).to_bf16()
    few = s3a.Pointmaps.from_batch(b, "cuda:0")
    n = 2 ** 31 + 50000
    planes = [torch.zeros(n, dtype=torch.int16, device="cuda:0") for _ in range(7)]
    for p, x in zip(planes, few.planes):
        p[-50000:] = x.view(torch.int16)
    many = s3a.Pointmaps(planes, torch.tensor([0, n], dtype=torch.int64, device="cuda:0"), s3a.BF16)
    ref = irls.irls_align(*b.decoded_pair(0), b.tau, b.delta, b.iters)
    h = handle()
    S, ib = h.align_pairs(many, b.tau, b.delta, b.iters)
    torch.cuda.synchronize()
    check_pair(s3a.sim3_to_numpy(S)[0], s3a.info_to_numpy(ib)[0], ref, where="stored past 2^31")
    S0, _ = h.align_pairs(few, b.tau, b.delta, b.iters)
    xi = torch.zeros((1, 7), dtype=torch.float64, device="cuda:0")
    L0, C0 = h.align_cost(few, S0, xi, b.tau)
    L, C = h.align_cost(many, S0, xi, b.tau)
    gS = torch.ones((1, 16), dtype=torch.float64, device="cuda:0")
    want = h.align_pairs_implicit_backward(few, S0, gS, b.tau, need=(False, False, True))
    got = h.align_pairs_implicit_backward(many, S0, gS, b.tau, need=(False, False, True))
    torch.cuda.synchronize()
    # FP64 sums in another order, and gradients rounded to FP32 from them
    assert abs(C.item() - C0.item()) <= 1e-12 * C0.item() and abs(L.item() - L0.item()) <= 1e-12 * L0.item()
    assert (got[2][-50000:] - want[2]).abs().max() <= 1e-6 * want[2].abs().max()
    assert not got[2][:-50000].any()
