"""Calls of as many pairs as the entry points take (2^24), most of them empty: a
workgroup per tile or per pair would be more than one launch holds."""

import numpy as np
import pytest
import torch

from synth import depthmaps

from gpu_util import ragged_batch

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")

AT = (0, 1, 2 ** 22, 2 ** 23 - 2)  # where the pairs that hold points lie


def handle():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return s3a.Handle(0)


def spread(offsets, n, last):
    """Offsets of n pairs: the given ones' at AT and at the last place, empty ones between."""
    size = np.zeros(n, np.int64)
    size[list(AT) + [last]] = np.diff(offsets)
    return torch.from_numpy(np.r_[0, np.cumsum(size)]).to("cuda:0")


def test_align():
    n = 2 ** 24
    b = ragged_batch([3000, 50, 9000, 4097, 700], seed=81)
    few = s3a.Pointmaps.from_batch(b, "cuda:0")
    many = s3a.Pointmaps(few.planes, spread(b.offsets, n, n - 1), few.dtype)
    h = handle()
    want, wi = h.align_pairs(few, b.tau, b.delta, 1, flags=s3a.FLAG_PLAIN)
    got, gi = h.align_pairs(many, b.tau, b.delta, 1)
    torch.cuda.synchronize()
    at = list(AT) + [n - 1]
    assert torch.equal(got[at], want) and torch.equal(gi[at], wi)
    empty = torch.ones(n, dtype=torch.bool, device="cuda:0")
    empty[at] = False
    assert (got[empty][:, [0, 4, 8, 12]] == 1).all()
    status = gi.view(torch.int32)[:, s3a.INFO_DTYPE.fields["status"][1] // 4]
    assert (status[empty] == s3a.PAIR_EMPTY).all() and (status[at] == 0).all()


def test_depth():
    n = 2 ** 23
    b = depthmaps.make_depth_batch([(30, 40, 1), (7, 9, 1), (150, 160, 1), (64, 64, 1), (20, 30, 1)], seed=82)
    few = s3a.DepthPointmaps.from_batch(b, "cuda:0")
    at = list(AT) + [n - 1]
    rec = few.pairs.view(5, -1)
    pairs = rec[:1].repeat(n, 1)
    pairs[at] = rec
    many = s3a.DepthPointmaps(few.planes, spread(b.offsets, n, n - 1), pairs.view(-1), few.dtype)
    h = handle()
    want, wi = h.align_depth_pairs(few, b.tau, b.delta, 1, flags=s3a.FLAG_PLAIN)
    got, gi = h.align_depth_pairs(many, b.tau, b.delta, 1)
    torch.cuda.synchronize()
    assert torch.equal(got[at], want) and torch.equal(gi[at], wi)


def test_cost_and_gradients():
    n = 2 ** 23
    b = ragged_batch([3000, 50, 9000, 4097, 700], seed=83)
    few = s3a.Pointmaps.from_batch(b, "cuda:0")
    many = s3a.Pointmaps(few.planes, spread(b.offsets, n, n - 1), few.dtype)
    at = list(AT) + [n - 1]
    h = handle()
    S0, _ = h.align_pairs(few, b.tau, b.delta, 3)
    S = S0[:1].repeat(n, 1)
    S[at] = S0
    xi = torch.zeros((n, 7), dtype=torch.float64, device="cuda:0")
    gL = torch.ones(n, dtype=torch.float64, device="cuda:0")
    L0, C0 = h.align_cost(few, S0, xi[:5], b.tau)
    L, C = h.align_cost(many, S, xi, b.tau)
    torch.cuda.synchronize()
    assert torch.equal(L[at], L0) and torch.equal(C[at], C0)
    want = h.align_pairs_backward(few, S0, xi[:5], L0, C0, gL[:5], b.tau)
    got = h.align_pairs_backward(many, S, xi, L, C, gL, b.tau)
    torch.cuda.synchronize()
    for i in range(3):
        assert torch.equal(got[i], want[i])
    assert torch.equal(got[3][at], want[3])
    gS = torch.ones((n, 16), dtype=torch.float64, device="cuda:0")
    want = h.align_pairs_implicit_backward(few, S0, gS[:5], b.tau)
    got = h.align_pairs_implicit_backward(many, S, gS, b.tau)
    torch.cuda.synchronize()
    assert (got[4][at] == 0).all() and (want[4] == 0).all()
    scale = max(float(t.abs().max()) for t in want[:3])
    for i in range(3):  # the Hessian's partial sums split differently
        assert (got[i] - want[i]).abs().max() <= 1e-6 * scale
