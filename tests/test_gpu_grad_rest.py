"""Gradient planes outside the pairs' ranges: the calls that write them as zero
against the calls that leave them, on planes cleared beforehand."""

import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")
from paper_2510_02080_amd import binding  # noqa: E402

N = 20003


@pytest.mark.parametrize("offsets", [
    [0, N], [0, 5000, 5000, N], [1, N], [0, N - 1], [4099, 9000, 9001, 17002], [7000, 7000], [0, 0], [N, N],
    [0, 9000, 8000, N], [-1, N], [0, N + 1]])
@pytest.mark.parametrize("tuned", [False, True])
def test_rest_is_zero(offsets, tuned):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = s3a.Handle(0)
    if tuned:
        h.set_tuning(s3a.F32, 256, 2, 1)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    planes = [torch.rand(N, generator=g, device="cuda:0") + 0.5 for _ in range(7)]
    off = torch.tensor(offsets, dtype=torch.int64, device="cuda:0")
    n = len(offsets) - 1
    pm = s3a.Pointmaps(planes, off, s3a.F32)
    S = torch.zeros((n, 16), dtype=torch.float64, device="cuda:0")
    S[:, [0, 4, 8, 12]] = 1.0
    xi = torch.zeros((n, 7), dtype=torch.float64, device="cuda:0")
    L, C = h.align_cost(pm, S, xi, 0.6)
    gL = torch.ones(n, dtype=torch.float64, device="cuda:0")
    gS = torch.ones((n, 16), dtype=torch.float64, device="cuda:0")
    d = pm.desc(0.6, 0.05, 0)
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    Np = (N + 3) // 4 * 4
    out = {}
    for zeroed, fill in (("", 0.0), ("_zeroed", float("nan"))):
        a, b = (torch.full((7, Np), fill, device="cuda:0") for _ in range(2))
        gxi, v = (torch.zeros((n, 7), dtype=torch.float64, device="cuda:0") for _ in range(2))
        st = torch.zeros(n, dtype=torch.int32, device="cuda:0")
        binding._check(getattr(h.lib, "s3a_align_pairs_backward" + zeroed)(
            h.h, ctypes.byref(d), P(S), P(xi), P(L), P(C), P(gL), *[P(a[i]) for i in range(7)], P(gxi), stream), h.h)
        binding._check(getattr(h.lib, "s3a_align_pairs_implicit_backward" + zeroed)(
            h.h, ctypes.byref(d), P(S), P(gS), 0, *[P(b[i]) for i in range(7)], P(v), P(st), stream), h.h)
        torch.cuda.synchronize()
        out[zeroed] = a[:, :N], b[:, :N]
    for want, got in zip(out[""], out["_zeroed"]):
        assert torch.equal(got, want)
    lo, hi = offsets[0], offsets[-1]
    if all(0 <= x <= y <= N for x, y in zip(offsets, offsets[1:])) and hi - lo > 1000:
        assert (out["_zeroed"][0][6][lo:hi] != 0).any()
