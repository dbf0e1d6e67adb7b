"""Gradient calls without pairs: the ones that write zeros outside every pair's
range write all entries, the others none."""

import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")
from paper_2510_02080_amd import binding  # noqa: E402


@pytest.mark.parametrize("n", [1, 63, 20003])
def test_no_pairs(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = s3a.Handle(0)
    planes = [torch.ones(n, device="cuda:0") for _ in range(7)]
    pm = s3a.Pointmaps(planes, torch.zeros(1, dtype=torch.int64, device="cuda:0"), s3a.F32)
    d = pm.desc(0.5, 0.05, 0)
    none = ctypes.c_void_p(None)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    Np = (n + 3) // 4 * 4
    for zeroed in ("_zeroed", ""):
        for wanted in (range(7), (0, 6)):
            for name, head in (("s3a_align_pairs_backward", [none] * 5), ("s3a_align_pairs_implicit_backward", [none] * 2 + [0])):
                g = torch.full((7, Np), 3.0, device="cuda:0")
                out = [ctypes.c_void_p(g[i].data_ptr()) if i in wanted else none for i in range(7)]
                tail = [none] if name.endswith("pairs_backward") else [none] * 2
                binding._check(getattr(h.lib, name + zeroed)(h.h, ctypes.byref(d), *head, *out, *tail, stream), h.h)
                torch.cuda.synchronize()
                for i in range(7):
                    want = 0.0 if zeroed and i in wanted else 3.0
                    assert (g[i, :n] == want).all() and (g[i, n:] == 3.0).all(), (name, zeroed, i)
    S = torch.zeros((0, 16), dtype=torch.float64, device="cuda:0")
    e = torch.zeros(0, dtype=torch.float64, device="cuda:0")
    gp, gq, gc, _ = h.align_pairs_backward(pm, S, e, e, e, e, 0.5)
    ip, iq, ic, _, _ = h.align_pairs_implicit_backward(pm, S, S, 0.5)
    for t in (gp, gq, gc, ip, iq, ic):
        assert (t == 0).all()
