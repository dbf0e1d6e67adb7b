"""Passes that solve the pass before themselves (untuned calls of few tiles)
against the plain path's finalize launches, which the alignment tests hold to
the oracle: the same partials, added and solved in the same order, so the same
bits. Sizes at the edges of tiles (4096 elements), of the gather's rounds (12
groups, 96 tiles), with pairs that fail among them; and the schedule of calls
with more pairs than its one-launch form takes."""

import numpy as np
import pytest
import torch

from synth.depthmaps import make_depth_batch
from synth.pointmaps import make_batch, make_targets, random_similarity

pytestmark = pytest.mark.gpu

s3a = pytest.importorskip("paper_2510_02080_amd")


@pytest.fixture(scope="module")
def h():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return s3a.Handle(0)


def batch(sizes, seed, fail=()):
    rng = np.random.default_rng(seed)
    pairs = []
    for k, n in enumerate(sizes):
        p = np.c_[rng.uniform(-2, 2, (n, 2)), rng.uniform(1, 6, n)]
        if k in fail:
            p[:] = p[:1] if n else p  # coincident points: degenerate
        s, R, t = random_similarity(rng)
        c = rng.uniform(1.0, 5.0, n)
        if n > 10:
            c[::7] = 0.5  # below the threshold
            p[3] = np.nan
        pairs.append((p, make_targets(rng, p, s, R, t), c, (s, R, t)))
    return make_batch(pairs, tau=1.0, name="edges")


def both(call):
    out = []
    for flags in (0, s3a.FLAG_PLAIN):
        S, ib = call(flags)
        torch.cuda.synchronize()
        out.append((S.cpu().numpy(), ib.cpu().numpy()))
    return out


CASES = {
    "one_tile": ([3072], ()),
    "tile_edges": ([1, 63, 64, 65, 4095, 4096, 4097, 8192, 0, 12289], (4,)),
    "gather_rounds": ([4096 * 11 + 5, 4096 * 12, 4096 * 13 - 1, 4096 * 95 + 1, 4096 * 96, 4096 * 97 + 1], ()),
    "failures": ([5000, 20000, 0, 30000], (0, 3)),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("iters,final", [(0, False), (1, False), (2, True), (6, False), (0, True)])
def test_solving_passes_equal_finalize_launches(h, name, dtype, iters, final):
    b = batch(CASES[name][0], seed=len(name), fail=CASES[name][1])
    b = b.to_bf16() if dtype == "bf16" else b
    pm = s3a.Pointmaps.from_batch(b, "cuda:0")
    f = s3a.FLAG_FINAL_COST if final else 0
    a, p = both(lambda flags: h.align_pairs(pm, b.tau, b.delta, iters, flags=flags | f))
    assert np.array_equal(a[0], p[0])
    assert a[1].tobytes() == p[1].tobytes()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("iters", [0, 1, 5])
def test_depth_solving_passes_equal_finalize_launches(h, dtype, iters):
    b = make_depth_batch([(48, 64, 1), (130, 131, 2), (200, 301, 1), (33, 47, 4)], seed=3)
    b.pairs[1]["width"] = 0  # invalid geometry
    b = b.to_bf16() if dtype == "bf16" else b
    dm = s3a.DepthPointmaps.from_batch(b, "cuda:0")
    a, p = both(lambda flags: h.align_depth_pairs(dm, b.tau, b.delta, iters, flags=flags))
    assert np.array_equal(a[0], p[0])
    assert a[1].tobytes() == p[1].tobytes()


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4500])
def test_schedule_of_many_pairs(h, n):
    """One call of n pairs against the same pairs in calls of at most 1000."""
    rng = np.random.default_rng(n)
    b = batch([int(x) for x in rng.integers(0, 200, n)], seed=n)
    pm = s3a.Pointmaps.from_batch(b, "cuda:0")
    S, ib = h.align_pairs(pm, b.tau, b.delta, 3)
    torch.cuda.synchronize()
    for k0 in range(0, n, 1000):
        k1 = min(n, k0 + 1000)
        part = s3a.Pointmaps(pm.planes, pm.offsets[k0:k1 + 1].contiguous(), pm.dtype)
        Sp, ip = h.align_pairs(part, b.tau, b.delta, 3)
        torch.cuda.synchronize()
        assert torch.equal(S[k0:k1], Sp)
        assert ib[k0:k1].cpu().numpy().tobytes() == ip.cpu().numpy().tobytes()
