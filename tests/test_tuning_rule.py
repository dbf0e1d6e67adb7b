"""Which launch shape a call takes, given what autotuning found for which kinds of
calls (host build of the library's rule). Shapes are told apart by their wg."""

import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_02080_amd", "libs3a_hostmath.so")


class Table:
    def __init__(self):
        if not os.path.exists(LIB):
            from paper_2510_02080_amd import build
            build.build()
        self.lib = ctypes.CDLL(LIB)
        self.lib.s3a_host_tune_new.restype = ctypes.c_void_p
        self.t = ctypes.c_void_p(self.lib.s3a_host_tune_new())

    def record(self, wg, points, pairs, dtype=0, persistent=False):
        self.lib.s3a_host_tune_record(self.t, dtype, ctypes.c_longlong(points), ctypes.c_longlong(pairs), int(persistent), wg)

    def find(self, points, pairs, dtype=0, persistent=False, solving=False):
        return self.lib.s3a_host_tune_find(self.t, dtype, ctypes.c_longlong(points), ctypes.c_longlong(pairs),
                                           int(persistent), int(solving))

    def last(self, points, dtype=0):
        return self.lib.s3a_host_tune_last(self.t, dtype, ctypes.c_longlong(points))

    def __del__(self):
        self.lib.s3a_host_tune_free(self.t)


@pytest.fixture
def t():
    return Table()


def test_nothing_tuned(t):
    assert t.find(1000, 1) == t.find(1000, 1, solving=True) == t.last(1000) == 0


def test_a_batch_says_nothing_about_small_calls_of_its_class(t):
    t.record(512, 3_000_000, 256)
    assert t.find(3_000_000, 256) == 512
    assert t.find(2_000_000, 200) == 512                 # the same kind
    assert t.find(2_000_000, 1, solving=True) == 0       # passes that solve
    assert t.find(2_000_000, 1) == 512                   # passes that do not: as before
    assert t.find(2_000_000, 1, dtype=1) == 0
    assert t.find(20_000_000, 256) == 0


def test_persistent_and_per_pass_are_kinds_of_their_own(t):
    t.record(256, 3_000_000, 64, persistent=True)
    assert t.find(3_000_000, 64, persistent=True) == 256
    assert t.find(3_000_000, 64, solving=True) == 0
    assert t.find(3_000_000, 64) == 256                  # nothing else known
    t.record(512, 3_000_000, 64)
    assert t.find(3_000_000, 64, persistent=True) == 256
    assert t.find(3_000_000, 64) == t.find(3_000_000, 64, solving=True) == 512
    assert t.last(3_000_000) == 512


def test_untuned_found_fastest(t):
    t.record(512, 3_000_000, 64)
    t.record(0, 3_000_000, 4)
    assert t.find(3_000_000, 4) == t.find(3_000_000, 3, solving=True) == 0
    assert t.find(3_000_000, 64) == 512
    assert t.last(3_000_000) == 0                        # found last
    t.record(256, 3_000_000, 4)                          # tuned again: replaced
    assert t.find(3_000_000, 4) == t.last(3_000_000) == 256


@pytest.mark.parametrize("a,b,same", [(0, 1, True), (1, 2, False), (2, 4, True), (4, 5, False), (16, 17, False),
                                      (65, 256, True), (256, 257, False), (2 ** 24, 2 ** 24 - 1, True)])
def test_pair_classes(t, a, b, same):
    t.record(512, 1000, a)
    assert (t.find(1000, b, solving=True) == 512) == same
