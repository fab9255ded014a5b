"""Small problems (Section 3.1's iteration in two launches) take one of many kernels: so many vectors to a lane, so many ways to split the codebook, scores or distances in
direct form. Whatever the rule picks for any size, the shapes that the GPU tests compare with the direct form have it launched."""
import ctypes
import math
import random

import pytest

import paper_2503_13089_amd as cc
from tests import test_gpu_small_scores


class Cut(ctypes.Structure):
    _fields_ = [("blocks", ctypes.c_uint32), ("per_block", ctypes.c_uint32), ("slices", ctypes.c_int32), ("lane", ctypes.c_int32), ("direct", ctypes.c_int32)]


@pytest.fixture(scope="module")
def rules():
    lib = cc.load_library()
    cut, small = lib._ZN2cc9small_cutEjjjb, lib._ZN2cc13small_problemEmjj   # cc::small_cut and cc::small_problem, host functions
    cut.restype, cut.argtypes = Cut, [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_bool]
    small.restype, small.argtypes = ctypes.c_bool, [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32]
    return cut, small


def variant(rules, N, d, K, sums):
    c = rules[0](N, d, K, sums)
    assert c.blocks <= 512 and (c.blocks - 1) * c.per_block < N <= c.blocks * c.per_block
    return d, c.lane, c.slices, c.direct, sums


def test_the_shapes_of_the_gpu_tests_reach_every_kernel(rules):
    tested = {variant(rules, *shape, sums) for shape in test_gpu_small_scores.SHAPES + [(4097, 16, 129)] for sums in (True, False) if rules[1](*shape)}
    rng = random.Random(1)
    picked = {}
    for _ in range(20000):
        d, N, K = rng.choice((4, 8, 16)), int(math.exp(rng.uniform(0, math.log(3e7)))), int(math.exp(rng.uniform(0, math.log(1500))))
        if rules[1](N, d, K):
            for sums in (True, False):
                picked[variant(rules, N, d, K, sums)] = (N, d, K)
    assert len(picked) >= 50
    assert not {v: at for v, at in picked.items() if v not in tested}
