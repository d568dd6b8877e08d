"""Which parameter tensors share a launch of the update: the rule is host code
without HIP, compiled here by itself and run on made-up addresses."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1711_10275_amd", "csrc")

WRAP = """
#include "sgd_batch.h"
struct Tensor { float* params; const float* grads; float* momentum_buf; void* params_bf16; int64_t count; };
extern "C" int batch(const Tensor* t, int n) { return sscn::sgd_batch(t, n); }
"""


class Tensor(ctypes.Structure):
    _fields_ = [("params", ctypes.c_void_p), ("grads", ctypes.c_void_p), ("momentum_buf", ctypes.c_void_p),
                ("params_bf16", ctypes.c_void_p), ("count", ctypes.c_int64)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    d = tmp_path_factory.mktemp("sgd")
    (d / "wrap.cpp").write_text(WRAP)
    so = str(d / "wrap.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)

    def run(tensors):
        """[tensors of each launch] as the library forms them."""
        arr, out, k = (Tensor * len(tensors))(*tensors), [], 0
        while k < len(tensors):
            m = lib.batch(ctypes.byref(arr, k * ctypes.sizeof(Tensor)), len(tensors) - k)
            assert 1 <= m <= len(tensors) - k
            out.append(list(range(k, k + m)))
            k += m
        return out

    return run


def _ranges(t):
    p, g, b, c, n = t
    return [(p, p + 4 * n, True), (g, g + 4 * n, False), (b, b + 4 * n, True)] + ([(c, c + 2 * n, True)] if c else [])


def _meet(a, b):
    return any((w or x) and lo < y and z < hi for lo, hi, w in _ranges(a) for z, y, x in _ranges(b))


def test_apart(launches):
    ts = [(1 << 20, 2 << 20, 3 << 20, 4 << 20, 1000), ((1 << 20) + 4000, (2 << 20) + 4000, (3 << 20) + 4000, None, 1000)]
    assert launches(ts) == [[0, 1]]
    assert launches([(1 << 20, 2 << 20, 3 << 20, None, 0)] * 3) == [[0, 1, 2]]  # empty tensors meet nothing
    many = [((i + 1) << 20, (i + 1001) << 20, (i + 2001) << 20, None, 7) for i in range(130)]
    assert [len(x) for x in launches(many)] == [64, 64, 2]


@pytest.mark.parametrize("second", [
    (0x100000 + 4 * 50, 0x900000, 0xa00000, None),  # the middle of the first one's parameters
    (0x800000, 0x100000 + 4 * 99, 0xa00000, None),  # a gradient that ends inside them
    (0x800000, 0x900000, 0x300000 - 4, None),       # momentum one element into momentum
    (0x800000, 0x900000, 0xa00000, 0x200000 + 2),   # a bf16 copy over the first one's gradient
    (0x200000 + 4 * 99, 0x900000, 0xa00000, None),  # parameters at the gradient's last element
])
def test_a_tensor_that_meets_an_earlier_one_starts_a_launch(launches, second):
    first = (0x100000, 0x200000, 0x300000, 0x400000, 100)
    assert launches([first, (*second, 100)]) == [[0], [1]]
    assert launches([(*second, 100), first]) == [[0], [1]]


def test_shared_gradients_do_not_meet(launches):
    assert launches([(0x100000, 0x200000, 0x300000, None, 100), (0x800000, 0x200000, 0x900000, None, 100)]) == [[0, 1]]


def test_against_pairs(launches):
    rng = random.Random(3)
    for _ in range(400):
        span = rng.choice([2000, 40000])
        addr = lambda: 4096 + 4 * rng.randrange(span)  # noqa: E731
        ts = [(addr(), addr(), addr(), addr() if rng.random() < 0.5 else None, rng.choice([0, 1, 5, 60]))
              for _ in range(rng.randrange(1, 90))]
        got = launches(ts)
        assert [i for x in got for i in x] == list(range(len(ts)))
        for x in got:
            live = [i for i in x if ts[i][4]]
            assert len(live) <= 64
            assert not any(_meet(ts[i], ts[j]) for i in live for j in live if i < j)
        for x, y in zip(got, got[1:]):  # no launch ends early
            full = sum(1 for i in x if ts[i][4]) == 64
            assert full or any(_meet(ts[i], ts[y[0]]) for i in x if ts[i][4])


def test_a_launch_stays_within_its_grid(launches):
    """A launch's workgroups of 256 threads stay far below the 2^32 threads that a
    grid may have, and 32-bit numbers hold them; a tensor of more is alone."""
    def groups(i, ts):
        return -(-ts[i][4] // 1024)

    big = [((3 * i + 1) << 36, (3 * i + 2) << 36, (3 * i + 3) << 36, None, 1 << 30) for i in range(17)]
    mixed = [(*t[:4], n) for t, n in zip(big, [5, (1 << 30) + 1, 7, 1 << 29, 1 << 29, 1, (1 << 33), 1 << 20, 3])]
    for ts in (big, mixed):
        got = launches(ts)
        assert [i for x in got for i in x] == list(range(len(ts)))
        for x in got:
            assert len(x) == 1 or sum(groups(i, ts) for i in x) <= 1 << 20
    assert len(launches(big)) == 17
    assert launches(mixed) == [[0], [1], [2, 3], [4, 5], [6], [7, 8]]
