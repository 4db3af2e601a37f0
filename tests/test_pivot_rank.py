"""Pivot selection's candidates, counted on the CPU: every token that may belong to the best P is
one, and they stay few whatever the norms look like -- each is read whole by one compute unit."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
TAU = 1e-6  # of the order of the norm pass's own bound


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rank") / "libpivot_rank.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC",
                    os.path.join(HERE, "pivot_rank_host.cpp"), "-o", lib], check=True)
    f = C.CDLL(lib).candidates
    f.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_float, C.c_void_p, C.c_void_p]

    def run(v, P):
        v = np.ascontiguousarray(v, np.float32)
        cand, looks = np.zeros(len(v), np.uint8), C.c_int()
        count = f(v.ctypes.data, len(v), P, TAU, cand.ctypes.data, C.byref(looks))
        assert count == cand.sum() and looks.value <= 34
        return cand.astype(bool)
    return run


def norms(kind, n, rng):
    x = 3268 + 30 * rng.standard_normal(n)  # row sums of 4096 normal elements
    if kind == "a zero row":
        x[rng.integers(n)] = 0
    elif kind == "zero padding":
        x[:n // 8] = 0
    elif kind == "a huge row":
        x[rng.integers(n)] = 1e7
    elif kind == "heavy":
        x *= np.where(rng.random(n) < 0.02, 1.5 + 2.5 * rng.random(n), 1)
    elif kind == "tiny":
        x *= 1e-30
    elif kind.startswith("frames"):         # the norm follows the place inside the frame
        per = int(kind.split()[1])
        place = 3268 + 30 * rng.standard_normal(per)
        x = np.tile(place, -(-n // per))[:n] + rng.standard_normal(n)
    return x


SIZES = [(5, 5), (256, 8), (576, 8), (1500, 64), (2880, 16), (9216, 32), (16384, 16)]


@pytest.mark.parametrize("kind", ["plain", "a zero row", "zero padding", "a huge row", "heavy", "tiny"]
                         + [f"frames {p}" for p in (16, 64, 144, 219, 256, 510, 576, 1024)])
def test_candidates_are_the_best_and_few(search, kind):
    for n, P in SIZES:
        x = norms(kind, n, np.random.default_rng(n + P))
        for v in (-x.astype(np.float32), x.astype(np.float32)):
            cand = search(v, P)
            last = np.sort(v)[P - 1]
            must = v <= last + 2 * TAU * abs(last)
            assert np.all(cand[must]), (n, P)
            assert cand.sum() <= max(2 * P + 8, must.sum()), (n, P)


@pytest.mark.parametrize("beyond", [1, 7, 100, 100000])  # norms that overflow fp32
def test_norms_beyond_fp32_are_candidates(search, beyond):
    for n, P in SIZES:
        rng = np.random.default_rng(n + beyond)
        x = 3268 + 30 * rng.standard_normal(n)
        x[rng.permutation(n)[:beyond]] = np.inf
        for v in (-x, x):
            cand = search(v, P)
            assert cand.sum() >= P and np.all(cand[v <= np.sort(v)[P - 1]]), (n, P)


def test_undefined_norms_are_passed_over(search):
    v = -(3268 + 30 * np.random.default_rng(1).standard_normal(2880))
    v[::3] = np.nan
    cand = search(v, 16)
    assert 16 <= cand.sum() <= 40 and not cand[::3].any()
    assert not search(np.full(300, np.nan), 4).any()
