"""CPU tests of the places of a reduced problem's columns (paper_1405_7537_amd/csrc/columns.h): the decreasing order
for eigenvalues in their intervals, and a permutation whatever the solver returned."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shim") / "libcolumns_shim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(HERE, "host", "columns_shim.cpp"), "-o", out])
    L = C.CDLL(out)
    dp = np.ctypeslib.ndpointer(np.float64, flags="C_CONTIGUOUS")
    L.shim_places.argtypes = [C.c_int64, C.c_int64, dp, dp, C.c_int, dp,
                              np.ctypeslib.ndpointer(np.int64, flags="C_CONTIGUOUS")]

    def places(lam, d, neg, val):
        n = lam.size + val.size
        out = np.empty(n, np.int64)
        pad = lambda x: np.ascontiguousarray(x if x.size else np.zeros(1))  # noqa: E731
        L.shim_places(n, lam.size, pad(lam), pad(d), neg, pad(val), out)
        return out
    return places


def problem(m, c, neg, seed):
    """Poles, eigenvalues inside their intervals and a reduction's columns, many of them equal to poles."""
    rng = np.random.default_rng(seed)
    d = np.sort(rng.standard_normal(m))[::-1].copy()
    ends = np.concatenate([[d[0] + 1.0], d]) if not neg else np.concatenate([d, [d[-1] - 1.0]])
    f = rng.random(m)
    lam = ends[1:] * f + ends[:-1] * (1.0 - f)
    if m > 3:
        lam[1] = ends[1]                           # on an end, where two intervals meet
        lam[2] = ends[2]
    val = np.sort(np.concatenate([rng.standard_normal(c - c // 2), rng.choice(np.concatenate([d, lam]), c // 2)]))
    return d, lam, val[::-1].copy()


SHAPES = [(1, 0), (1, 3), (2, 2), (40, 0), (40, 1), (37, 50), (300, 30)]


@pytest.mark.parametrize("neg", [0, 1])
@pytest.mark.parametrize("m,c", SHAPES)
def test_places_are_the_stable_decreasing_order(shim, m, c, neg):
    d, lam, val = problem(m, c, neg, m + c)
    place = shim(lam, d, neg, val)
    # the reduction's columns first among equal values
    order = np.argsort(-np.concatenate([val, lam]), kind="stable")
    want = np.empty(m + c, np.int64)
    want[order] = np.arange(m + c)
    assert np.array_equal(place, np.concatenate([want[c:], want[:c]]))


@pytest.mark.parametrize("neg", [0, 1])
@pytest.mark.parametrize("m,c", SHAPES)
def test_places_are_a_permutation_whatever_was_computed(shim, m, c, neg):
    rng = np.random.default_rng(m)
    d, lam, val = problem(m, c, neg, m + c)
    for kind in range(5):
        x = lam.copy()
        if kind == 0:                              # a few roundings off, out of order
            x = x * (1.0 + 4e-16 * rng.integers(-3, 4, m))
            x[1::2] = x[: 2 * (m // 2) : 2] * (1.0 + 2.3e-16)
        elif kind == 1:
            rng.shuffle(x)
        elif kind == 2:
            x[rng.random(m) < 0.5] = np.nan
        elif kind == 3:
            x[:] = rng.choice([np.inf, -np.inf, np.nan, 0.0], m)
        else:
            x = x[::-1].copy()
        assert np.array_equal(np.sort(shim(x, d, neg, val)), np.arange(m + c)), kind
