"""The paper grid's pruned search (the kernels' source, compiled for the host)
against the oracle's search of every breakpoint: the error of the scale it
takes is the oracle's, to the rounding of the sums."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ETA = 2.0 ** -10


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "paper_search.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "paper_2002_09049_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "paper_search_host.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    lib.paper_search_host.restype = ctypes.c_longlong
    lib.paper_search_host.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_double,
                                      ctypes.c_longlong, ctypes.c_void_p]

    def run(r, M, gamma, count):
        r = np.ascontiguousarray(r, dtype=np.float64)
        E = ctypes.c_double()
        g = lib.paper_search_host(r.ctypes.data, r.size, M, gamma, count, ctypes.byref(E))
        return int(g), E.value
    return run


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


def outlier_rows(kind, d, seed):
    """Rows as pruned or binarized layers have them: near one magnitude, and one large weight."""
    rng = np.random.default_rng(seed)
    if kind == "binary":
        r = rng.choice([-1.0, 1.0], d)
    elif kind == "ternary":
        r = rng.choice([-1.0, 0.0, 1.0], d)
    elif kind == "narrow":
        r = (rng.uniform(1.0, 1.17, d) * rng.choice([-1, 1], d)).astype(np.float32)
    elif kind == "dyadic":
        r = rng.integers(16, 20, d) / 16.0
    elif kind == "small":
        r = np.float32(0.05) * (1 + np.float32(0.05) * rng.standard_normal(d).astype(np.float32))
    else:
        r = rng.standard_normal(d).astype(np.float32)
    r = np.asarray(r, dtype=np.float32).astype(np.float64)
    r[d // 2] = np.float32(rng.choice([2.0, 12.0, 16.0, 25.0]) * np.abs(r).max())
    return r


def check(search, orc, r, bits, eta):
    gamma, count = orc.paper_grid(r, bits, eta)
    go, eo = orc.paper_grid_search(r, bits, gamma, count)
    g, e = search(r, (1 << (bits - 1)) - 1, gamma, count)
    # both sum d M terms of A and B in fp64, each product at most 2 ||r||^2 near the optimum
    slack = 1e-13 * float(r @ r)
    assert (g > 0) == (go > 0)
    assert go == 0 or abs(e - eo) <= slack, (g, e, go, eo, gamma, count)


def test_all_at_the_largest_code(search, orc):
    """Where the best scale saturates every weight, it lies left of every breakpoint."""
    for d, big, bits in ((200, 12.0, 2), (999, 16.0, 2), (300, 9.0, 3)):
        r = np.ones(d)
        r[::2] = -1.0
        r[d // 3] = big
        check(search, orc, r, bits, ETA)
    r = np.float32(0.05) * (1 + np.float32(0.05) * np.random.default_rng(1).standard_normal(1152).astype(np.float32))
    r = r.astype(np.float64)
    r[7] = np.float32(0.6)
    check(search, orc, r, 2, ETA)
    for seed in range(40):
        for kind in ("binary", "small", "narrow"):
            check(search, orc, outlier_rows(kind, 100 + seed, seed), 2, [ETA, 2.0 ** -6, 0.3125][seed % 3])


def test_grid_points_on_breakpoints(search, orc):
    """gamma is a fraction of a gap, so that breakpoints fall on grid points, and their quotient a rounding off."""
    for seed in range(60):
        d = 150 + 7 * seed % 220
        for kind in ("narrow", "dyadic", "ternary"):
            for bits in (3, 4, 5):
                check(search, orc, outlier_rows(kind, d, 1000 + seed), bits, ETA)


def test_other_rows(search, orc):
    """Ordinary rows, and gaps so small that a grid point's number exceeds a double's precision."""
    for seed in range(20):
        for bits in (2, 3, 4, 5, 6):
            check(search, orc, outlier_rows("normal", 40 + 9 * seed, seed), bits, ETA)
        r = np.random.default_rng(seed).standard_normal(30 + seed).astype(np.float32).astype(np.float64)
        r[3] = r[4] * (1 + 2.0 ** -40)
        r[5] = r[6] + 2.0 ** -48
        for bits in (2, 3, 5):
            check(search, orc, r, bits, ETA)
