"""The histogram search's kernels against each other: the same channels fitted
by the variant of four wavefronts per channel (a call of few channels) and by
the one that a call of many channels takes must agree bit for bit, in every
mode (a default grid's lattice, linear and wide modes, and a caller's grid),
at the edges of the variants' lengths.  The rows include elements exactly on
code boundaries, tiny scales, outliers and equal magnitudes (many finalists),
and are themselves checked in lockstep against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import assert_parity, gpu_fit, say   # noqa: E402
from test_gpu_parity import _lattice_rows           # noqa: E402


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


@pytest.mark.parametrize("d", [257, 512, 513, 768, 769, 1023, 1280, 1281, 2304, 2560, 3072, 4608, 4609, 5120])
def test_few_and_many_channels_agree(orc, d):
    rng = np.random.default_rng(d)
    W = _lattice_rows(d, rng)
    many = np.ascontiguousarray(np.concatenate([W, rng.standard_normal((520, d)).astype(np.float32)]))
    geo = np.exp(np.linspace(np.log(0.05), 0.0, 200)).astype(np.float32)
    for bits, G, P, tol, grid in ((4, 256, 4, 0.0, None), (3, 100, 3, 1e-4, None), (2, 300, 3, 0.0, None),
                                  (5, 64, 3, 1e-5, None), (8, 256, 3, 1e-7, None), (4, 200, 3, 1e-4, geo)):
        say(f"case few/many d={d} bits={bits} G={G} grid={'own' if grid is not None else 'default'}")
        few = gpu_fit(W, bits, P, G, tol, grid=grid)
        assert_parity(orc, W, bits, P, G, tol, few, grid=grid)
        out = gpu_fit(many, bits, P, G, tol, grid=grid)
        for a, b in zip(few, out):
            assert np.array_equal(a, b[:len(W)])


@pytest.mark.parametrize("d,G", [(17, 4096), (64, 1), (65, 3), (128, 1024), (300, 4096), (1100, 1200), (2000, 1)])
def test_grid_sizes(orc, d, G):
    """Grids of one candidate to the largest, in the modes they select."""
    rng = np.random.default_rng([d, G])
    W = _lattice_rows(d, rng)[[0, 3, 4]]
    for bits in (2, 4, 8):
        say(f"case grid size d={d} G={G} bits={bits}")
        assert_parity(orc, W, bits, 3, G, 1e-6, gpu_fit(W, bits, 3, G, 1e-6))
        grid = np.sort(rng.choice(np.arange(1, 1 << 16), G, replace=False)).astype(np.float32) / np.float32(1 << 16)
        assert_parity(orc, W, bits, 3, G, 1e-6, gpu_fit(W, bits, 3, G, 1e-6, grid=grid), grid=grid)


def test_sparse_rows(orc):
    """Rows of mostly zeros (every zero falls below the lattice's first point)."""
    rng = np.random.default_rng(5)
    W = rng.standard_normal((6, 3000)).astype(np.float32)
    W[rng.random(W.shape) < 0.9] = 0.0
    for bits, G in ((4, 256), (8, 128)):
        assert_parity(orc, W, bits, 4, G, 1e-5, gpu_fit(W, bits, 4, G, 1e-5))


def _edge_grids(G, rng):
    """Multipliers on and beside the count table's entries (1024ths), all within one entry, tiny ones."""
    i = np.sort(rng.choice(np.arange(1, 1025), min(G, 1024), replace=False)).astype(np.float32) / np.float32(1024)
    yield i
    yield np.nextafter(i, np.float32(0))
    up = np.nextafter(i, np.float32(2))
    yield up[up <= 1]
    near = ((i * 1024 - np.float32(0.001)) / 1024).astype(np.float32)       # an entry's own value
    yield np.unique(np.concatenate([near, np.nextafter(near, np.float32(2)), np.nextafter(near, np.float32(0))]))
    yield np.float32(0.7) + np.arange(G, dtype=np.float32) * np.float32(2.0 ** -24)
    yield np.unique(np.geomspace(1e-6, 1.0, G).astype(np.float32))


@pytest.mark.parametrize("C,d,bits,G", [(3, 40, 4, 1), (4, 300, 2, 65), (5, 200, 8, 300), (2, 1300, 3, 1000), (2, 5000, 4, 130)])
def test_caller_grid_at_the_table_entries(orc, C, d, bits, G):
    rng = np.random.default_rng(G)
    W = (rng.standard_normal((C, d)) * np.exp(rng.standard_normal((C, 1)))).astype(np.float32)
    for k, grid in enumerate(_edge_grids(G, rng)):
        grid = np.ascontiguousarray(grid[:4096], dtype=np.float32)
        say(f"case table grid {k} C={C} d={d} bits={bits} G={grid.size}")
        out = gpu_fit(W, bits, 3, grid.size, 1e-4, grid=grid)
        assert_parity(orc, W, bits, 3, grid.size, 1e-4, out, grid=grid)


@pytest.mark.parametrize("d", [257, 512, 769, 1280])
def test_few_and_many_channels_agree_on_a_caller_grid(d):
    """On a caller's grid up to 1024 channels of one wavefront count as few: the same bits on both sides."""
    rng = np.random.default_rng(7 * d)
    rows = np.concatenate([_lattice_rows(d, rng), rng.standard_normal((1030, d)).astype(np.float32)])
    geo = np.exp(np.linspace(np.log(0.05), 0.0, 130)).astype(np.float32)
    for bits, tol in ((4, 1e-4), (2, 1e-2), (8, 1e-7)):
        say(f"case few/many on a caller's grid d={d} bits={bits}")
        few = gpu_fit(np.ascontiguousarray(rows[:1024]), bits, 3, geo.size, tol, grid=geo)
        many = gpu_fit(np.ascontiguousarray(rows), bits, 3, geo.size, tol, grid=geo)
        for a, b in zip(few, many):
            assert np.array_equal(a, b[:1024])
