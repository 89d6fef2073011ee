"""The paper's grid where the search's range of scales can go wrong: one level
to 127, grids of a few points (a large eta against the weights), equal
magnitudes (no gap), lone large and sparse weights (bimodal errors), lengths at
powers of two, in lockstep against the oracle (the call takes eta in fp32: the
values here are fp32 values)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import say   # noqa: E402
from test_gpu_variants import _fit_paper, _ok   # noqa: E402


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


def _rows(d, seed):
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((8, d)).astype(np.float32)
    W[1] = np.float32(0.75) * rng.choice([-1, 1], d)          # one magnitude
    W[2, rng.random(d) < 0.9] = 0.0                             # sparse
    W[3] *= np.float32(0.01)
    W[3, d // 2] = 5.0                                          # a lone large weight
    W[4] = rng.integers(-3, 4, d)                               # many equal magnitudes
    W[5] *= np.float32(2.0 ** -12)                              # below eta
    W[6] = 0.0
    W[7] = np.where(np.arange(d) % 2, W[7], W[7] * np.float32(64.0))   # two scales
    return W


@pytest.mark.parametrize("d", [1, 2, 63, 64, 65, 128, 300, 513])
@pytest.mark.parametrize("bits,eta", [(2, 2.0 ** -10), (3, 0.5), (4, 2.0 ** -10), (4, 0.3125), (5, 2.0 ** -6), (8, 2.0 ** -10)])
def test_range_search(orc, d, bits, eta):
    if bits == 8 and d > 128:
        pytest.skip("the oracle's exact search costs O(d^2 M)")
    say(f"case paper search d={d} bits={bits} eta={eta}")
    W = _rows(d, 10 * d + bits)
    _ok(orc.verify_paper(W, bits, 3, 0.0, *_fit_paper(W, bits, 3, 0.0, eta), eta=eta))


@pytest.mark.parametrize("bits", [2, 3])
def test_all_weights_at_the_largest_code(orc, bits):
    """Rows near one magnitude with one large weight, whose best scale saturates every weight, left of all
    breakpoints."""
    say(f"case paper search, saturated, bits={bits}")
    rng = np.random.default_rng(40 + bits)
    d = 200
    W = np.empty((5, d), dtype=np.float32)
    W[0] = rng.choice([-1.0, 1.0], d)
    W[1] = np.abs(W[0])
    W[2] = np.float32(0.05) * (1 + np.float32(0.05) * rng.standard_normal(d).astype(np.float32))
    W[3] = rng.choice([-1.0, 0.0, 1.0], d)
    W[4] = rng.uniform(1.0, 1.17, d)
    W[:, 7] = np.float32(12.0 if bits == 2 else 25.0) * np.abs(W).max(1)
    out = _fit_paper(W, bits, 2, 0.0, 2.0 ** -10)
    assert (out[2] >= 1).all()
    _ok(orc.verify_paper(W, bits, 2, 0.0, *out))


@pytest.mark.parametrize("bits", [3, 5])
def test_grid_points_on_breakpoints(orc, bits):
    """Magnitudes in a narrow range, their gaps multiples of one spacing, and one large weight: breakpoints that fall
    on grid points."""
    say(f"case paper search, breakpoints on the grid, bits={bits}")
    rng = np.random.default_rng(50 + bits)
    d = 160
    W = np.empty((12, d), dtype=np.float32)
    W[:6] = rng.uniform(1.0, 1.17, (6, d))
    W[6:] = rng.integers(16, 20, (6, d)) / np.float32(16)
    W[:, d // 2] = np.float32([12, 16, 25] * 4)
    _ok(orc.verify_paper(W, bits, 2, 0.0, *_fit_paper(W, bits, 2, 0.0, 2.0 ** -10)))


def test_long_channels_at_the_largest_code(orc):
    """The same on the kernel for long channels (their sorted magnitudes in global memory)."""
    say("case paper search, saturated, d=8300")
    rng = np.random.default_rng(60)
    d = 8300
    W = np.empty((2, d), dtype=np.float32)
    W[0] = rng.choice([-1.0, 1.0], d)
    W[1] = np.float32(0.05) * (1 + np.float32(0.05) * rng.standard_normal(d).astype(np.float32))
    W[:, 11] = np.float32(40.0) * np.abs(W).max(1)
    out = _fit_paper(W, 2, 1, 0.0, 2.0 ** -10)
    assert (out[2] == 1).all() and (out[1][:, 0] < 2 * np.abs(W[:, 0])).all()
    _ok(orc.verify_paper(W, 2, 1, 0.0, *out))
