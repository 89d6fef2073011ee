"""The output error on both sides of the rule that chooses the GEMM's operand
pieces (layers of at least 256 rows, 384 for a large X, of at least 128, and an X whose features' root mean squares lie within 2^10
of its largest value, take fp16 ones): ranges within, just past and far past it, with a row of X of
zeros (bf16 ones) and without, tiny and huge scales, and non-finite values; formed rows (with the reference error), rows the
fit wrote, and a calibration fit's listed rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import gpu_fit, say   # noqa: E402
from test_gpu_parity import _gpu_err, _oracle_err   # noqa: E402


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


def _rows(C, d, n, spread, seed):
    """W, X: feature k of X has largest magnitude 2^e, e from 0 down to -spread; channels that live on
    the small features only among the others."""
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((C, d)).astype(np.float32)
    X = np.clip(rng.standard_normal((d, n)), -1, 1).astype(np.float32)
    X[:, 0] = 1.0
    e = -np.round(np.linspace(0, spread, d))
    X = (X * np.ldexp(1.0, e.astype(int))[:, None]).astype(np.float32)
    W[:: 3, : d // 2] *= np.float32(2.0 ** -20)
    W[1] = 0.0
    W[1, -1] = 1.0
    return W, X


@pytest.mark.parametrize("C,d,n", [(256, 129, 7), (300, 128, 200), (257, 1600, 130), (256, 127, 301), (255, 600, 90), (260, 2047, 33)])
@pytest.mark.parametrize("spread,xs,ws", [(0, 0, 0), (10, 0, 0), (11, 0, 0), (40, 0, 0), (10, -90, 20), (3, 90, -60)])
def test_against_oracle(orc, C, d, n, spread, xs, ws):
    say(f"case pieces C={C} d={d} n={n} spread={spread} xs={xs} ws={ws}")
    W, X = _rows(C, d, n, spread, C + d)
    X[d // 3] = 0.0
    W = (W * np.float32(2.0 ** ws)).astype(np.float32)
    X = (X * np.float32(2.0 ** xs)).astype(np.float32)
    out = gpu_fit(W, 4, 3, 64, 1e-3)
    eo, ro = _oracle_err(orc, W, out, X)
    eg, rg = _gpu_err(W, out, X)
    # fp32's own range: where the mean square is a normal fp32 value
    for g, o in ((eg, eo), (rg, ro)):
        ok = (o > 1e-36) & (o < 1e38)
        assert np.all(np.abs(g - o)[ok] <= 1e-5 * o[ok]), np.max(np.abs(g - o)[ok] / o[ok])


def test_whole_path_and_calibration(orc):
    """Rows of D from the fit, and listed rows, on both sides of the rule: equal to the error of formed rows."""
    import torch
    from paper_2002_09049_amd import mpq
    shapes = [(70, 12, 200), (300, 600, 200), (256, 900, 130)]
    for spread in (4, 30):
        Ws, Xs = zip(*(_rows(C, d, n, spread, 7 + d) for C, d, n in shapes))
        say(f"case whole path, spread={spread}")
        net = mpq.LayerSet([torch.from_numpy(w).cuda() for w in Ws], 3, calib=[torch.from_numpy(x).cuda() for x in Xs])
        net.quantize(4, 64, 1e-3)
        torch.cuda.synchronize()
        for i, (W, X) in enumerate(zip(Ws, Xs)):
            out = tuple(v[i].cpu().numpy() for v in (net.codes, net.scales, net.counts))
            eo, _ = orc.output_error(W, *out, X)
            g = net.err[i].cpu().numpy()
            assert np.all(np.abs(g - eo) <= 1e-5 * eo)
            # alone (a small step, its launches one after the other): the same bits
            one = mpq.LayerSet([torch.from_numpy(W).cuda()], 3, calib=[torch.from_numpy(X).cuda()])
            one.quantize(4, 64, 1e-3)
            torch.cuda.synchronize()
            for kind in ("codes", "scales", "counts", "fit_err", "err", "W_hat"):
                assert torch.equal(getattr(one, kind)[0], getattr(net, kind)[i]), kind
        net.fit_calib(4, 64, 1e-3, relative=True)
        torch.cuda.synchronize()
        for i, (W, X) in enumerate(zip(Ws, Xs)):
            codes, scales, counts = (v[i].cpu().numpy() for v in (net.codes, net.scales, net.counts))
            eo, _ = orc.output_error(W, codes, scales, counts, X)
            xe = net.xerr[i].cpu().numpy()
            live = counts > 0
            last = xe[np.arange(len(counts)), np.maximum(counts - 1, 0)]
            assert np.all(np.abs(last - eo)[live] <= 1e-5 * eo[live])


def test_not_finite():
    """An infinity or a NaN in a channel or in X gives what the products give: NaN in the rows that meet it."""
    C, d, n = 256, 200, 100
    say("case not finite")
    rng = np.random.default_rng(3)
    W = rng.standard_normal((C, d)).astype(np.float32)
    X = rng.standard_normal((d, n)).astype(np.float32)
    out = gpu_fit(W, 4, 2, 64, 1e-3)
    good, ref = _gpu_err(W, out, X)
    W2 = W.copy()
    W2[3, 5], W2[7, 100] = np.inf, np.nan
    eg, rg = _gpu_err(W2, out, X)
    for v, g in ((eg, good), (rg, ref)):
        assert np.all(np.isnan(v[[3, 7]]))
        rest = np.delete(np.arange(C), [3, 7])
        assert np.array_equal(v[rest], g[rest])
    for bad in (np.inf, np.nan):
        X2 = X.copy()
        X2[9, 11] = bad
        eg, rg = _gpu_err(W, out, X2)
        assert not np.any(np.isfinite(eg)) and not np.any(np.isfinite(rg))


@pytest.mark.parametrize("feature", ["dead", "once"])
@pytest.mark.parametrize("e", [18, 24, 28])
def test_large_weights_on_features_that_hardly_occur(feature, e):
    """Rows whose largest weights sit on features of X that are zero, or nonzero in one sample of many: the other
    weights, 2^-e of them, make the output error."""
    import torch
    from paper_2002_09049_amd import mpq
    C, d, n = 256, 512, 1024
    say(f"case rare features {feature} e={e}")
    rng = np.random.default_rng(e)
    W = (rng.uniform(0.5, 1.0, (C, d)) * rng.choice([-1.0, 1.0], (C, d)) * 2.0 ** -e).astype(np.float32)
    X = np.clip(rng.standard_normal((d, n)), -1, 1).astype(np.float32)
    rare = rng.choice(d, 4, replace=False)
    W[:, rare] = rng.uniform(0.5, 1.0, (C, 4))
    X[rare] = 0.0
    if feature == "once":
        X[rare, 5 + np.arange(4)] = np.float32(2.0 ** -9)
    codes = torch.zeros((C, 1, d), dtype=torch.int8, device="cuda")
    scales = torch.zeros((C, 1), device="cuda")
    counts = torch.zeros((C,), dtype=torch.int32, device="cuda")
    err, ref = mpq.output_error(torch.from_numpy(W).cuda(), codes, scales, counts, torch.from_numpy(X).cuda(), with_ref=True)
    want = ((W.astype(np.float64) @ X.astype(np.float64)) ** 2).mean(1)
    for got in (err, ref):
        # fp32 sums of 512 products of random signs, the mean over 1024 samples and one rounding: 2e-7 at most
        assert np.max(np.abs(got.cpu().numpy() - want) / want) <= 1e-6


@pytest.mark.parametrize("d,n", [(128, 1), (129, 3), (300, 4), (257, 17), (200, 260), (4097, 65), (131, 4096), (130, 4097),
                                 (600, 4100), (20000, 12)])
def test_scan_finds_its_features(orc, d, n):
    """A feature that the rule must not miss, at each place of the scan's rows and samples: a dead one under the largest
    weights, a value far past the others."""
    import torch
    from paper_2002_09049_amd import mpq
    C = 256
    say(f"case scan d={d} n={n}")
    rng = np.random.default_rng(d + n)
    X = rng.uniform(0.25, 1.0, (d, n)).astype(np.float32)
    Wn = (rng.uniform(0.5, 1.0, (C, d)) * 2.0 ** -28).astype(np.float32)
    codes = torch.zeros((C, 1, d), dtype=torch.int8, device="cuda")
    scales = torch.zeros((C, 1), device="cuda")
    counts = torch.zeros((C,), dtype=torch.int32, device="cuda")
    for j in sorted({0, 1, d // 3, 15, 16, 17, d - 2, d - 1}):
        W, Xd, Xt = Wn.copy(), X.copy(), X.copy()
        W[:, j] = 1.0
        Xd[j] = 0.0
        for x, w in ((Xd, W), (Xt, Wn)):
            if w is Wn:
                x[j, (7 * j) % n] = np.float32(2.0 ** 20)
            err = mpq.output_error(torch.from_numpy(w).cuda(), codes, scales, counts, torch.from_numpy(x).cuda())
            if isinstance(err, tuple):
                err = err[0]
            # in pieces of samples: sums of positive products, of d terms in fp32
            want = sum(((w.astype(np.float64) @ x[:, a:a + 4096].astype(np.float64)) ** 2).sum(1) for a in range(0, n, 4096)) / n
            rel = np.max(np.abs(err.cpu().numpy() - want) / want)
            assert rel <= 4e-6, (j, w is Wn, rel)


@pytest.mark.parametrize("C,d", [(256, 4096), (257, 4097), (300, 8224), (256, 140000), (16, 140000), (255, 4100)])
def test_row_maxima_of_long_rows(C, d):
    """Rows formed in several pieces, each row's largest weight far past the others and at another place (unseen, its
    fp16 pieces would overflow); layers whose maxima nobody needs beside them."""
    import torch
    from paper_2002_09049_amd import mpq
    n = 5
    say(f"case long rows C={C} d={d}")
    g = torch.Generator(device="cuda").manual_seed(d + C)
    W = torch.randn((C, d), generator=g, device="cuda")
    at = (torch.arange(C, device="cuda") * 7919 * 31) % d
    at[0], at[1], at[2] = 0, d - 1, d // 2
    W[torch.arange(C, device="cuda"), at] = 2.0 ** 17
    X = torch.rand((d, n), generator=g, device="cuda") + 0.5
    codes = torch.zeros((C, 1, d), dtype=torch.int8, device="cuda")
    codes[:, 0, d // 3] = 3
    scales = torch.full((C, 1), 0.25, device="cuda")
    counts = torch.ones((C,), dtype=torch.int32, device="cuda")
    err, ref = mpq.output_error(W, codes, scales, counts, X, with_ref=True)
    D = W.double()
    for got, want in ((ref, (D @ X.double()).square().mean(1)),
                      (err, ((D - 0.25 * codes[:, 0].double()) @ X.double()).square().mean(1))):
        # one product of 2^17 among d of random signs: fp32 sums, to a few of its roundings
        assert ((got.double() - want).abs() / want).max().item() <= 4e-6


def test_workspace_limit_at_the_scratch(monkeypatch):
    """MPQ_WORKSPACE_LIMIT at what the error's scratch takes, without the ranges and maxima beside it (an allocation of
    their own then): the same results; one byte less is refused."""
    import re
    import torch
    from paper_2002_09049_amd import mpq
    C, d, n = 300, 600, 200
    say("case workspace limit")
    W, X = (torch.from_numpy(a).cuda() for a in _rows(C, d, n, 4, 5))
    net = mpq.LayerSet([W], 3, calib=[X])

    def whole():
        net.quantize(4, 64, 1e-3)
        return net.err[0].clone(), net.W_hat[0].clone()

    def alone():
        return mpq.output_error(W, net.codes[0], net.scales[0], net.counts[0], X, with_ref=True)

    for call in (whole, alone):
        want = call()
        monkeypatch.setenv("MPQ_WORKSPACE_LIMIT", "64")
        with pytest.raises(mpq.MPQError) as e:
            call()
        assert e.value.status == mpq.MPQ_ERR_NOMEM
        total = int(re.search(r"scratch of (\d+) bytes", str(e.value)).group(1))
        monkeypatch.setenv("MPQ_WORKSPACE_LIMIT", str(total - 1))
        with pytest.raises(mpq.MPQError):
            call()
        monkeypatch.setenv("MPQ_WORKSPACE_LIMIT", str(total))
        got = call()
        monkeypatch.delenv("MPQ_WORKSPACE_LIMIT")
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("C", [255, 256, 383, 384])
@pytest.mark.parametrize("d,n", [(768, 4096), (769, 4096)])
def test_channels_where_the_pieces_change(orc, C, d, n):
    """Both sides of the fewest channels that take fp16 pieces, for X of 3 2^20 values and of more."""
    say(f"case fewest channels C={C} d={d} n={n}")
    W, X = _rows(C, d, n, 4, C + d)
    out = gpu_fit(W, 4, 2, 64, 1e-3)
    eo, ro = _oracle_err(orc, W, out, X)
    eg, rg = _gpu_err(W, out, X)
    assert np.all(np.abs(eg - eo) <= 1e-5 * eo) and np.all(np.abs(rg - ro) <= 1e-5 * ro)


@pytest.mark.parametrize("C,d,n", [(256, 129, 7), (300, 128, 200), (257, 1600, 130), (260, 2047, 33)])
@pytest.mark.parametrize("spread,xs,ws", [(0, 0, 0), (9, 0, 0), (10, 0, 0), (9, -49, 20), (9, -52, 20), (8, 60, -70)])
def test_against_oracle_without_dead_features(orc, C, d, n, spread, xs, ws):
    """The smallest feature's root mean square on both sides of 2^-10 of X's largest value (0.7 to 0.8 of its own
    largest one, 2^-spread), that value on both sides of 2^-50, and a large X with small weights."""
    say(f"case pieces, every feature alive, C={C} d={d} n={n} spread={spread} xs={xs} ws={ws}")
    W, X = _rows(C, d, n, spread, 3 * C + d)
    W = (W * np.float32(2.0 ** ws)).astype(np.float32)
    X = (X * np.float32(2.0 ** xs)).astype(np.float32)
    out = gpu_fit(W, 4, 3, 64, 1e-3)
    eo, ro = _oracle_err(orc, W, out, X)
    eg, rg = _gpu_err(W, out, X)
    for g, o in ((eg, eo), (rg, ro)):
        ok = (o > 1e-36) & (o < 1e38)
        assert np.all(np.abs(g - o)[ok] <= 1e-5 * o[ok]), np.max(np.abs(g - o)[ok] / o[ok])
