"""The calls whose speed on one GPU matters to a user of this library, as cases.

A case is one call of a public entry point at one size.  `listed` are the
calls a quantization of the networks in `workloads` makes, from one small
layer to VGG-16's classifier; `draw` gives others of the same ranges (odd
lengths, few and many channels, other bit widths, grids and batches).
Weights, batches and activations are drawn on the GPU from the distributions
of `workloads`.
"""
import math

import torch

from paper_2002_09049_amd import mpq, workloads as wl

DEV = "cuda"
ETA = 2.0 ** -10      # the paper's maximal grid step
SHIFT = 16            # p of Eq. (14)
IMAGES = 8            # images of 224 x 224 in a deployment batch


def listed():
    return [
        # one small conv layer, the whole path: what a call costs when latency and launches count
        dict(name="net_conv64x576", kind="net", layers="conv64x576", bits=4, points=4, grid=128, tol=1e-3, n=256),
        # whole networks, the whole path in one call: an ordinary one, the default benchmark,
        # one of many short (depthwise and pointwise) channels, and the largest layers there are
        dict(name="net_resnet18", kind="net", layers="resnet18", bits=4, points=4, grid=256, tol=1e-3, n=1024),
        dict(name="net_resnet50", kind="net", layers="resnet50", bits=4, points=8, grid=256, tol=1e-3, n=1024),
        dict(name="net_mobilenetv2", kind="net", layers="mobilenetv2", bits=4, points=8, grid=512, tol=1e-3, n=1024),
        dict(name="net_vgg16fc", kind="net", layers="vgg16fc", bits=3, points=8, grid=512, tol=5e-4, n=2048),
        # Algorithm 2 with its calibration batch: a fit step and a scoring of every layer per point
        dict(name="calib_resnet18", kind="calib", layers="resnet18", bits=4, points=4, grid=256, tol=1e-3, n=1024),
        # one layer at a time: 8-bit codes (a network's classifier), and a caller's own grid
        # with the least-squares refit
        dict(name="layer_w8", kind="layer", c=1000, d=2048, bits=8, points=4, grid=256, tol=1e-6, own_grid=False,
             option="none"),
        dict(name="layer_own_grid", kind="layer", c=256, d=1152, bits=4, points=4, grid=200, tol=1e-3, own_grid=True,
             option="refit"),
        # the paper's own grid of Eq. (11), two points a channel (a third one is often the code of a single large
        # weight, for which a scale a at code 5 and a scale 5 a at code 1 have the same error)
        dict(name="layer_paper_grid", kind="paper", c=128, d=1152, bits=4, points=2, tol=1e-3),
        # scoring one layer of odd sizes on a batch, with the reference error
        dict(name="error_odd", kind="error", c=999, d=2047, bits=4, points=4, n=1001),
        # deployment: the integer forward of a whole network on a batch of images, and of one
        # classifier on a few vectors
        dict(name="int_resnet50", kind="int", layers="resnet50", bits=4, points=8),
        dict(name="int_fc", kind="int", layers="1000x2048@8", bits=4, points=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _stack(rng, most):
    """1 to 6 layers of at most `most` weights each."""
    out = []
    for _ in range(rng.randint(1, 6)):
        d = _log(rng, 9, 25088) if rng.random() < 0.25 else _log(rng, 9, 4608)
        if rng.random() < 0.5:
            d = max(16, d // 16 * 16)
        out.append("%dx%d" % (min(_log(rng, 16, 2048), max(1, most // d)), d))
    return ",".join(out)


def draw(rng):
    kind = rng.choice(["net", "net", "net", "calib", "layer", "layer", "paper", "error", "int", "int"])
    bits = rng.choice([2, 3, 4, 4, 4, 5, 8])
    points = rng.choice([2, 3, 4, 4, 6, 8])
    grid = rng.choice([64, 100, 128, 200, 256, 256, 300, 512])
    tol = {2: 1e-2, 3: 1e-3, 4: 1e-3, 5: 2e-4, 8: 1e-6}[bits]
    if kind in ("net", "calib"):
        return dict(kind=kind, layers=_stack(rng, 1 << 22), bits=bits, points=points, grid=grid, tol=tol,
                    n=_log(rng, 64, 2048))
    d = _log(rng, 9, 4608)
    if rng.random() < 0.5:
        d = max(16, d // 16 * 16)
    if kind == "layer":
        return dict(kind=kind, c=_log(rng, 16, 2048), d=d, bits=bits, points=points, grid=grid, tol=tol,
                    own_grid=rng.random() < 0.4, option=rng.choice(["none", "refit", "asym"]))
    if kind == "paper":
        return dict(kind=kind, c=_log(rng, 16, 128), d=_log(rng, 64, 2304), bits=rng.choice([3, 4]), points=2, tol=1e-3)
    if kind == "error":
        return dict(kind=kind, c=_log(rng, 16, 2048), d=d, bits=bits, points=points, n=_log(rng, 64, 2048))
    return dict(kind=kind, layers="%dx%d@%d" % (_log(rng, 16, 1024), d, _log(rng, 1, 25088)), bits=bits, points=points)


# ------------------------------------------------------------------ inputs
def _shapes(case):
    """(C, d) of every layer, and the columns of its batch."""
    s = case["layers"]
    if s in wl.WORKLOADS:
        shapes = list(wl.get(s).layers)
        if case["kind"] == "int":
            return [(c, d, IMAGES * hw * hw) for (c, d), hw in zip(shapes, wl.resnet50_out_hw())]
        return [(c, d, case["n"]) for c, d in shapes]
    out = []
    for t in s.split(","):
        t, _, n = t.partition("@")
        c, _, d = t.partition("x")
        out.append((int(c), int(d), int(n) if n else case["n"]))
    return out


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _weights(gen, c, d, laplace):
    """Rows of `workloads`: N(0, 2 / d) with a log-normal factor per channel, or Laplace with 0.1% of outliers."""
    sigma = math.sqrt(2.0 / d)
    if laplace:
        u = torch.rand((c, d), generator=gen, device=DEV, dtype=torch.float32) - 0.5
        w = -sigma / math.sqrt(2.0) * torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999))
        out = torch.rand((c, d), generator=gen, device=DEV) < 0.001
        return torch.where(out, torch.sign(w) * 8.0 * sigma, w).contiguous()
    w = torch.randn((c, d), generator=gen, device=DEV) * sigma
    return w * torch.exp(0.5 * torch.randn((c, 1), generator=gen, device=DEV))


def _batch(gen, d, n, relu):
    x = torch.randn((d, n), generator=gen, device=DEV)
    return x.clamp_(min=0.0) if relu else x


def _net_inputs(case, seed):
    gen = _gen(seed)
    laplace = case["layers"] == "resnet50"
    relu = case["layers"] in ("resnet18", "resnet50")
    shapes = _shapes(case)
    W = [_weights(gen, c, d, laplace) for c, d, _ in shapes]
    X = [_batch(gen, d, n, relu) for _, d, n in shapes]
    return W, X


def _multipliers(case):
    """A caller's grid: geometric, from 1 / 8 to 1."""
    g = case["grid"]
    return torch.exp(torch.linspace(math.log(0.125), 0.0, g, dtype=torch.float64)).float().clamp(max=1.0).numpy()


def _some_points(gen, W, bits, points):
    """Points as a fit leaves them: each the rounding of the residual, at 0.8 of its largest magnitude; mostly 2 or 3."""
    M = (1 << (bits - 1)) - 1
    c, d = W.shape
    codes = torch.zeros((c, points, d), dtype=torch.int8, device=DEV)
    scales = torch.zeros((c, points), device=DEV)
    u = torch.rand((c,), generator=gen, device=DEV)
    counts = (2 + (u > 0.6).int() + (u > 0.9).int() + (u > 0.97).int()).clamp(max=points).int()
    r = W
    for i in range(min(points, 5)):
        a = (r.abs().amax(1, keepdim=True) * 0.8 / M).clamp(min=1e-30)
        q = torch.round(r / a).clamp(-M, M)
        live = (counts > i)[:, None]
        codes[:, i] = torch.where(live, q, 0.0).to(torch.int8)
        scales[:, i] = torch.where(live, a, 0.0)[:, 0]
        r = torch.where(live, r - a * q, r)
    return codes, scales, counts


def _int_inputs(case, seed):
    """Fitted codes, integer scales and int8 activations (im2col rows of 0 .. 127) of every layer."""
    gen = _gen(seed)
    out = []
    for c, d, n in _shapes(case):
        codes, scales, counts = _some_points(gen, _weights(gen, c, d, False), case["bits"], case["points"])
        A = torch.round(scales.double() * 2.0 ** SHIFT).to(torch.int32)
        X = torch.empty((n, d), dtype=torch.int8, device=DEV)
        for a in range(0, n, 1 << 15):
            X[a:a + (1 << 15)] = (torch.randn((min(n - a, 1 << 15), d), generator=gen, device=DEV) * 40.0).clamp_(0.0, 127.0)
        out.append((codes, A, counts, X))
    return out


# --------------------------------------------------------- outputs of a network
def _offsets(sizes):
    """Starts of segments of these sizes, each a multiple of 64 values, and their end."""
    at, cur = [], 0
    for s in sizes:
        at.append(cur)
        cur += (s + 63) // 64 * 64
    return at, cur


def _flat(parts):
    """The parts' values in one buffer, laid out as _Net lays them out."""
    at, end = _offsets([p.numel() for p in parts])
    out = torch.zeros((max(end, 1),), dtype=parts[0].dtype, device=DEV)
    for a, p in zip(at, parts):
        out[a:a + p.numel()] = p.reshape(-1)
    return out


class _Net(mpq.LayerSet):
    """A LayerSet whose outputs lie one layer behind the other in one buffer per kind, as a program that stores or
    ships a quantized network holds them."""

    KINDS = ("codes", "scales", "counts", "fit_err", "err", "W_hat", "xerr", "offsets")
    FIELD = {"err": "out_err", "xerr": "fit_xerr"}

    def __init__(self, weights, max_points, calib=None):
        super().__init__(weights, max_points, calib=calib)
        self.flat = {}
        for kind in self.KINDS:
            parts = getattr(self, kind)
            if parts[0] is None:
                continue
            at, end = _offsets([p.numel() for p in parts])
            buf = torch.zeros((max(end, 1),), dtype=parts[0].dtype, device=DEV)
            self.flat[kind] = buf
            for i, p in enumerate(parts):
                parts[i] = buf[at[i]:at[i] + p.numel()].view(p.shape)
                name = self.FIELD.get(kind, kind)
                if getattr(self.arr[i], name) is not None:
                    setattr(self.arr[i], name, parts[i].data_ptr())

    def outputs(self, *kinds):
        return {k: self.flat[k] for k in kinds}


# --------------------------------------------------------------------- the calls
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("net", "calib"):
        W, X = _net_inputs(case, seed)
        return dict(case=case, net=_Net(W, case["points"], X))
    if kind in ("layer", "paper"):
        gen = _gen(seed)
        W = _weights(gen, case["c"], case["d"], False)
        st = dict(case=case, W=W)
        if kind == "paper" or case["option"] != "none":
            st["net"] = _Net([W], case["points"])
        if kind == "layer":
            st["grid"] = _multipliers(case) if case["own_grid"] else None
        return st
    if kind == "error":
        gen = _gen(seed)
        W = _weights(gen, case["c"], case["d"], False)
        return dict(case=case, W=W, points=_some_points(gen, W, case["bits"], case["points"]),
                    X=_batch(gen, case["d"], case["n"], True))
    layers = _int_inputs(case, seed)
    at, end = _offsets([c.shape[0] * X.shape[0] for c, _, _, X in layers])
    Y = torch.zeros((end,), dtype=torch.int64, device=DEV)
    full = [(c, A, k, X, Y[a:a + c.shape[0] * X.shape[0]].view(c.shape[0], X.shape[0]))
            for a, (c, A, k, X) in zip(at, layers)]
    return dict(case=case, layers=full, Y=Y)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "net":
        state["net"].quantize(case["bits"], case["grid"], case["tol"])
        return state["net"].outputs("codes", "scales", "counts", "fit_err", "err", "W_hat")
    if kind == "calib":
        state["net"].fit_calib(case["bits"], case["grid"], case["tol"], relative=True)
        return state["net"].outputs("codes", "scales", "counts", "fit_err", "xerr")
    if kind == "layer" and case["option"] == "none":
        codes, scales, counts, err = mpq.fit_layer(state["W"], case["bits"], case["points"], case["grid"], case["tol"],
                                                   grid=state["grid"])
        return dict(codes=codes, scales=scales, counts=counts, fit_err=err)
    if kind == "layer":
        opt = case["option"]
        state["net"].fit_ex(case["bits"], case["grid"], case["tol"], refit=opt == "refit", asym=opt == "asym",
                            grid=state["grid"])
        return state["net"].outputs("codes", "scales", "counts", "fit_err", *(["offsets"] if opt == "asym" else []))
    if kind == "paper":
        state["net"].fit_ex(case["bits"], 256, case["tol"], paper_eta=ETA)
        return state["net"].outputs("codes", "scales", "counts", "fit_err")
    if kind == "error":
        err, ref = mpq.output_error(state["W"], *state["points"], state["X"], with_ref=True)
        return dict(err=err, ref=ref)
    if len(state["layers"]) == 1:
        codes, A, counts, X, Y = state["layers"][0]
        mpq.integer_forward(codes, A, counts, X, SHIFT, out=Y)
    else:
        mpq.integer_forward_layers(state["layers"], case["points"], SHIFT)
    return state["Y"]


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: the products of the contractions (the fit's search
    has no count that every method needs)."""
    kind = case["kind"]
    P = case["points"]
    if kind in ("net", "calib"):
        b = f = 0.0
        for c, d, n in _shapes(case):
            b += 4.0 * c * d + 4.0 * d * n + 1.0 * P * c * d + c * (8.0 * P + 8.0)
            f += 2.0 * c * d * n * (1 if kind == "net" else 3)
            if kind == "net":
                b += 4.0 * c * d
        return dict(bytes=b, flops=f)
    if kind in ("layer", "paper"):
        c, d = case["c"], case["d"]
        return dict(bytes=c * d * (4.0 + P) + c * (8.0 * P + 4.0), flops=0.0)
    if kind == "error":
        c, d, n = case["c"], case["d"], case["n"]
        return dict(bytes=c * d * (4.0 + 2.5) + 4.0 * d * n + 8.0 * c, flops=4.0 * c * d * n)
    b = f = 0.0
    for c, d, n in _shapes(case):
        b += 2.5 * c * d + 1.0 * n * d + 8.0 * c * n
        f += 2.0 * 2.5 * c * d * n
    return dict(bytes=b, flops=f)


def tolerance(case):
    kind = case["kind"]
    if kind == "int":
        return "exact"
    # fp32 evaluation of the output error over up to 25,088 terms (1.2e-7 against 64 bits, and up to 1e-6 for one row);
    # the fit's own errors are fp64 sums in fp32 (3e-8).  Codes, scales and counts are the argmin's: another order of
    # summation may flip a tie of two candidates in a channel.
    return {"rel": 1e-5, "max": 2e-4, "differ": 1e-5}


# ---------------------------------------------------------------- in 64 bits
def _fit64(W, M, P, mult, stop, refit=False, asym=False):
    """Algorithm 1 with every candidate evaluated: (scales, err, points, offsets); stop(rows, n, r2, what) says which
    rows end before point n + 1."""
    w = W.double()
    beta = ((w.amax(1) + w.amin(1)) / 2).float() if asym else torch.zeros((w.shape[0],), device=DEV)
    r = w - beta.double()[:, None]
    C, d = w.shape
    scales = torch.zeros((C, P), device=DEV)
    err = torch.zeros((C, P), dtype=torch.float64, device=DEV)
    what = beta.double()[:, None].repeat(1, d)
    rows = torch.arange(C, device=DEV)
    G = mult.numel()
    step = max(1, (1 << 26) // (d * G))
    for n in range(P):
        r2 = r[rows].square().sum(1)
        rows = rows[(r2 > 0) & ~stop(rows, n, r2, what)]
        for k in range(0, rows.numel(), step):
            part = rows[k:k + step]
            rp = r[part]
            a = (rp.abs().amax(1).float().double()[:, None] * mult / M).float().double()
            q = (rp.abs()[:, :, None] / a[:, None, :]).round_().clamp_(max=M)
            e = q.mul_(a[:, None, :]).sub_(rp.abs()[:, :, None]).square_().sum(1)
            e[a == 0] = math.inf
            best = a.gather(1, e.argmin(1, keepdim=True))
            q = (rp / best).round_().clamp_(-M, M)
            if refit:
                best = ((rp * q).sum(1, keepdim=True) / q.square().sum(1, keepdim=True)).float().double()
            scales[part, n] = best[:, 0].float()
            r[part] = rp - best * q
            what[part] += best * q
            err[part, n] = r[part].square().sum(1)
        if rows.numel() == 0:
            break
    return scales, err, what, beta


def _paper64(W, M, P, tol):
    """The fit on Eq. (11)'s grid: every grid point next to a breakpoint of E or to the vertex of its piece."""
    r = W.double()
    C, d = r.shape
    scales = torch.zeros((C, P), device=DEV)
    err = torch.zeros((C, P), dtype=torch.float64, device=DEV)
    w2 = r.square().sum(1)
    live = torch.ones((C,), dtype=torch.bool, device=DEV)
    for n in range(P):
        r2 = r.square().sum(1)
        live = live & (r2 > 0) & ((r2 > tol * w2) if n else torch.ones_like(live))
        s = r.abs().sort(1).values
        S = torch.cat([torch.zeros((C, 1), dtype=torch.float64, device=DEV), s.flip(1).cumsum(1)], 1)
        gap = s.diff(dim=1)
        gap = torch.where(gap > 0, gap, math.inf).amin(1)
        gamma = torch.clamp(gap / 2 / M, max=ETA)[:, None]
        count = torch.floor(2 * M * r2.sqrt()[:, None] / gamma)

        def sums(g):
            a = g * gamma
            A, B = torch.zeros_like(a), torch.zeros_like(a)
            for k in range(M):
                c = d - torch.searchsorted(s, (a * (k + 0.5)).contiguous(), right=k % 2 == 0)
                A += S.gather(1, c)
                B += (2 * k + 1) * c
            E = r2[:, None] - 2 * a * A + a * a * B
            return torch.where((g >= 1) & (g <= count), E, math.inf), A, B

        best_e = torch.full((C,), math.inf, dtype=torch.float64, device=DEV)
        best_g = torch.zeros_like(best_e)
        for k in range(M):
            for off in (-1, 0, 1):
                g = torch.floor(s / (k + 0.5) / gamma) + off
                E, A, B = sums(g)
                gv = torch.floor(A / B.clamp(min=1) / gamma)
                for E, g in ((E, g), (sums(gv)[0], gv), (sums(gv + 1)[0], gv + 1)):
                    e, at = E.min(1)
                    better = e < best_e
                    best_e = torch.where(better, e, best_e)
                    best_g = torch.where(better, g.gather(1, at[:, None])[:, 0], best_g)
        a = torch.where(live, (best_g * gamma[:, 0]).float(), 0.0)
        q = torch.where(live[:, None], (r / a.double()[:, None]).round().clamp(-M, M), 0.0)
        r = r - a.double()[:, None] * q
        scales[:, n] = a
        err[:, n] = torch.where(live, r.square().sum(1), 0.0)
    return scales, err


def _grid64(case):
    if case.get("own_grid"):
        return torch.from_numpy(_multipliers(case)).to(DEV).double()
    g = case["grid"]
    return (torch.arange(1, g + 1, dtype=torch.float64) / g).float().double().to(DEV)


def _error64(D, X):
    return (D.double() @ X.double()).square().mean(1)


def exact(case, seed):
    """The floating outputs of run() in 64 bits, None in the place of whole ones."""
    kind = case["kind"]
    P = case["points"]
    M = (1 << (case["bits"] - 1)) - 1
    tol = torch.tensor(case.get("tol", 0.0)).double().item()   # the fp32 value
    if kind in ("net", "calib"):
        W, X = _net_inputs(case, seed)
        if sum(w.numel() for w in W) * case["grid"] > 2e11:
            return None
        mult = _grid64(case)
        got = []
        for w, x in zip(W, X):
            w2 = w.double().square().sum(1)
            if kind == "net":
                s, e, what, _ = _fit64(w, M, P, mult, lambda rows, n, r2, _w: (r2 <= tol * w2[rows]) & (n > 0))
                got.append((s, e, _error64(w.double() - what, x), what))
                continue
            ref = _error64(w, x)
            xerr = torch.zeros((w.shape[0], P), dtype=torch.float64, device=DEV)

            def stop(rows, n, r2, what):
                if n == 0:
                    return torch.zeros_like(r2, dtype=torch.bool)
                xerr[rows, n - 1] = _error64(w[rows].double() - what[rows], x)
                return xerr[rows, n - 1] <= tol * ref[rows]

            s, e, what, _ = _fit64(w, M, P, mult, stop)
            full = s[:, P - 1] != 0
            xerr[full, P - 1] = _error64(w[full].double() - what[full], x)
            got.append((s, e, xerr))
        parts = [_flat([g[i] for g in got]) for i in range(len(got[0]))]
        names = ("scales", "fit_err", "err", "W_hat") if kind == "net" else ("scales", "fit_err", "xerr")
        return dict(zip(names, parts), codes=None, counts=None)
    if kind in ("layer", "paper"):
        W = _weights(_gen(seed), case["c"], case["d"], False)
        opt = case.get("option", "none")
        beta = None
        if kind == "paper":
            s, e = _paper64(W, M, P, tol)
        else:
            w2 = W.double().square().sum(1)
            s, e, _, beta = _fit64(W, M, P, _grid64(case), lambda rows, n, r2, _w: (r2 <= tol * w2[rows]) & (n > 0),
                                   refit=opt == "refit", asym=opt == "asym")
        if kind == "paper" or opt != "none":
            s, e = _flat([s]), _flat([e])
        out = dict(codes=None, scales=s, counts=None, fit_err=e)
        if opt == "asym":
            out["offsets"] = _flat([beta])
        return out
    if kind == "error":
        gen = _gen(seed)
        W = _weights(gen, case["c"], case["d"], False)
        codes, scales, _ = _some_points(gen, W, case["bits"], P)
        X = _batch(gen, case["d"], case["n"], True)
        D = W.double() - (scales.double()[:, :, None] * codes.double()).sum(1)
        return dict(err=_error64(D, X), ref=_error64(W, X))
    out = []
    for codes, A, counts, X in _int_inputs(case, seed):
        c, P, d = codes.shape
        y = torch.zeros((c, X.shape[0]), dtype=torch.int64, device=DEV)
        Xt = X.t().double()
        for i in range(P):
            y += A[:, i, None].long() * torch.round(codes[:, i].double() @ Xt).long()
        out.append(y >> SHIFT)
    return _flat(out)
