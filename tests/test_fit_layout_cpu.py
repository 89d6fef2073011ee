"""Host-side check of where the fit's variants that hold groups of four
consecutive elements per thread (j = 4 (t + T v) + c) write their rows of the
output error's residual D: tiles of 128 rows by 32 k, row-major inside.  A
group is one float4 at ((j0 / 32) 4096 + j0 % 32) floats past the row's first
element, stored while j0 < 32 ceil(d / 32)."""
import os
import re

import numpy as np
import pytest

from test_layout_cpu import tiled_slot

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2002_09049_amd", "csrc", "fit_hist.hip")


def _variants(table):
    body = re.search(table + r"\[\]\s*=\s*\{(.*?)\};", open(SRC).read(), re.S).group(1)
    return [(int(t), int(e)) for t, e, quad in re.findall(r"\{\s*(\d+)\s*,\s*(\d+)\s*,\s*(true|false)\s*\}", body)
            if quad == "true"]


@pytest.mark.parametrize("T,EPT", _variants("kVariants") + _variants("kWide"))
def test_quad_rows_land_in_their_row(T, EPT):
    cap = T * EPT
    for d in sorted({1, 33, cap // 2 + 1, cap - 31, cap - 1, cap}):
        if d > 32768:
            continue
        nkb = (d + 31) // 32
        j0 = 4 * (np.arange(T)[:, None] + T * np.arange(EPT // 4)[None, :])
        j0 = j0[j0 < nkb * 32]
        assert cap >= 32 * nkb and (j0 % 4 == 0).all()
        for k in (0, 127, 300):
            base = (k // 128) * nkb * 4096 + (k % 128) * 32
            first = base + (j0 // 32) * 4096 + j0 % 32
            assert (first % 4 == 0).all()                      # one aligned float4
            addr = (first[:, None] + np.arange(4)).ravel()
            j = (j0[:, None] + np.arange(4)).ravel()
            assert sorted(j.tolist()) == list(range(32 * nkb))  # the row and its padding, once
            assert np.array_equal(addr, tiled_slot(k, j, nkb))


def test_every_variant_has_its_kernels():
    """Each mode's source lists every variant that the dispatch can choose with it: all of them, for the lattice those
    of at least 1024 elements."""
    text = open(SRC).read()
    table = [(int(t), int(e)) for name in ("kVariants", "kWide")
             for t, e in re.findall(r"\{\s*(\d+)\s*,\s*(\d+)\s*,", re.search(name + r"\[\]\s*=\s*\{(.*?)\};", text, re.S).group(1))]
    assert len(table) == 16 and "cap >= 1024" in text
    for mode in ("grid", "wide", "linear1", "linear3", "linear7", "lattice1", "lattice3", "lattice7", "lattice15"):
        src = open(SRC.replace("fit_hist.hip", f"fit_hist_{mode}.hip")).read()
        name, levels = re.fullmatch(r"([a-z]+)(\d*)", mode).groups()
        got = re.findall(r"if \(T == (\d+) && ept == (\d+)\) return launch_hist_t<(\d+), (\d+), kHist(\w+), (\d+)>", src)
        assert all((t, e) == (t2, e2) and m.lower() == name and k == (levels or "0") for t, e, t2, e2, m, k in got)
        want = [v for v in table if name != "lattice" or v[0] * v[1] >= 1024]
        assert sorted((int(t), int(e)) for t, e, *_ in got) == sorted(want), mode
