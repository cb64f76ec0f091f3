"""Long lookups in tables that no bucket key spreads (the points of one bucket
are too many to compare), and at the size where segments no longer fit: bit for
bit the oracle's."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32
N = (1 << 21) + 3

TABLES = {
    "tail": np.concatenate([np.arange(0, 101, 5), [200, 500, 13000]]).astype(F),
    "signed": np.concatenate([[-1e4], np.arange(-5, 5.5, 0.5), [1e4]]).astype(F),
    "cluster": np.concatenate([[-1e6], 1 + np.arange(30) * 1e-4, [1e6]]).astype(F),
    "254 edges": np.concatenate([[-1e9], 1 + np.arange(252) * 1e-3, [1e9]]).astype(F),
}


def values(e, seed):
    rng = np.random.default_rng(seed)
    m = ((e[:-1] + e[1:]) * F(0.5)).astype(F)
    near = np.concatenate([e, m])
    s = np.concatenate([near, np.nextafter(near, F(np.inf)), np.nextafter(near, F(-np.inf)),
                        np.array([0, -0.0, np.nan, np.inf, -np.inf], F)])
    x = np.concatenate([s, rng.uniform(*sorted((e[1] - 1, e[-2] + 1)), N - s.size).astype(F)])
    rng.shuffle(x)
    return x


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def same(got, want):
    got = got.cpu().numpy()
    ok = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
    assert np.all(ok), f"{np.count_nonzero(~ok)} differ"


@pytest.mark.parametrize("name", list(TABLES))
def test_one_dimension(name):
    print("crowded table", name, flush=True)
    e = TABLES[name]
    c = np.random.default_rng(1).normal(1, 0.3, len(e) + 1).astype(F)
    x = values(e, 2)
    y = dev(np.concatenate([x[:1], x]))[1:]  # not aligned to four elements
    with np.errstate(invalid="ignore"):
        for v in (dev(x), y):
            same(H.get_bin_contents(v, dev(e), dev(c)), ref.get_bin_contents(x, e, c))
            same(H.interp(v, dev(e), dev(c)), ref.interp(x, e, c))


@pytest.mark.parametrize("rows,cols", [("cluster", "24"), ("4", "cluster"), ("signed", "tail"), ("3", "254 edges"),
                                       ("8", "127"), ("8", "128"), ("128", "7"), ("1", "254")])
def test_two_dimensions(rows, cols):
    """1024 segments fit: 8 rows of 127 columns are the last that do."""
    print("crowded table 2d", rows, cols, flush=True)
    re = TABLES[rows] if rows in TABLES else np.linspace(0, 5, int(rows) + 1).astype(F)
    ce = TABLES[cols] if cols in TABLES else np.geomspace(20, 1000, int(cols) + 1).astype(F)
    d = np.random.default_rng(3).normal(0, 0.05, (len(re) - 1, len(ce) - 1)).astype(F)
    pt, eta = values(ce, 4), values(re, 5)
    with np.errstate(invalid="ignore"):
        same(H.jes_delta(dev(pt), dev(eta), dev(re), dev(ce), dev(d)), ref.jes_delta(pt, eta, re, ce, d))


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("cols", [1, 2, 15, 16])
@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + (1 << 19) - 1, (1 << 21) + (1 << 19)])
def test_route_limits(n, cols, dtype):
    """Shifts on either side of the sizes from which the bucket tables are taken."""
    print("bucket table limits", n, cols, dtype, flush=True)
    rng = np.random.default_rng(n + cols)
    re, ce = np.linspace(0, 5, 5).astype(F), np.geomspace(20, 1000, cols + 1).astype(F)
    d = rng.normal(0, 0.05, (4, cols)).astype(F)
    pt, eta = (rng.uniform(a, b, n).astype(np.float16 if dtype == "f16" else F) for a, b in ((0, 1100), (-6, 6)))
    same(H.jes_delta(dev(pt), dev(eta), dev(re), dev(ce), dev(d)), ref.jes_delta(pt, eta, re, ce, d))
