"""Lookups through bucket tables, bit for bit against the oracle: inputs long
enough for that path, tables that spread well on a linear key (uniform), on
the float's bits (logarithmic), on neither, and at the size limits."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
N = (1 << 21) + 5


def edges_of(name):
    rng = np.random.default_rng(4)
    f = np.float32
    if name == "uniform":
        return np.linspace(0, 80, 81).astype(f)
    if name == "log":
        return np.geomspace(20, 1000, 25).astype(f)
    if name == "from zero":
        return np.array([0, 0.5, 1, 1.5, 2, 2.5, 3, 5], f)
    if name == "minus zero":
        return np.array([-0.0, 1e-30, 1, 7, 100], f)
    if name == "signed":
        return np.sort(rng.uniform(-5, 5, 40)).astype(f)
    if name == "crowded":  # 30 edges in one bucket of either key
        return np.concatenate([[-1e6], 1 + np.arange(30) * 1e-4, [1e6]]).astype(f)
    if name == "neighbours":  # centres of adjacent floats coincide
        e = [f(1)]
        for _ in range(6):
            e.append(np.nextafter(e[-1], f(2)))
        return np.array(e + [2, 3], f)
    if name == "one bin":
        return np.array([25, 40], f)
    k = int(name)
    return np.unique(rng.lognormal(3, 1, 4 * k).astype(f))[:k + 1]


def values(edges, dtype):
    rng = np.random.default_rng(5)
    f = np.float32
    c = ((edges[:-1] + edges[1:]) * f(0.5)).astype(f)
    near = np.concatenate([edges, c])
    s = np.concatenate([near, np.nextafter(near, f(np.inf)), np.nextafter(near, f(-np.inf)),
                        np.array([0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45, 3e38, -3e38], f)])
    span = float(edges[-1]) - float(edges[0])
    body = rng.uniform(float(edges[0]) - 0.1 * span, float(edges[-1]) + 0.1 * span, N - s.size).astype(f)
    x = np.concatenate([s, body])
    rng.shuffle(x)
    with np.errstate(over="ignore"):
        return x.astype(np.float16 if dtype == "f16" else f)


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def same(got, want, what):
    got = got.cpu().numpy()
    ok = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
    assert np.all(ok), f"{what}: {np.count_nonzero(~ok)} differ, first {got[~ok][0]!r} vs {want[~ok][0]!r}"


NAMES = ["uniform", "log", "from zero", "minus zero", "signed", "crowded", "neighbours", "one bin", "253", "254", "255"]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("name", NAMES)
def test_bucket_tables(name, dtype):
    print("bucket tables", name, dtype, flush=True)
    e = edges_of(name)
    c = np.random.default_rng(6).normal(1, 0.3, len(e) + 1).astype(np.float32)
    c[1], c[-2] = -0.0, 0.0
    x = values(e, dtype)
    with np.errstate(invalid="ignore"):
        same(H.get_bin_contents(dev(x), dev(e), dev(c)), ref.get_bin_contents(x, e, c), "contents")
        same(H.interp(dev(x), dev(e), dev(c)), ref.interp(x, e, c), "interpolation")
        y = dev(np.concatenate([x[:1], x]))[1:]  # not aligned to four elements
        same(H.interp(y, dev(e), dev(c)), ref.interp(x, e, c), "unaligned")


@pytest.mark.parametrize("rows", ["from zero", "signed", "one bin", "crowded"])
@pytest.mark.parametrize("cols", ["log", "uniform", "crowded", "one bin", "253"])
def test_bucket_tables_2d(rows, cols):
    print("bucket tables 2d", rows, cols, flush=True)
    re, ce = edges_of(rows), edges_of(cols)
    d = np.random.default_rng(8).normal(0, 0.05, (len(re) - 1, len(ce) - 1)).astype(np.float32)
    for dtype in ("f32", "f16"):
        pt, eta = values(ce, dtype), values(re, dtype)
        same(H.jes_delta(dev(pt), dev(eta), dev(re), dev(ce), dev(d)), ref.jes_delta(pt, eta, re, ce, d), dtype)
