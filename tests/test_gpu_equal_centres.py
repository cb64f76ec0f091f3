"""Interpolation where the first bin centres round to the same float32: up to
the first centre the value is the first one, on every path, bit for bit the
oracle's."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32


def edges(name):
    if name == "integers":  # centres 1 and 2 are both 16777220
        return np.array([16777218, 16777220, 16777222, 16777224, 16777240, 33554432], F)
    e = [np.nextafter(F(1), F(2))]
    for _ in range(5):
        e.append(np.nextafter(e[-1], F(2)))
    return np.array(e + [3, 4], F)


def same(got, want):
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("name", ["integers", "after one"])
@pytest.mark.parametrize("n", [1000, (1 << 21) + 1])
def test_interpolation(name, n):
    import torch
    print("equal centres", name, n, flush=True)
    e = edges(name)
    m = ((e[:-1] + e[1:]) * F(0.5)).astype(F)
    assert m[0] == m[1]
    near = np.concatenate([e, m])
    near = np.concatenate([near, np.nextafter(near, F(np.inf)), np.nextafter(near, F(-np.inf))])
    rng = np.random.default_rng(3)
    x, eta = rng.choice(near, n), rng.uniform(-5, 5, n).astype(F)
    c = np.arange(len(e) + 1).astype(F)
    rows = np.array([0, 1, 2, 5], F)
    d = rng.normal(0, 1, (3, len(e) - 1)).astype(F)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    same(H.interp(dev(x), dev(e), dev(c)), ref.interp(x, e, c))
    same(H.jes_delta(dev(x), dev(eta), dev(rows), dev(e), dev(d)), ref.jes_delta(x, eta, rows, e, d))


def test_fused_pass():
    """Jets at the first centres of the shift table: ordinary events and one
    read object by object take the same shift, so H_T falls into the oracle's
    bins."""
    print("equal centres, fused pass", flush=True)
    e = edges("integers")
    rng = np.random.default_rng(4)
    n = 640
    nj = rng.poisson(4.0, n)
    nj[100] = 600
    off = np.concatenate([[0], np.cumsum(nj)]).astype(np.int64)
    moff = np.arange(n + 1, dtype=np.int64)
    z = lambda k, a, b: rng.uniform(a, b, k).astype(F)  # noqa: E731
    jets = datagen.Collection(off, {"pt": rng.choice(e[:4], off[-1]), "eta": z(off[-1], -2, 2), "phi": z(off[-1], -3, 3)})
    mu = datagen.Collection(moff, {"pt": z(n, 25, 60), "eta": z(n, -2, 2), "phi": z(n, -3, 3), "iso": z(n, 0, 0.1)})
    ds = datagen.Dataset(n, jets, mu, np.ones(n, F), None, "f32")
    table = (np.array([0, 5], F), e, np.array([[0.0, 1.0, 2.0, 3.0, 4.0]], F))
    for shifts in ([1.0], [0.5, 1.0, 1.5]):
        q = datagen.Query(jet_pt=1e6, min_jet=1, jes=table, scales=np.array(shifts, F),
                          edges_lead=np.array([0, 1.7e7, 2.5e7, 4e7, 1e8], F), edges_ht=np.geomspace(1e7, 1e11, 200).astype(F))
        plan = H.Plan([H.DeviceDataset(ds)], [q])
        s, c = plan.new_hists()
        plan.run(s, c)
        got = plan.split(s, c)[0]
        plan.close()
        want = ref.pipeline(ds, [q])
        for v in range(len(shifts)):
            for h in range(3):
                assert np.array_equal(got[0][v][h][1].astype(np.uint64), want[0][v][h][1].astype(np.uint64)), f"v{v} h{h}"
                assert np.array_equal(got[0][v][h][0], want[0][v][h][0])
