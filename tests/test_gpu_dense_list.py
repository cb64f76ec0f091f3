"""The fused pass at the edges of its dense candidate list.

The candidates (jets that can be selected at some energy scale) of the events
that can still pass are listed in LDS, a bounded number per pass over a tile.
Datasets that fill a tile's registers exactly, exceed the list several times
over, hold events at and beyond its bound, and jets at the exact pt thresholds
must give the oracle's histograms: counts equal, weight sums within 1e-5 per
bin (the float64 sums of float32 weights are exact but for their order).
"""
import sys

import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
RTOL = 1e-5


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    H.load()
    yield
    torch.cuda.synchronize()


def build(seed, jets, muons, ext, dtype):
    """Events of the given jet and muon counts, nearly every object passing
    its kinematic cuts, the muons far from most jets."""
    rng = np.random.default_rng(seed)
    n = len(jets)
    dt = np.float16 if dtype == "f16" else np.float32

    def coll(counts, names, lo):
        off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        m = int(off[-1])
        cols = {"pt": lo + rng.exponential(40.0, m), "eta": rng.uniform(-2.6, 2.6, m),
                "phi": rng.uniform(-np.pi, np.pi, m)}
        for k in names:
            cols[k] = rng.uniform(0.0, 0.16, m) if k == "iso" else rng.uniform(0.3, 1.0, m)
        return datagen.Collection(off, {k: v.astype(dt) for k, v in cols.items()})

    j = coll(jets, ["btag"] if ext else [], 29.0)
    mu = coll(muons, ["iso"], 19.0)
    el = coll(rng.poisson(0.8, n), [], 19.0) if ext else None
    w = rng.normal(1.0, 0.1, n).astype(np.float32)
    return datagen.Dataset(n, j, mu, w, el, dtype)


def shapes(name, n=1500):
    rng = np.random.default_rng(3)
    jets, muons = rng.poisson(5.0, n), rng.poisson(1.5, n)
    if name == "full tiles":      # 448 jets and 128 muons in every 64 events
        jets[:], muons[:] = 7, 2
    elif name == "one beyond":    # 449 jets: every tile in two
        jets[:], muons[:] = 7, 2
        jets[::64] = 8
    elif name == "long events":   # at and beyond the list's bound of one event
        for i, k in enumerate((127, 128, 129, 191, 192, 193, 447, 448, 449, 1000)):
            jets[100 * i + 50], muons[100 * i + 50] = k, 2 + i
    elif name == "few":           # tiles without any event that can pass
        muons[64:1200] = 0
    return jets, muons


def check(ds, queries, tune=None):
    plan = H.Plan([H.DeviceDataset(ds)], queries, tune)
    s, c = plan.new_hists()
    plan.run(s, c)
    got = plan.split(s, c)[0]
    plan.close()
    want = ref.pipeline(ds, queries)
    for qi, q in enumerate(queries):
        for v in range(q.n_scale):
            for h in range(3):
                (gs, gc), (ws, wc) = got[qi][v][h], want[qi][v][h]
                assert np.array_equal(gc.astype(np.uint64), wc.astype(np.uint64)), f"q{qi} v{v} h{h} counts"
                assert np.all(np.abs(gs - ws) <= RTOL * np.abs(ws)), f"q{qi} v{v} h{h} sumw"


@pytest.mark.parametrize("tune", [None, dict(block=512, ev_per_thread=2, hist_mode=0),
                                  dict(block=256, ev_per_thread=1, hist_mode=1)])
@pytest.mark.parametrize("ext,dtype", [(False, "f32"), (False, "f16"), (True, "f32"), (True, "f16")])
@pytest.mark.parametrize("shape", ["full tiles", "one beyond", "long events", "few"])
def test_dense_list(shape, ext, dtype, tune):
    print("dense list", shape, ext, dtype, tune, flush=True)
    sys.stdout.flush()
    ds = build(5, *shapes(shape), ext, dtype)
    b = 1 if ext else 0
    loose = datagen.Query(min_jet=0, min_mu=0, min_b=b)
    negative = datagen.Query(jet_pt=-1.0, min_jet=2, min_b=b)  # every jet inside |eta| is a candidate
    check(ds, [datagen.Query(min_b=b), loose, negative], tune)
    check(ds, [datagen.Query(min_b=b, scales=datagen.jes_scales())], tune)


@pytest.mark.parametrize("shape", ["full tiles", "long events"])
@pytest.mark.parametrize("table", ["as drawn", "steep", "negative factor", "not finite"])
def test_dense_list_shifts(shape, table):
    """Shifted energies: the candidate bound must hold for any table."""
    print("dense list shifts", shape, table, flush=True)
    ds = datagen.with_pileup(build(6, *shapes(shape), True, "f16"), 6)
    q = datagen.lookup_query()
    e, p, d = (np.array(a, np.float32) for a in q.jes)
    if table == "steep":
        d = d * np.float32(8.0) * np.where(np.arange(d.size).reshape(d.shape) % 2, 1, -1).astype(np.float32) / 8
    elif table == "negative factor":
        d = d - np.float32(0.9)
    elif table == "not finite":
        d = d.copy()
        d[1, 3] = np.inf
        d[2, 5] = np.nan
    q.jes = (e, p, d)
    check(ds, [q])


@pytest.mark.parametrize("scale", [1.0, 0.93, 1.1, 1e-30, 3e30])
@pytest.mark.parametrize("cut", [0.0, 30.0, 1e-40, np.float32(3.4e38), np.inf])
def test_pt_thresholds(scale, cut):
    """Jets at, just below and just above the smallest pt that passes."""
    print("pt thresholds", scale, cut, flush=True)
    s, c = np.float32(scale), np.float32(cut)
    with np.errstate(over="ignore", invalid="ignore"):
        t = np.float32(np.float64(c) / np.float64(s))
    near = [t]
    for _ in range(3):
        near = [np.nextafter(near[0], np.float32(-np.inf))] + near + [np.nextafter(near[-1], np.float32(np.inf))]
    pts = np.array(near + [0.0, -0.0, -30.0, 1e-45, np.inf, -np.inf, np.nan], np.float32)
    n = 256
    ds = build(7, np.full(n, 5), np.full(n, 1), False, "f32")
    rng = np.random.default_rng(1)
    ds.jets.cols["pt"][:] = rng.choice(pts, ds.jets.cols["pt"].size)
    check(ds, [datagen.Query(jet_pt=float(c), min_jet=1, min_mu=0, scales=np.array([s], np.float32))])
    check(ds, [datagen.Query(jet_pt=float(c), min_jet=1, min_mu=0, scales=np.array([s, s * np.float32(0.5)], np.float32))])
