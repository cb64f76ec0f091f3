"""Events of hundreds of jets among ordinary ones: each is taken alone (or, with
few enough candidates, in its tile), with more than 64 muons or scales too;
histograms and every event's record as the oracle has them."""
import numpy as np
import pytest
import test_gpu_records as records

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32


def events(where, ext, dtype, lo):
    """1300 ordinary events; `where`: a long one at these places of each tile."""
    rng = np.random.default_rng(7)
    n = 1300
    jets, muons = rng.poisson(4.0, n), rng.poisson(1.5, n)
    for t in range(n // 64):
        for k in where:
            jets[64 * t + k] = (130, 200, 300, 448, 449, 700)[(t + k) % 6]
            muons[64 * t + k] = (0, 1, 3, 63, 65, 140)[(t + 2 * k) % 6]
    dt = np.float16 if dtype == "f16" else F

    def coll(c, extra, a):
        off = np.concatenate([[0], np.cumsum(c)]).astype(np.int64)
        m = off[-1]
        cols = {"pt": a + rng.exponential(40.0, m), "eta": rng.normal(0, 1.5, m), "phi": rng.uniform(-3.1, 3.1, m)}
        if extra:
            cols[extra] = rng.exponential(0.1, m) if extra == "iso" else rng.uniform(0, 1.0, m)
        return datagen.Collection(off, {k: v.astype(dt) for k, v in cols.items()})

    el = rng.poisson(0.8, n)
    el[where[0]::256] = 90
    return datagen.Dataset(n, coll(jets, "btag" if ext else None, lo), coll(muons, "iso", 19.0),
                           rng.normal(1, 0.1, n).astype(F), coll(el, None, 19.0) if ext else None, dtype)


@pytest.mark.parametrize("shape", [None, dict(block=256, ev_per_thread=2, hist_mode=0)])
@pytest.mark.parametrize("ext,dtype", [(False, "f32"), (True, "f16")])
@pytest.mark.parametrize("where", [(0,), (63,), (0, 1, 2), (5, 31, 32, 62)])
@pytest.mark.parametrize("lo", [5.0, 40.0])  # few of a long event's jets are candidates, or most
def test_long_events(where, ext, dtype, shape, lo):
    print("long events", where, ext, dtype, shape, lo, flush=True)
    ds = events(where, ext, dtype, lo)
    many = np.concatenate([datagen.jes_scales(), np.linspace(0.5, 2.0, 50).astype(F)])
    qs = [datagen.Query(min_jet=2), datagen.Query(jet_pt=-1.0, min_mu=0, min_jet=0), datagen.Query(dr=0.05, mu_pt=30.0)]
    records.check_records(ds, qs, shape, "one scale")
    records.check_records(ds, [datagen.Query(min_jet=2, scales=many), datagen.Query(jet_pt=60.0, scales=many[:3])], shape, "70 scales")


@pytest.mark.parametrize("where", [(0,), (5, 31, 32, 62)])
def test_long_events_lookups(where):
    print("long events, lookups", where, flush=True)
    ds = datagen.with_pileup(events(where, True, "f16", 25.0), 3)
    q = datagen.lookup_query(min_b=0)
    records.check_records(ds, [q], None, "lookups")
    plan = H.Plan([H.DeviceDataset(ds)], [q])
    s, c = plan.new_hists()
    plan.run(s, c)
    got = plan.split(s, c)[0][0]
    plan.close()
    want = ref.pipeline(ds, [q])[0]
    for v in range(q.n_scale):
        for h in range(3):
            assert np.array_equal(got[v][h][1].astype(np.uint64), want[v][h][1].astype(np.uint64)), f"v{v} h{h}"
            assert np.all(np.abs(got[v][h][0] - want[v][h][0]) <= 1e-5 * np.abs(want[v][h][0]))
