"""Tiles with more muons than the registers hold: the rest of the last slot is
read from memory.  128 muons of 64 events (256 of 128) are held, 192 (320) in
all; tiles at and around both, with every mix of selected ones, give the oracle's
histograms and records."""
import numpy as np
import pytest
import test_gpu_records as records

from paper_1906_06242_amd import datagen

pytestmark = pytest.mark.gpu
F = np.float32

MUONS = {"128": [2] * 64, "129": [2] * 63 + [3], "129 first": [66] + [1] * 63, "191": [3] * 63 + [2], "192": [3] * 64,
         "193": [3] * 63 + [4], "one event": [192] + [0] * 63, "last event": [0] * 63 + [150], "256": [4] * 64, "5": [5] * 64}


def events(name, ext, dtype, iso):
    rng = np.random.default_rng(8)
    nm = np.array(MUONS[name] * 7 + [2, 0, 9], int)
    n = nm.size
    dt = np.float16 if dtype == "f16" else F

    def coll(c, extra, lo):
        off = np.concatenate([[0], np.cumsum(c)]).astype(np.int64)
        m = off[-1]
        cols = {"pt": lo + rng.exponential(20.0, m), "eta": rng.normal(0, 1.5, m), "phi": rng.uniform(-3.1, 3.1, m)}
        if extra:
            cols[extra] = rng.exponential(0.1, m) if extra == "iso" else rng.uniform(0.3, 1.0, m)
        return datagen.Collection(off, {k: v.astype(dt) for k, v in cols.items()})

    return datagen.Dataset(n, coll(rng.poisson(4.0, n), "btag" if ext else None, 25.0), coll(nm, "iso" if iso else None, 15.0),
                           rng.normal(1, 0.1, n).astype(F), coll(rng.poisson(0.8, n), None, 15.0) if ext else None, dtype)


@pytest.mark.parametrize("shape", [None, dict(block=512, ev_per_thread=2, hist_mode=0)])
@pytest.mark.parametrize("ext,dtype,iso", [(False, "f32", True), (False, "f16", False), (True, "f32", True), (True, "f16", True)])
@pytest.mark.parametrize("name", list(MUONS))
def test_muon_slots(name, ext, dtype, iso, shape):
    print("muon slots", name, ext, dtype, iso, shape, flush=True)
    ds = events(name, ext, dtype, iso)
    qs = [datagen.Query(min_jet=1, dr=0.6), datagen.Query(mu_pt=30.0, min_mu=2, min_jet=0, jet_pt=-1.0)]
    records.check_records(ds, qs, shape, name)
    records.check_records(ds, [datagen.Query(min_jet=1, dr=0.6, scales=datagen.jes_scales())], shape, name + " scales")


@pytest.mark.parametrize("name", ["129", "192", "193", "5"])
def test_muon_slots_lookups(name):
    print("muon slots, lookups", name, flush=True)
    ds = datagen.with_pileup(events(name, True, "f16", True), 2)
    records.check_records(ds, [datagen.lookup_query(min_b=0)], None, name)
