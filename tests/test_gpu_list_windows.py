"""Tiles that list more candidates than the dense list holds, with the events'
jets spread so that the passes end at every kind of place: after the first
event, at the last, at an event that fills the list exactly, before runs of
events without candidates.  Histograms and every event's record as the oracle
has them."""
import numpy as np
import pytest
import test_gpu_records as records

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32

# jets of the events of a tile, repeated
PATTERNS = {
    "even": [7] * 64,
    "first fills": [128] + [5] * 63,
    "last fills": [5] * 63 + [128],
    "192 and gaps": [192, 0, 0, 64, 0, 192] + [0] * 58,
    "128 + 64": ([64, 64, 64] + [0] * 13) * 2 + [0] * 32,
    "ones": [1] * 64,
    "long after empty": [0] * 62 + [127, 128],
}


def events(name, ext, dtype, seed):
    rng = np.random.default_rng(seed)
    counts = np.array(PATTERNS[name] * 9 + [3, 130, 7], int)
    n = counts.size
    dt = np.float16 if dtype == "f16" else F

    def coll(c, extra, lo):
        off = np.concatenate([[0], np.cumsum(c)]).astype(np.int64)
        m = off[-1]
        cols = {"pt": lo + rng.exponential(40.0, m), "eta": rng.uniform(-2.6, 2.6, m), "phi": rng.uniform(-3.1, 3.1, m)}
        if extra:
            cols[extra] = rng.uniform(0.0, 0.16, m) if extra == "iso" else rng.uniform(0.4, 1.0, m)
        return datagen.Collection(off, {k: v.astype(dt) for k, v in cols.items()})

    return datagen.Dataset(n, coll(counts, "btag" if ext else None, 29.0), coll(rng.integers(0, 3, n), "iso", 19.0),
                           rng.normal(1, 0.1, n).astype(F), coll(rng.integers(0, 2, n), None, 19.0) if ext else None, dtype)


@pytest.mark.parametrize("shape", [None, dict(block=512, ev_per_thread=2, hist_mode=0)])
@pytest.mark.parametrize("ext,dtype", [(False, "f32"), (True, "f32"), (True, "f16")])
@pytest.mark.parametrize("name", list(PATTERNS))
def test_windows(name, ext, dtype, shape):
    print("list windows", name, ext, dtype, shape, flush=True)
    ds = events(name, ext, dtype, 3)
    loose = dict(jet_pt=10.0, jet_abseta=5.0, min_mu=0, min_jet=0, dr=0.2)
    nominal = dict(min_mu=1, min_jet=2)
    for qs in ([datagen.Query(**loose), datagen.Query(**nominal)],
               [datagen.Query(scales=datagen.jes_scales(), **loose), datagen.Query(scales=datagen.jes_scales(), **nominal)]):
        plan = H.Plan([H.DeviceDataset(ds)], qs, shape)
        s, c = plan.new_hists()
        plan.run(s, c)
        got = plan.split(s, c)[0]
        plan.close()
        want = ref.pipeline(ds, qs)
        for i, q in enumerate(qs):
            for v in range(q.n_scale):
                for h in range(3):
                    (gs, gc), (ws, wc) = got[i][v][h], want[i][v][h]
                    assert np.array_equal(gc.astype(np.uint64), wc.astype(np.uint64)), f"q{i} v{v} h{h}"
                    assert np.all(np.abs(gs - ws) <= 1e-5 * np.abs(ws)), f"q{i} v{v} h{h} sumw"
        records.check_records(ds, qs, shape, name)
