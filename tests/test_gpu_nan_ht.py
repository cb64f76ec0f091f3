"""A NaN H_T (jets of negative energy summing to -inf, then +inf) is not
filled, the event's other observables are: histograms equal to the oracle's."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu

EVENTS = [[-2e38, -2e38, np.inf], [-2e38, np.inf, -2e38], [-2e38, -2e38, 50.0], [np.inf], [-2e38], [np.nan, -2e38, -2e38, np.inf],
          [40.0, 50.0, 60.0], [-2e38, -2e38, 3e38, 3e38]]


def dataset(n, ext):
    rng = np.random.default_rng(2)
    ev = [EVENTS[i] for i in rng.integers(0, len(EVENTS), n)]
    ev[7] = EVENTS[0] + [30.0] * 500  # read event by event
    pt = np.concatenate(ev).astype(np.float32)

    def coll(counts, pt, extra):
        off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        z = lambda lo, hi: rng.uniform(lo, hi, off[-1]).astype(np.float32)  # noqa: E731
        cols = {"pt": pt if pt is not None else z(25, 60), "eta": z(-2, 2), "phi": z(-3, 3)}
        if extra:
            cols[extra] = z(0, 0.1) if extra == "iso" else z(0.6, 1)
        return datagen.Collection(off, cols)

    jets = coll([len(e) for e in ev], pt, "btag" if ext else None)
    el = coll(np.zeros(n, int), None, None) if ext else None
    return datagen.Dataset(n, jets, coll(rng.integers(0, 2, n), None, "iso"), np.ones(n, np.float32), el, "f32")


@pytest.mark.parametrize("hist_mode", [0, 1])
@pytest.mark.parametrize("scales", [[1.0], [1.1], [1.0, 0.9, 1.1, 3.0, 1e-3]])
@pytest.mark.parametrize("kind", ["base", "extended", "lookup"])
def test_nan_ht(kind, scales, hist_mode):
    print("nan ht", kind, scales, hist_mode, flush=True)
    ds = dataset(700, kind != "base")
    qs = []
    for cut in (-3e38, -np.inf, -1.0, 30.0):
        q = datagen.Query(jet_pt=cut, jet_abseta=5.0, dr=0.01, min_mu=0, min_jet=1, scales=np.array(scales, np.float32))
        if kind == "lookup":
            q.pu, q.sf, q.jes = datagen.pileup_table(), datagen.muon_sf_table(), datagen.jes_table()
            q.scales = q.scales - np.float32(1.0)
        qs.append(q)
    if kind == "lookup":
        ds = datagen.with_pileup(ds, 3)
    plan = H.Plan([H.DeviceDataset(ds)], qs, dict(block=512, ev_per_thread=1, hist_mode=hist_mode))
    s, c = plan.new_hists()
    plan.run(s, c)
    got = plan.split(s, c)[0]
    plan.close()
    want = ref.pipeline(ds, qs)
    skipped = 0
    for i, q in enumerate(qs):
        for v in range(q.n_scale):
            (_, n0), (_, n1) = want[i][v][0], want[i][v][1]
            skipped += int(n1.sum()) - int(n0.sum())
            for h in range(3):
                (gs, gc), (ws, wc) = got[i][v][h], want[i][v][h]
                assert np.array_equal(gc.astype(np.uint64), wc.astype(np.uint64)), f"q{i} v{v} h{h} counts"
                assert np.all(np.abs(gs - ws) <= 1e-5 * np.abs(ws)), f"q{i} v{v} h{h} sumw"
    assert skipped > 0  # (the inputs do reach a NaN H_T)
