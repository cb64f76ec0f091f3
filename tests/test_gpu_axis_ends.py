"""Values below, at, and beyond the ends of a histogram axis, and in its last
bin: the fused pass fills the oracle's slots, for cuts on either side of zero
(a negative cut lets values a rounding below an axis that starts at 0 through)."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32

AXES = {
    "183 from 0": datagen.uniform_edges(183, 0.0, 2000.0),
    "100 from 0": datagen.uniform_edges(100, 0.0, 300.0),
    "183 inside": datagen.uniform_edges(183, 200.0, 1000.0),
    "from below 0": datagen.uniform_edges(77, -50.0, 400.0),
    "one bin": np.array([0, 100], F),
    "to infinity": np.array([0, 10, 100, np.inf], F),
    "from -infinity": np.array([-np.inf, 0, 50], F),
    "uneven": np.array([0, 1e-30, 1, 90, 91, 300], F),
}


@pytest.mark.parametrize("cut", [0.0, -1.0, -100.0])
@pytest.mark.parametrize("name", list(AXES))
def test_axis_ends(name, cut):
    print("axis ends", name, cut, flush=True)
    e = AXES[name]
    ends = np.concatenate([e[:3], e[-3:]])
    x = np.concatenate([ends, np.nextafter(ends, F(np.inf)), np.nextafter(ends, F(-np.inf)), ends - F(1), ends * F(2),
                        np.array([1e-45, -1e-45, 1e-38, -1e-38, -0.0, 0.0, -0.5, 45, 1e30, 3e38, np.inf], F)])
    x = x[~np.isnan(x)]
    rng = np.random.default_rng(1)
    pt = np.concatenate([x, rng.choice(x, 900)]).astype(F)
    nj = np.concatenate([np.ones(x.size, int), np.full(300, 3)])
    n = nj.size + 50  # (and events without jets)
    nj = np.concatenate([nj, np.zeros(50, int)])
    off = np.concatenate([[0], np.cumsum(nj)]).astype(np.int64)
    z = lambda k, v: np.full(k, v, F)  # noqa: E731
    jets = datagen.Collection(off, {"pt": pt, "eta": z(off[-1], 0.0), "phi": z(off[-1], 0.0)})
    mu = datagen.Collection(np.arange(n + 1, dtype=np.int64), {"pt": z(n, 50), "eta": z(n, 1.5), "phi": z(n, 3), "iso": z(n, 0)})
    ds = datagen.Dataset(n, jets, mu, rng.normal(1, 0.1, n).astype(F), None, "f32")
    kw = dict(jet_pt=cut, min_jet=0, edges_ht=e, edges_lead=e, edges_njet=np.array([-1, 0, 1, 3], F))
    queries = [datagen.Query(**kw), datagen.Query(scales=np.array([1, 0.5, 2, 1e-3, 1e3], F), **kw)]
    for qs in ([queries[0]], queries):
        for mode in (0, 1):
            plan = H.Plan([H.DeviceDataset(ds)], qs, dict(block=512, ev_per_thread=1, hist_mode=mode))
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
