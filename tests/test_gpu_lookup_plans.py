"""Plans of one to five lookup queries, with shift tables from one value to more
than LDS takes: whichever of the tables and their segments go to LDS, the
histograms are the oracle's."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32


def table(rows, cols):
    rng = np.random.default_rng(rows * 1000 + cols)
    return (np.linspace(0, 4.7, rows + 1).astype(F), np.geomspace(20, 1000, cols + 1).astype(F),
            rng.normal(0.0, 0.03, (rows, cols)).astype(F))


def query(i, shape, bins, shifts):
    q = datagen.lookup_query(min_b=0)
    q.mu_pt, q.min_jet = 20.0 + i, 2
    q.scales = q.scales[:shifts]
    q.jes = table(*shape)
    q.edges_ht, q.edges_lead = datagen.uniform_edges(bins, 0.0, 1500.0), datagen.uniform_edges(bins, 0.0, 500.0)
    if i % 3 == 2:
        q.pu = None
    return q


CASES = {
    "one small": ([(1, 1)], 50, 20),
    "segments in budget": ([(7, 24), (2, 5)], 40, 1),
    "second without": ([(7, 24), (7, 24)], 40, 1),
    "budget used by tables": ([(7, 24)] * 4, 40, 1),
    "tables beyond LDS": ([(7, 24)] * 5, 60, 1),
    "large table": ([(20, 80), (3, 7)], 40, 2),
    "histograms short of LDS": ([(7, 24)], 165, 20),
    "histograms beyond LDS": ([(7, 24)], 240, 20),
    "both": ([(7, 24), (7, 24)], 85, 20),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lookup_plans(name):
    import torch
    print("lookup plans", name, flush=True)
    shapes, bins, shifts = CASES[name]
    ds = datagen.with_pileup(datagen.make_dataset(3, 4000, extended=True, content_dtype="f16"), 3)
    qs = [query(i, s, bins, shifts) for i, s in enumerate(shapes)]
    plan = H.Plan([H.DeviceDataset(ds)], qs)
    s, c = plan.new_hists()
    s2 = torch.zeros_like(s)
    plan.run_w2(s, s2, c)
    got = plan.split(s, c)[0]
    plan.close()
    want = ref.pipeline(ds, qs)
    for i, q in enumerate(qs):
        for v in range(q.n_scale):
            for h in range(3):
                (gs, gc), (ws, wc) = got[i][v][h], want[i][v][h]
                assert np.array_equal(gc.astype(np.uint64), wc.astype(np.uint64)), f"q{i} v{v} h{h}"
                assert np.all(np.abs(gs - ws) <= 1e-5 * np.abs(ws)), f"q{i} v{v} h{h} sumw"
