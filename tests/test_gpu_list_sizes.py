"""The candidate list takes the LDS that the histograms and tables leave: from
all of a tile's jets beside small histograms down to its least size beside
large ones.  Tiles that fit, just fit, do not fit and hold single events beyond
the list must give the oracle's histograms at every size, also when a query set
later changes the size between launches and graph launches of one plan."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import datagen
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu
F = np.float32


def events(ext, dtype):
    rng = np.random.default_rng(5)
    tile = {0: [7] * 64, 1: [448] + [0] * 63, 2: [2] * 30 + [385] + [1] * 33, 3: [193, 192, 63] + [0] * 61,
            4: [256, 192] + [0] * 62, 5: [129, 128, 127, 64] + [0] * 60, 6: [5] * 64}
    counts = np.concatenate([tile[i % 7] for i in range(21)] + [[3, 200, 0, 700, 2]]).astype(int)
    n = counts.size
    dt = np.float16 if dtype == "f16" else F

    def coll(c, extra):
        off = np.concatenate([[0], np.cumsum(c)]).astype(np.int64)
        m = off[-1]
        cols = {"pt": 25 + rng.exponential(40.0, m), "eta": rng.uniform(-2.4, 2.4, m), "phi": rng.uniform(-3.1, 3.1, m)}
        if extra:
            cols[extra] = rng.uniform(0.0, 0.16, m) if extra == "iso" else rng.uniform(0.4, 1.0, m)
        return datagen.Collection(off, {k: v.astype(dt) for k, v in cols.items()})

    return datagen.Dataset(n, coll(counts, "btag" if ext else None), coll(rng.integers(0, 3, n), "iso"),
                           rng.normal(1, 0.1, n).astype(F), coll(rng.integers(0, 2, n), None) if ext else None, dtype)


def query(bins, scales=None, **kw):
    q = datagen.Query(min_mu=0, min_jet=0, dr=0.1, edges_ht=datagen.uniform_edges(bins, 0.0, 4000.0), **kw)
    if scales is not None:
        q.scales = scales
    return q


def check(plan, hists, ds, queries, runs=1):
    got = plan.split(*hists)[0]
    want = ref.pipeline(ds, [q for q in queries if q is not None])
    k = 0
    for i, q in enumerate(queries):
        if q is None:
            continue
        for v in range(q.n_scale):
            for h in range(3):
                (gs, gc), (ws, wc) = got[i][v][h], want[k][v][h]
                assert np.array_equal(gc.astype(np.uint64), runs * wc.astype(np.uint64)), f"q{i} v{v} h{h}"
                assert np.all(np.abs(gs - runs * ws) <= 1e-5 * np.abs(runs * ws)), f"q{i} v{v} h{h} sumw"
        k += 1


@pytest.mark.parametrize("shape", [(512, 1), (512, 2), (256, 1), (1024, 1)])
@pytest.mark.parametrize("ext,dtype", [(False, "f32"), (True, "f32"), (True, "f16")])
@pytest.mark.parametrize("bins", [50, 2500, 5000, 7000, 8000, 9500, 11500])
def test_list_sizes(bins, ext, dtype, shape):
    print("list sizes", bins, ext, dtype, shape, flush=True)
    ds = events(ext, dtype)
    tune = dict(block=shape[0], ev_per_thread=shape[1], hist_mode=0)
    for q in (query(bins), query(bins // 3, np.array([0.9, 1.0, 1.1], F))):
        plan = H.Plan([H.DeviceDataset(ds)], [q], tune)
        hists = plan.new_hists()
        plan.run(*hists)
        check(plan, hists, ds, [q])
        plan.close()


@pytest.mark.parametrize("ext,dtype", [(False, "f32"), (True, "f16")])
def test_list_size_changes(ext, dtype):
    print("list size changes", ext, dtype, flush=True)
    ds = events(ext, dtype)
    plan = H.Plan([H.DeviceDataset(ds)], [query(60), query(60)], reserve_bins=9000)
    for bins in (9000, 60, 4000, 11, 8999, 60):
        plan.set_query(1, query(bins, jet_pt=20.0))
        for run in (plan.run, plan.run_graph, plan.run_graph):
            hists = plan.new_hists()
            run(*hists)
            check(plan, hists, ds, [query(60), query(bins, jet_pt=20.0)])
    plan.set_query(0, None)
    hists = plan.new_hists()
    plan.run_graph(*hists)
    check(plan, hists, ds, [None, query(60, jet_pt=20.0)])
    plan.close()


@pytest.mark.parametrize("bins", [30, 100, 160, 175, 190])
def test_list_sizes_lookups(bins):
    print("list sizes, lookups", bins, flush=True)
    ds = datagen.with_pileup(events(True, "f16"), 4)
    q = datagen.lookup_query(min_b=0)
    q.min_mu = q.min_jet = 0
    q.edges_ht, q.edges_lead = datagen.uniform_edges(bins, 0.0, 4000.0), datagen.uniform_edges(bins, 0.0, 1000.0)
    plan = H.Plan([H.DeviceDataset(ds)], [q])
    s, c = plan.new_hists()
    import torch
    plan.run_w2(s, torch.zeros_like(s), c)
    check(plan, (s, c), ds, [q])
    plan.close()
