"""Performance cases: the work a user of hepk has it do, through its public
entry points, from the smallest calls to the largest.

A case is a dict of plain values.  `prepare` draws the inputs on the GPU and
makes the plan or streamer a program would keep, `run` is one pass through the
library, `work` the bytes (inputs read once, outputs written once) and
operations it cannot do without, `exact` the same outputs in float64 by plain
torch.

Kinds:
  pass         the fused analysis pass (Plan.run, run_w2 with lookup
               corrections), one dataset, one or several co-batched queries
  batch        the fused pass over many uneven datasets, one graph launch
  stream       the fused pass over a dataset in host memory (Streamer)
  chain        the same analysis as a chain of single-purpose calls (plain.run)
  positional   lepton-pair and leading-jet selection: cuts, opposite-sign
               pairs, leading element, counts with offsets, compaction
  corrections  event weights and jet-energy shifts from lookup histograms
  top          four-momenta and the jet triplet closest to the top-quark mass
"""
import math
import random

import numpy as np
import torch

from paper_1906_06242_amd import datagen, plain
from paper_1906_06242_amd import hepk as H


def listed():
    return [
        # the nominal selection over a small skim: one launch, latency
        {"name": "pass-1e5", "kind": "pass", "schema": "base", "dtype": "f32", "events": 99_991, "queries": 1},
        # the same over a sample of ordinary size (the benchmark's headline)
        {"name": "pass-1e7", "kind": "pass", "schema": "base", "dtype": "f32", "events": 10_000_000, "queries": 1},
        # eight analysts' selections served from one scan of a resident chunk
        {"name": "pass-8-queries", "kind": "pass", "schema": "base", "dtype": "f32", "events": 6_250_000,
         "queries": 8},
        # systematics: electrons, b-tag, 20 jet-energy scales, 60 histograms
        {"name": "pass-20-scales-f16", "kind": "pass", "schema": "extended", "dtype": "f16",
         "events": 20_000_003, "queries": 1},
        # the same with lookup weights, interpolated shifts and squared weights
        {"name": "pass-lookups-f16", "kind": "pass", "schema": "lookup", "dtype": "f16", "events": 10_000_019,
         "queries": 1},
        # all samples of an analysis at once: 64 datasets of 1e4 to 1e6 events
        {"name": "batch-64", "kind": "batch", "datasets": 64, "lo": 10_000, "hi": 1_000_000},
        # a cache of columns in host memory, larger than one batch
        {"name": "stream-1e7", "kind": "stream", "events": 10_000_000},
        # interactive steering, call by call, on a small skim: launches
        {"name": "chain-1e5", "kind": "chain", "schema": "base", "dtype": "f32", "events": 100_003},
        # the same call by call over a large half-precision sample
        {"name": "chain-1e7-f16", "kind": "chain", "schema": "extended", "dtype": "f16", "events": 10_000_000},
        # picking objects by position and gathering the selected ones
        {"name": "positional-5e6", "kind": "positional", "dtype": "f32", "events": 5_000_011},
        # weights and energy shifts looked up per event, muon and jet
        {"name": "corrections-1e7-f16", "kind": "corrections", "dtype": "f16", "events": 10_000_000},
        # high-level variable: all jet triplets of every event
        {"name": "top-3e6", "kind": "top", "events": 3_000_001},
    ]


# largest event count of a kind (and schema): that of the listed cases
_MOST = {"base": 10_000_000, "extended": 20_000_000, "lookup": 10_000_000, "stream": 10_000_000,
         "chain": 10_000_000, "positional": 5_000_000, "corrections": 10_000_000, "top": 3_000_000}


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng: random.Random):
    kind = rng.choice(["pass"] * 5 + ["batch", "stream"] + ["chain"] * 2 + ["positional", "corrections", "top"])
    if kind == "pass":
        schema = rng.choice(["base", "base", "extended", "lookup"])
        nq = rng.choice([1, 1, 2, 3, 5, 8]) if schema == "base" else 1
        return {"kind": kind, "schema": schema, "dtype": rng.choice(["f32", "f16"]),
                "events": _log_int(rng, 10_000, _MOST[schema] // (2 if nq > 1 else 1)), "queries": nq}
    if kind == "batch":
        hi = _log_int(rng, 50_000, 1_000_000)
        return {"kind": kind, "datasets": rng.randint(2, 64), "lo": _log_int(rng, 1000, hi // 4), "hi": hi}
    lo = 100_000 if kind == "stream" else 10_000
    case = {"kind": kind, "events": _log_int(rng, lo, _MOST[kind])}
    if kind == "chain":
        case.update(schema=rng.choice(["base", "extended"]), dtype=rng.choice(["f32", "f16"]))
    if kind in ("positional", "corrections"):
        case["dtype"] = rng.choice(["f32", "f16"])
    return case


# ---------------------------------------------------------------- inputs

def _queries(case):
    schema = case.get("schema", "base")
    if schema == "extended":
        if case["kind"] == "chain":  # the chain takes the nominal scale
            return [datagen.Query(min_b=1)]
        return [datagen.extended_query()]
    if schema == "lookup":
        return [datagen.lookup_query()]
    if case.get("queries", 1) > 1:
        return datagen.draw_queries(11, case["queries"])
    return [datagen.Query()]


def _events(case, seed):
    """Device columns of the case (a list of them for a batch)."""
    if case["kind"] == "batch":
        sizes = datagen.batch_sizes(1, case["datasets"], case["lo"], case["hi"])
        return [datagen.make_dataset_device(seed * 64 + d, int(n)) for d, n in enumerate(sizes)]
    schema = case.get("schema", "base")
    if case["kind"] == "corrections":
        schema = "lookup"
    t = datagen.make_dataset_device(seed, case["events"], extended=schema in ("extended", "lookup"),
                                    content_dtype=case.get("dtype", "f32"))
    if schema == "lookup":
        t = datagen.with_pileup_device(t, seed)
    if case["kind"] in ("positional", "corrections", "top"):
        _fix_totals(t, case["events"])
    if case["kind"] == "positional":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        t["muons.charge"] = torch.randint(0, 2, (t["muons.pt"].numel(),), generator=g, device="cuda",
                                          dtype=torch.int32) * 2 - 1
    return t


def _fix_totals(t, n):
    """Cut every collection to a number of objects that depends on the event
    count alone (five standard deviations below the mean; the last few events
    are left without objects), so per-object outputs of any seed compare."""
    for name, mean in (("jets", 5.0), ("muons", 1.5), ("electrons", 0.8)):
        if f"{name}.offsets" not in t:
            continue
        m = max(1, int(mean * n - 5 * math.sqrt(mean * n)))
        off = t[f"{name}.offsets"]
        m = min(m, int(off[-1].item()))
        t[f"{name}.offsets"] = off.clamp(max=m)
        for k in [k for k in t if k.startswith(name + ".") and not k.endswith(".offsets")]:
            t[k] = t[k][:m].clone()


def prepare(case, seed):
    kind = case["kind"]
    t = _events(case, seed)
    s = {"kind": kind}
    if kind in ("pass", "batch"):
        dds = [H.DeviceDataset.from_tensors(x) for x in (t if kind == "batch" else [t])]
        s["plan"] = H.Plan(dds, _queries(case))
        s["hists"] = s["plan"].new_hists()
        if case.get("schema") == "lookup":
            s["sumw2"] = torch.zeros_like(s["hists"][0])
    elif kind == "stream":
        ds = datagen.host_slice(t, 0, case["events"])
        s["streamer"] = H.Streamer(ds, _queries(case))
        s["hists"] = s["streamer"].new_hists()
    elif kind == "chain":
        s["data"] = H.DeviceDataset.from_tensors(t)
        s["query"] = _queries(case)[0]
    else:
        s["t"] = t
        s["query"] = datagen.lookup_query()
        if kind == "positional":
            s["kept"] = torch.zeros_like(t["jets.pt"])
        if kind == "corrections":
            s["tables"] = [torch.from_numpy(a).cuda() for a in s["query"].pu + s["query"].sf + s["query"].jes]
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind in ("pass", "batch", "stream"):
        sumw, counts = s["hists"]
        if "sumw2" in s:
            s["plan"].run_w2(sumw, s["sumw2"], counts)
            return sumw, counts, s["sumw2"]
        if kind == "pass":
            s["plan"].run(sumw, counts)
        elif kind == "batch":
            s["plan"].run_graph(sumw, counts)
        else:
            s["streamer"].run(sumw, counts)
        return sumw, counts
    if kind == "chain":
        return plain.run(s["data"], s["query"])
    t, q = s["t"], s["query"]
    if kind == "positional":
        return _positional(t, q, s["kept"])
    if kind == "corrections":
        return _corrections(t, s["tables"])
    return _top(t, q)


def _positional(t, q, kept):
    mpt, jpt, joff = t["muons.pt"], t["jets.pt"], t["jets.offsets"]
    msel = H.select([(mpt, H.GT, q.mu_pt), (t["muons.eta"], H.ABS_LT, q.mu_abseta), (t["muons.iso"], H.LT, q.mu_iso)],
                    mpt.numel())
    pair = H.select_opposite_sign(t["muons.offsets"], mpt, t["muons.charge"], obj_mask=msel)
    jsel = H.select([(jpt, H.GT, q.jet_pt), (t["jets.eta"], H.ABS_LT, q.jet_abseta)], jpt.numel())
    lead, at = H.get_in_offsets(joff, jpt, n=0, obj_mask=jsel)
    n, off = H.reduce(H.COUNT, joff, obj_mask=jsel, want_offsets=True)
    H.compact(joff, jpt, off, int(off[-1].item()), obj_mask=jsel, out=kept)
    return pair, lead, at, n, off, kept


def _corrections(t, tables):
    pu_e, pu_c, sf_e, sf_c, eta_e, pt_e, delta = tables
    pu = H.get_bin_contents(t["npu"], pu_e, pu_c)
    sf = H.get_bin_contents(t["muons.pt"], sf_e, sf_c)
    weight = H.reduce(H.PROD, t["muons.offsets"], sf)
    smooth = H.interp(t["muons.pt"], sf_e, sf_c)
    shift = H.jes_delta(t["jets.pt"], t["jets.eta"], eta_e, pt_e, delta)
    return pu, sf, weight, smooth, shift


def _top(t, q):
    jpt = t["jets.pt"]
    sel = H.select([(jpt, H.GT, q.jet_pt), (t["jets.eta"], H.ABS_LT, q.jet_abseta)], jpt.numel())
    p4 = H.p4(jpt, t["jets.eta"], t["jets.phi"], t["jets.mass"])
    mass, at = H.best_triplet(t["jets.offsets"], *p4, obj_mask=sel)
    return sel, p4, mass, at


# ---------------------------------------------------------------- work

def work(case):
    """From the mean multiplicities of the drawn events (5 jets, 1.5 muons and
    0.8 electrons each)."""
    kind = case["kind"]
    n = case.get("events", 0)
    if kind == "batch":
        n = int(datagen.batch_sizes(1, case["datasets"], case["lo"], case["hi"]).sum())
    e = 2 if case.get("dtype") == "f16" else 4
    if kind in ("pass", "batch", "stream", "chain"):
        schema = case.get("schema", "base")
        ext = schema != "base"
        per = 2 * 8 + 4 + e * (5 * 3 + 1.5 * 4) + (8 + e * (5 + 0.8 * 3) if ext else 0) + (4 if schema == "lookup" else 0)
        return {"bytes": n * per, "flops": n * 60.0 * case.get("queries", 1)}
    if kind == "positional":
        per = 8 * 2 + 1.5 * (3 * e + 4) + 5 * 2 * e  # offsets, muon and jet columns
        out = 1.5 + 4 + 4 + 4 + 8 + 3.2 * e          # pair mask, lead, index, count, offsets, kept jets
        return {"bytes": n * (per + out), "flops": n * 20.0}
    if kind == "corrections":
        per = 4 + 8 + 1.5 * e + 5 * 2 * e
        out = 4 + 1.5 * 4 + 4 + 1.5 * 4 + 5 * 4
        return {"bytes": n * (per + out), "flops": n * 100.0}
    # top: read 4 columns, write 4, the mask and 16 bytes per event
    return {"bytes": n * (8 + 5 * 32 + 5 + 16), "flops": n * (5 * 60.0 + 5.7 * 24)}


# ---------------------------------------------------------------- float64

def _rows(off):
    """The event of every object."""
    n = off.numel() - 1
    return torch.repeat_interleave(torch.arange(n, device=off.device), off[1:] - off[:-1])


def _slot(x, edges):
    """Histogram slots: 0 below the first edge, nbins + 1 from the last on."""
    e = torch.as_tensor(np.asarray(edges, np.float32), device=x.device).double()
    return torch.searchsorted(e, x.contiguous(), right=True)


def _interp64(x, edges, values):
    """Linear between bin centres, constant beyond them; values [..., nbins] by row."""
    m = 0.5 * (edges[:-1] + edges[1:])
    i = (torch.searchsorted(m, x.contiguous(), right=True) - 1).clamp(0, m.numel() - 2)
    v0, v1 = values(i), values(i + 1)
    y = v0 + (x - m[i]) * (v1 - v0) / (m[i + 1] - m[i])
    return torch.where(x <= m[0], values(torch.zeros_like(i)),
                       torch.where(x >= m[-1], values(torch.full_like(i, m.numel() - 1)), y))


def _jes64(pt, eta, jes):
    ee, pe, d = (torch.as_tensor(np.asarray(a, np.float32), device=pt.device).double() for a in jes)
    row = (torch.searchsorted(ee, eta.abs().contiguous(), right=True) - 1).clamp(0, d.shape[0] - 1)
    return _interp64(pt, pe, lambda i: d[row, i])


def _pass64(t, q, w2=False):
    """The histograms of one query: [sumw] (and [sumw2]) in slot order."""
    n = int(t["n_events"])
    f = lambda x: float(np.float32(x))  # noqa: E731
    cols = {k: v.double() for k, v in t.items() if isinstance(v, torch.Tensor) and not k.endswith(".offsets")}
    jo = t["jets.offsets"]
    ej = _rows(jo)
    hit = torch.zeros(ej.numel(), dtype=torch.bool, device=ej.device)
    nmu = None
    w = cols["weight"]
    for name in ("muons", "electrons"):
        if f"{name}.offsets" not in t:
            continue
        off, pt, eta, phi = t[f"{name}.offsets"], *(cols[f"{name}.{k}"] for k in ("pt", "eta", "phi"))
        if name == "muons":
            sel = (pt > f(q.mu_pt)) & (eta.abs() < f(q.mu_abseta)) & (cols["muons.iso"] < f(q.mu_iso))
            em = _rows(off)
            nmu = torch.bincount(em[sel], minlength=n)
            if q.pu is not None:
                w = w * torch.as_tensor(q.pu[1], device=w.device).double()[_slot(cols["npu"], q.pu[0])]
            if q.sf is not None:
                sf = torch.as_tensor(q.sf[1], device=w.device).double()[_slot(pt, q.sf[0])].log()
                w = w * torch.bincount(em[sel], weights=sf[sel], minlength=n).exp()
        else:
            sel = (pt > f(q.el_pt)) & (eta.abs() < f(q.el_abseta))
        if not pt.numel():
            continue
        lo, hi = off[ej], off[ej + 1]
        for k in range(int((off[1:] - off[:-1]).max())):
            at = (lo + k).clamp(max=pt.numel() - 1)
            dphi = (cols["jets.phi"] - phi[at]).abs()
            dphi = torch.minimum(dphi, 2 * math.pi - dphi)
            dr2 = (cols["jets.eta"] - eta[at]) ** 2 + dphi ** 2
            hit |= (lo + k < hi) & sel[at] & (dr2 <= float(np.float32(q.dr) * np.float32(q.dr)))
    ok = ~hit & (cols["jets.eta"].abs() < f(q.jet_abseta))
    ej, pt = ej[ok], t["jets.pt"].float()[ok]
    tag = (cols["jets.btag"] > f(q.btag))[ok] if "jets.btag" in t else None
    shift = _jes64(pt.double(), cols["jets.eta"][ok], q.jes) if q.jes is not None else None
    sums, sums2 = [], []
    for s in np.asarray(q.scales, np.float32):
        x = pt.double() * (1 + float(s) * shift) if shift is not None else (pt * float(s)).double()
        sel = x > f(q.jet_pt)
        es, xs = ej[sel], x[sel]
        nj = torch.bincount(es, minlength=n)
        ht = torch.bincount(es, weights=xs, minlength=n)
        lead = torch.full((n,), -math.inf, dtype=torch.float64, device=es.device)
        lead.scatter_reduce_(0, es, xs, "amax")
        good = (nmu >= q.min_mu) & (nj >= q.min_jet)
        if tag is not None:
            good &= torch.bincount(es[tag[sel]], minlength=n) >= q.min_b
        for v, e in ((ht, q.edges_ht), (lead, q.edges_lead), (nj.double(), q.edges_njet)):
            at = _slot(v[good], e)
            sums.append(torch.bincount(at, weights=w[good], minlength=len(e) + 1))
            sums2.append(torch.bincount(at, weights=w[good] ** 2, minlength=len(e) + 1))
    return sums, (sums2 if w2 else None)


def exact(case, seed):
    kind = case["kind"]
    t = _events(case, seed)
    if kind in ("pass", "batch", "stream", "chain"):
        qs = _queries(case)
        if kind == "chain":
            return [(v, None) for v in _pass64(t, qs[0])[0]]
        sums, sums2 = [], []
        for d in (t if kind == "batch" else [t]):
            for q in qs:
                a, b = _pass64(d, q, w2=case.get("schema") == "lookup")
                sums += a
                sums2 += b or []
        return (torch.cat(sums), None) + ((torch.cat(sums2),) if sums2 else ())
    q = datagen.lookup_query()
    f = lambda k: t[k].double()  # noqa: E731
    if kind == "top":
        pt, eta, phi, m = (f(f"jets.{k}") for k in ("pt", "eta", "phi", "mass"))
        p = (pt * phi.cos(), pt * phi.sin(), pt * eta.sinh())
        return None, p + ((p[0] ** 2 + p[1] ** 2 + p[2] ** 2 + m ** 2).sqrt(),), None, None
    if kind == "positional":
        sel = (f("jets.pt") > q.jet_pt) & (f("jets.eta").abs() < q.jet_abseta)
        es, kept = _rows(t["jets.offsets"])[sel], f("jets.pt")[sel]
        n = torch.bincount(es, minlength=case["events"])
        first = torch.cumsum(n, 0) - n
        lead = torch.where(n > 0, kept[first.clamp(max=max(0, kept.numel() - 1))], torch.zeros((), device=n.device).double())
        return None, lead, None, None, None, torch.nn.functional.pad(kept, (0, sel.numel() - kept.numel()))
    con = lambda x, tab: torch.as_tensor(tab[1], device=x.device).double()[_slot(x, tab[0])]  # noqa: E731
    mpt = f("muons.pt")
    sf = con(mpt, q.sf)
    em = _rows(t["muons.offsets"])
    weight = torch.bincount(em, weights=sf.log(), minlength=case["events"]).exp()
    se, sc = (torch.as_tensor(a, device=mpt.device).double() for a in q.sf)
    return (con(f("npu"), q.pu), sf, weight, _interp64(mpt, se, lambda i: sc[i + 1]),
            _jes64(f("jets.pt"), f("jets.eta"), q.jes))
