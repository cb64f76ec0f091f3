// The fused analysis kernel of hepk_pipeline and its launch-shape table,
// shared by the translation units that instantiate it.
//
// The whole analysis pass of Sec. IV (object selection,
// lepton-jet Delta-R cleaning, per-event reductions, event selection,
// weighted histograms, jet-energy-scale variations) fused into one
// persistent kernel, for any number of datasets and queries at once.
//
// Sec. IV observes that hundreds of small kernel calls per pass left the GPU
// half idle and names fusion as the fix; here every intermediate (object
// masks, per-event counts and sums, event masks) lives in registers and LDS,
// so a pass reads each input column from HBM once and writes only the
// histograms.
//
// Work decomposition.  Each wavefront owns tiles of TW = 64 * EVPL
// consecutive events and works through them without waiting for the other
// wavefronts of its workgroup (no workgroup barrier inside a tile: the up to
// sixteen wavefronts of a workgroup only share the LDS histograms, updated
// with atomics).  A launch covers whole datasets (one chunk each); every
// workgroup takes an equal slice of their concatenated tiles, so uneven
// datasets never unbalance the launch, and merges its LDS histograms into
// HBM when its slice leaves a dataset.  For one tile a wavefront
//   1. reads the tile's object ranges with scalar loads (one tile ahead),
//      then issues all of its loads at once -- offsets (their low 32-bit
//      words) and weight of its events, up to JK jets, MK muons and EK
//      electrons per lane (consecutive lanes, consecutive objects:
//      coalesced) -- into registers, and waits once;
//   2. per query: muon (and electron) lanes evaluate the cuts; the selected
//      leptons are compacted by wavefront ballot into LDS in tile order,
//      with the count of selected leptons before each lepton (muons beyond
//      the MK per lane, up to one more each, are read from memory here);
//   3. jet lanes mark the candidate jets (inside |eta|, pt above jet_pt at the
//      largest energy any scale gives it) and write the number of candidates
//      (and b-tagged candidates) before each jet; event lanes read both ends
//      of their ranges and keep the events that can still pass: enough
//      selected muons, candidates and b-tagged candidates (cuts only remove
//      jets, so no other event can);
//   4. the candidates of those events alone are compacted into LDS, and the
//      cone test runs over that dense list, a lane per candidate: most jets
//      of a tile never reach it (base selection: 86 of 320, with a b-tag 47).
//      The list's length is the launch's (list_fit); a tile with more
//      candidates runs steps 4 and 5 in several passes over its events, each
//      as many as fit, and an event longer than the list alone the per-event
//      way;
//   5. event lanes walk their candidates in order: ptv = pt * s, the jet cut,
//      the count, the left-to-right float32 H_T, the maximum, the b-tag count;
//      then the event cut and three fills into the workgroup's LDS
//      histograms (float64 sums, uint32 counts).  With several jet-energy
//      scales a lane takes an (event, group of kG scales) pair instead and
//      one walk serves the group.  The bins of all of a lane's fills are
//      found together.
// Steps 2-5 exchange data through the wavefront's own LDS region; a
// wavefront's LDS operations complete in issue order, so only compiler
// ordering fences are needed between them.  A tile whose objects exceed the
// capacity (for 64 events 448 jets, 192 muons, 128 electrons) runs as smaller
// sub-tiles; a single event beyond it is read straight from HBM, with the
// same arithmetic.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "lookup.hpp"

namespace hepk {

struct DsDev {
    int64_t n_events;
    const int64_t *joff, *moff, *eoff;
    const void *jpt, *jeta, *jphi, *jbt;
    const void *mpt, *meta, *mphi, *miso;
    const void *ept, *eeta, *ephi;
    const float *w;
    const float *npu;  // pileup per event (lookup weights); NULL: absent
    int64_t hist0;  // first slot of this dataset's block of histograms
    int64_t ev0;    // events of the datasets before this one (per-event records)
};

// A bucket table (PointLut) in the plan's edge table: first point, first word
// of the buckets, and the key's constants.
struct LutDev {
    int32_t p, l, np, shift, use_bits, M;
    float lo, hi, scale;
};

template <typename LT>
__device__ __forceinline__ PointLut lut_at(const LT &d, const float *E) {
    return PointLut{E + d.p, reinterpret_cast<const uint8_t *>(E + d.l), d.np, d.lo, d.hi, d.scale, d.shift,
                    d.use_bits != 0, d.M};
}

struct QDev {
    float mu_pt, mu_abseta, mu_iso, el_pt, el_abseta, jet_pt, jet_abseta, thr2, btag;
    int32_t min_mu, min_jet, min_b;
    int32_t n_scale, scale0;
    float smax;          // largest scale; used only when jet_pt >= 0
    // A jet with pt < ptmin (or NaN) is selected at no scale: the smallest pt
    // with pt * smax > jet_pt (with shifted energies a lower bound of it over
    // the table); -inf when jet_pt < 0, NaN when no pt is selected.
    float ptmin;
    int32_t active;      // 0: idle query slot, skipped
    int32_t nbins[3];
    int32_t ebase[3];    // first edge of each observable in the plan's edge table
    float lo[3], hi[3];  // first and last edge of each observable
    float inv_w[3];      // nbins / (hi - lo): start value of the bin search
    // The guess g = (x - lo) * inv_w (float32), clamped to [-0.5, top], can
    // name a wrong slot only where its fraction f = g - floor(g) has
    // |f - 0.5| >= chk (a bound the plan derives from the edges,
    // guess_bound); only such guesses are checked against the edges.
    float chk[3];
    float top[3];  // nbins + 0.5
    // Histogram of (scale v, observable h) starts at slot0 + v * per_scale +
    // hoff[h]: in the workgroup's LDS copy (compact over the active queries)
    // and in the dataset's block in HBM (fixed per query slot).
    int32_t lslot0, lper_scale, lhoff[3];
    int32_t gslot0, gper_scale, ghoff[3];
    // Lookup corrections (read by the LK kernels only).  Tables live in the
    // plan's edge table: pileup and muon scale-factor histograms (bins, first
    // edge, first slot content; pu_nb / sf_nb 0: that weight factor is
    // absent) and, with jes_mode 1, the jet-energy-scale shift table (rows of
    // |eta| bins, columns of pt bins, values row-major from jd); scales are
    // then shifts s with ptv = pt * (1 + s * delta).  smin: smallest scale.
    int32_t pu_nb, pu_e, pu_c, sf_nb, sf_e, sf_c;
    int32_t jes_mode, jr_nb, jr_e, jc_nb, jc_e, jd;
    float pu_lo, pu_hi, pu_iw, sf_lo, sf_hi, sf_iw;
    float jr_lo, jr_hi, jr_iw, jc_lo, jc_hi, jc_iw;
    float smin;
    // the shift table's bucket tables (centres of its columns, edges of its
    // rows) and segments (rows of jc_nb + 1, 4 floats each), when jseg >= 0
    int32_t jseg;
    LutDev jlr, jlc;
};

struct Chunk {
    int32_t d, pad;
    int64_t t0, t1;  // tiles [t0, t1) of dataset d
    int64_t pre;     // tiles of the chunks before this one
};

struct PipeArgs {
    const DsDev *ds;
    const QDev *qs;
    const float *scales;
    const Chunk *chunks;
    const float *edges;  // all queries' bin edges, concatenated
    int32_t chunk_begin, chunk_end;  // chunks [chunk_begin, chunk_end) of `chunks`
    int32_t n_q, ds_slots, n_edges, edges_in_lds;  // ds_slots: LDS histogram slots
    int32_t n_scales, scales_in_lds;               // the scale table, copied to LDS when small
    // the candidate lists in dynamic LDS: byte offset of the first wavefront's,
    // bytes of each, candidates each holds (list_fit)
    int32_t list_at, list_bytes, list_cap;
    double *sumw;
    uint64_t *counts;
    double *sumw2;  // LK kernels: sums of squared weights (NULL: not kept)
    // per-event records (kernels instantiated with DBG only): the record of
    // event e of dataset d for scale v of query q is
    // rec[(q.scale0 + v) * rec_events + d.ev0 + e]
    hepk_event_record *rec;
    int64_t rec_events;
};

// Writes the record of one event and scale (DBG kernels only).
__device__ __forceinline__ hepk_event_record *rec_at(const PipeArgs &P, int row, int64_t ev) {
    return P.rec + static_cast<int64_t>(row) * P.rec_events + ev;
}

template <bool LDSH, bool W2 = false>
struct HistSink {
    double *sw;        // LDS (LDSH) or the dataset's block in HBM
    uint32_t *c32;     // LDS (LDSH)
    uint64_t *c64;     // HBM (!LDSH)
    double *sw2;       // W2: squared weights (LDS or HBM like sw; NULL: not kept)

    __device__ __forceinline__ void add(int slot, double w) const {
        atomic_add_f64(&sw[slot], w);
        if (W2 && sw2) atomic_add_f64(&sw2[slot], w * w);
        if (LDSH)
            atomicAdd(&c32[slot], 1u);
        else
            atomic_add_u64(&c64[slot], 1u);
    }
    // LDS histograms: adds w (and one count) where f holds and +0 / 0 where
    // it does not, without a branch (adding +0 changes no sum of finite
    // weights but a -0 one, which compares equal)
    __device__ __forceinline__ void add_if(int slot, double w, bool f) const {
        atomic_add_f64(&sw[slot], f ? w : 0.0);
        if (W2 && sw2) atomic_add_f64(&sw2[slot], f ? w * w : 0.0);
        atomicAdd(&c32[slot], f ? 1u : 0u);
    }
};

// The lookup tables of one query as axes over the edge table E.
struct LkAxes {
    Axis pu, sf, jr, jc;
};

template <typename QT>
__device__ __forceinline__ LkAxes lk_axes(const QT &Q, const float *E) {
    LkAxes a;
    a.pu = Axis{E + Q.pu_e, Q.pu_nb, Q.pu_lo, Q.pu_hi, Q.pu_iw};
    a.sf = Axis{E + Q.sf_e, Q.sf_nb, Q.sf_lo, Q.sf_hi, Q.sf_iw};
    a.jr = Axis{E + Q.jr_e, Q.jr_nb, Q.jr_lo, Q.jr_hi, Q.jr_iw};
    a.jc = Axis{E + Q.jc_e, Q.jc_nb, Q.jc_lo, Q.jc_hi, Q.jc_iw};
    return a;
}

// The jet-energy-scale shift of a jet (pt, eta) from the query's table.
__device__ __forceinline__ float jes_shift(const LkAxes &a, const float *E, int jd, float pt, float eta) {
    const int row = lookup_row(a.jr, fabsf(eta));
    return lookup_interp(a.jc, E + jd + (row - 1) * a.jc.nb, pt);
}

// jes_shift of N jets at once (lookup2_n over the query's table).
template <int N>
__device__ __forceinline__ void jes_shift_n(const LkAxes &a, const float *E, int jd, const float (&pt)[N],
                                            const float (&eta)[N], float (&out)[N]) {
    lookup2_n<N>(a.jr, a.jc, E + jd, pt, eta, out);
}

// The same from the query's bucket tables and segments (lookup.hpp: the same
// bits with five LDS reads per jet instead of seventeen and no division:
// lookup pass over 1e7 events 719 -> 670 us).
template <int N, typename QT>
__device__ __forceinline__ void jes_lut_n(const QT &Q, const float *E, const float (&pt)[N], const float (&eta)[N],
                                          float (&out)[N]) {
    float ae[N];
    int row[N], pos[N];
#pragma unroll
    for (int n = 0; n < N; ++n) ae[n] = (eta[n] != eta[n]) ? -INFINITY : fabsf(eta[n]);  // NaN: the first row
    lut_count_n<N, true>(lut_at(Q.jlr, E), ae, row);
    lut_count_n<N, true>(lut_at(Q.jlc, E), pt, pos);
    const int nr = Q.jr_nb, nc = Q.jc_nb;
    const float mfirst = E[Q.jlc.p], mlast = E[Q.jlc.p + nc - 1];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const float *g =
            E + Q.jseg + 4 * ((min(max(row[n], 1), nr) - 1) * (nc + 1) + segment_of(pos[n], pt[n], mfirst));
        out[n] = segment_at(Segment{g[0], g[1], g[2], 0.0f}, pt[n], mfirst, mlast);
    }
}

// Largest pt * (1 + s * d) over the scales in [smin, smax]: the factor is
// monotone in s (its rounding is monotone) and the product monotone in the
// factor, so the extremes are at smin or smax.  NaN when pt or d is NaN.
__device__ __forceinline__ float shifted_pt_bound(float pt, float d, float smin, float smax) {
    const float f_hi = 1.0f + smax * d, f_lo = 1.0f + smin * d;
    const float a = pt * f_hi, b = pt * f_lo;
    return (a != a) ? b : (b != b ? a : fmaxf(a, b));
}

// Histogram constants of one query, read once per query and held in
// registers: they are uniform, and without the pin the compiler reloads each
// field from memory (and waits for it) next to every use.
struct FillC {
    int32_t base, per;  // first slot of scale 0, slots per scale (LDS or global layout)
    int32_t off[3];
    float lo[3], iw[3], ck[3], top[3];
};

template <typename X>
__device__ __forceinline__ X pin(X x) {
    asm volatile("" : "+s"(x));
    return x;
}

// All fields are read first and pinned by one statement, so their loads are
// issued together and waited for once.
template <bool LDSH, typename QT>
__device__ __forceinline__ FillC fill_consts(const QT &Q) {
    FillC F;
    F.base = LDSH ? Q.lslot0 : Q.gslot0;
    F.per = LDSH ? Q.lper_scale : Q.gper_scale;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        F.off[h] = LDSH ? Q.lhoff[h] : Q.ghoff[h];
        F.lo[h] = Q.lo[h];
        F.iw[h] = Q.inv_w[h];
        F.ck[h] = Q.chk[h];
        F.top[h] = Q.top[h];
    }
    asm volatile(""
                 : "+s"(F.base), "+s"(F.per), "+s"(F.off[0]), "+s"(F.off[1]), "+s"(F.off[2]), "+s"(F.lo[0]),
                   "+s"(F.lo[1]), "+s"(F.lo[2]), "+s"(F.iw[0]), "+s"(F.iw[1]), "+s"(F.iw[2]), "+s"(F.ck[0]),
                   "+s"(F.ck[1]), "+s"(F.ck[2]), "+s"(F.top[0]), "+s"(F.top[1]), "+s"(F.top[2]));
    return F;
}

// Slots of N values, x[n] going to observable n % 3 (H_T, lead, nJet): the
// same slot as hist_slot_lohi.  The guess from the uniform-bin formula, one bin
// beyond either end of the axis, is taken as exact unless its fraction is
// within the plan's bound of 0 or 1 (chk), so only lanes with such a guess
// read edges -- rarely any lane of a wavefront, so the round trip is usually
// skipped (eight queries, whose edges stay in HBM: 588 -> 544 us per 6.25e6
// events against checking every guess).  A value outside the axis is clamped
// to a fraction of 0.5 and never flagged (clamped to the bins instead, it was
// whenever the bound flagged anything: 20 scales over 3e6 events with 183 bins
// up to 300, a tail beyond them, 237 -> 189 us; without a tail 192 -> 184).  A
// binary search replaces a guess that was off.  The fills are a third of the
// multi-scale kernels' instructions, so no operation here is spare.
template <int N, typename QT>
__device__ __forceinline__ void find_bins(const FillC &F, const QT &Q, const float *edges, const float (&x)[N],
                                          int (&s)[N]) {
    bool chk = false;  // some value of this lane needs the edges
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int h = n % 3;
        const float g = (x[n] - F.lo[h]) * F.iw[h];
        const float c = __builtin_amdgcn_fmed3f(g, -0.5f, F.top[h]);
        s[n] = static_cast<int>(floorf(c)) + 1;
        chk |= !(fabsf(__builtin_amdgcn_fractf(c) - 0.5f) < F.ck[h]);
    }
    if (chk) {
        // every value of the lane by the edges (a right guess is kept)
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int h = n % 3, nb = Q.nbins[h];
            const float *E = edges + Q.ebase[h];
            const int k = min(max(s[n], 1), nb);
            const bool in = (x[n] >= Q.lo[h]) & (x[n] < Q.hi[h]);
            s[n] = x[n] >= Q.hi[h] ? nb + 1 : (in ? k : 0);
            if (in && (x[n] < E[k - 1] || x[n] >= E[k])) s[n] = bin_search(E, nb, x[n]);
        }
    }
}

// Fills H_T, lead and nJet of one passing event for scale v of query Q (a
// table entry read in place, so its fields are fetched where they are used).
template <bool LDSH, bool W2, typename QT>
__device__ __forceinline__ void fill3(const HistSink<LDSH, W2> &sink, const QT &Q, const float *edges, int v,
                                      float ht, float lead, int nj, double w) {
    const int base = LDSH ? Q.lslot0 + v * Q.lper_scale : Q.gslot0 + v * Q.gper_scale;
    const float xs[3] = {ht, lead, static_cast<float>(nj)};
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        const float x = xs[h];
        if (x != x) continue;
        const int s = hist_slot_lohi(x, edges + Q.ebase[h], Q.nbins[h], Q.lo[h], Q.hi[h], Q.inv_w[h]);
        sink.add(base + (LDSH ? Q.lhoff[h] : Q.ghoff[h]) + s, w);
    }
}

// Value of x in lane l (l uniform).
__device__ __forceinline__ float lane_f(float x, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}

// One event by the whole wavefront, columns read straight from HBM (events
// beyond the on-chip capacity): a lane per object, 64 at a time, for the cuts,
// the cone test and the lookups; then a lane per jet-energy scale takes the
// jets that are left one by one, in order, so that all scales share one
// reading of the columns.  LK: lookup event weights and, with jes_mode 1,
// shifted jet energies.
template <typename T, bool EXT, bool LDSH, bool DBG, bool LK>
__device__ __forceinline__ void event_direct(const PipeArgs &P, const DsDev &D, int64_t e, int lane,
                                             const float *edges, const HistSink<LDSH, LK> &sink) {
    const bool has_iso = D.miso != nullptr;
    const bool has_el = EXT && D.eoff != nullptr;
    const bool has_bt = EXT && D.jbt != nullptr;
    const int64_t j0 = as_const(D.joff)[e], m0 = as_const(D.moff)[e], l0 = has_el ? as_const(D.eoff)[e] : 0;
    const int64_t nj_all = as_const(D.joff)[e + 1] - j0, nm_all = as_const(D.moff)[e + 1] - m0;
    const int64_t nl_all = has_el ? as_const(D.eoff)[e + 1] - l0 : 0;
    const T *jpt = static_cast<const T *>(D.jpt) + j0, *jeta = static_cast<const T *>(D.jeta) + j0;
    const T *jphi = static_cast<const T *>(D.jphi) + j0, *jbt = static_cast<const T *>(D.jbt) + (has_bt ? j0 : 0);
    const T *mpt = static_cast<const T *>(D.mpt) + m0, *meta = static_cast<const T *>(D.meta) + m0;
    const T *mphi = static_cast<const T *>(D.mphi) + m0;
    const T *miso = static_cast<const T *>(D.miso) + (has_iso ? m0 : 0);
    const T *ept = static_cast<const T *>(D.ept) + l0, *eeta = static_cast<const T *>(D.eeta) + l0;
    const T *ephi = static_cast<const T *>(D.ephi) + l0;
    for (int q = 0; q < P.n_q; ++q) {
        const auto &Q = as_const(P.qs)[q];
        if (!Q.active) continue;
        auto mu_sel = [&](int64_t m) {
            return ldf(mpt, m) > Q.mu_pt && fabsf(ldf(meta, m)) < Q.mu_abseta &&
                   (!has_iso || ldf(miso, m) < Q.mu_iso);
        };
        auto el_sel = [&](int64_t m) { return ldf(ept, m) > Q.el_pt && fabsf(ldf(eeta, m)) < Q.el_abseta; };
        // event weight: w, times the pileup lookup, times the product (left
        // to right from 1) of the selected muons' scale factors
        const bool use_sf = LK && Q.sf_nb > 0;
        LkAxes ax{};
        if (LK) ax = lk_axes(Q, edges);
        int nmu = 0;
        float prod = 1.0f;
        for (int64_t m = 0; m < nm_all; m += 64) {
            const bool sel = m + lane < nm_all && mu_sel(m + lane);
            uint64_t b = __ballot(sel);
            nmu += __popcll(b);
            if (use_sf) {
                const float f = sel ? lookup_bin(ax.sf, edges + Q.sf_c, ldf(mpt, m + lane)) : 1.0f;
                for (; b; b &= b - 1) prod = prod * lane_f(f, __builtin_ctzll(b));
            }
        }
        float wq = D.w ? as_const(D.w)[e] : 1.0f;
        if (LK && Q.pu_nb > 0 && D.npu) wq = wq * lookup_bin(ax.pu, edges + Q.pu_c, as_const(D.npu)[e]);
        if (use_sf) wq = wq * prod;
        const bool shift = LK && Q.jes_mode == 1;
        const int V = Q.n_scale;
        for (int v0 = 0; v0 < V; v0 += 64) {
            const int v = v0 + lane;
            const float s = P.scales[Q.scale0 + min(v, V - 1)];
            int nj = 0, nb = 0;
            float ht = 0.0f, lead = -INFINITY;
            for (int64_t j = 0; j < nj_all; j += 64) {
                const int64_t i = j + lane;
                float pt = 0.0f, eta = 0.0f, phi = 0.0f, d = 0.0f;
                bool keep = false, tag = false;
                if (i < nj_all) {
                    pt = ldf(jpt, i);
                    eta = ldf(jeta, i);
                    phi = ldf(jphi, i);
                    keep = (pt >= Q.ptmin) & (fabsf(eta) < Q.jet_abseta);
                    if (has_bt) tag = ldf(jbt, i) > Q.btag;
                }
                if (__ballot(keep) == 0) continue;
                // (leptons 64 at a time too, the selected ones broadcast)
                auto cone = [&](int64_t n, const T *le, const T *lp, auto &&sel) {
                    for (int64_t m = 0; m < n; m += 64) {
                        const bool in = m + lane < n;
                        const float ve = in ? ldf(le, m + lane) : 0.0f, vp = in ? ldf(lp, m + lane) : 0.0f;
                        for (uint64_t b = __ballot(in && sel(m + lane)); b; b &= b - 1) {
                            const int l = __builtin_ctzll(b);
                            keep = keep & !(delta_r2(eta, phi, lane_f(ve, l), lane_f(vp, l)) <= Q.thr2);
                        }
                    }
                };
                cone(nm_all, meta, mphi, mu_sel);
                if (EXT) cone(nl_all, eeta, ephi, el_sel);
                if (shift && keep) d = jes_shift(ax, edges, Q.jd, pt, eta);
                const uint64_t tags = __ballot(keep && tag);
                for (uint64_t b = __ballot(keep); b; b &= b - 1) {
                    const int l = __builtin_ctzll(b);
                    const float p = lane_f(pt, l);
                    const float x = shift ? p * (1.0f + s * lane_f(d, l)) : p * s;
                    const bool sel = x > Q.jet_pt;
                    const float hs = ht + x;
                    ht = sel ? hs : ht;
                    lead = sel ? fmaxf(lead, x) : lead;
                    nj += sel ? 1 : 0;
                    nb += sel ? static_cast<int>((tags >> l) & 1u) : 0;
                }
            }
            const bool pass = nmu >= Q.min_mu && nj >= Q.min_jet && (!has_bt || nb >= Q.min_b);
            if (v < V) {
                if (DBG)
                    *rec_at(P, Q.scale0 + v, D.ev0 + e) =
                        hepk_event_record{nmu, nj, nb, pass ? 3 : 2, ht, lead, wq, 0};
                if (pass) fill3(sink, Q, edges, v, ht, lead, nj, static_cast<double>(wq));
            }
        }
    }
}

template <int EVPL, bool EXT, bool LK>
struct Caps {
    static constexpr int TW = 64 * EVPL;             // events per wavefront tile
    // (Seven jet slots where six hold the paper's five per event with 3.5 sigma
    // to spare: at six per event six slots split most tiles, 2e6 events 68 us
    // against 50; at five they would be 2% faster.)
    static constexpr int JK = 6 * EVPL + 1;          // jet slots per lane
    static constexpr int MK = 2 * EVPL;              // muon slots per lane
    // One more slot of muons that no register holds: read per query in the
    // tiles that have so many (at two muons per event half of the tiles do).
    // 3e6 events of 2.3 muons, those tiles split in two / with the slot: base
    // 109 / 76 us, eight queries 516 / 353, extended 170 / 109.  A third
    // register slot would leave five wavefronts per SIMD instead of six.  The
    // lookup kernels, whose LDS is full, split.
    static constexpr int MX = LK ? 0 : 1;
    static constexpr int EK = EXT ? 2 * EVPL : 1;    // electron slots per lane
    static constexpr int JC = 64 * JK, MC = 64 * (MK + MX), EC = 64 * EK;
    // The least the dense list of candidates holds (a tile with more takes
    // its events in several passes, each as many as fit); a launch takes as
    // much as the LDS leaves at its occupancy, up to all JC jets (list_fit).
    // The base selection lists 86 candidates of a 64-event tile on average
    // (99%: 123), the extended one 47 (83), a selection without cuts all 320.
    // (The extended schema at two events per lane runs eight wavefronts per CU
    // whatever its list.)
    static constexpr int CAP_MIN = EXT ? (EVPL == 1 ? 128 : 512) : (EVPL == 1 ? 128 : 256);
};

template <bool P>
using cpre_t = std::conditional_t<P, uint32_t, uint16_t>;

// eta and phi in LDS: the content's own type in the extended schema at one
// event per lane (LDS is what limits its wavefronts), else float32 (float16
// copies would take registers beside the values of the cuts).
template <typename T, int EVPL, bool EXT>
using lds_t = std::conditional_t<EXT && EVPL == 1, T, float>;

// A dense candidate: pt until the cone test, then NaN for a removed one (with
// one scale and jet_pt >= 0: pt * s, +0 for a removed one), eta, phi, and with
// lookups the energy shift.  The b-tags are bytes of their own behind the list.
template <typename TL, bool LK>
struct Cand {
    float pt;
    TL eta, phi;
};
template <typename TL>
struct Cand<TL, true> {
    float pt, jd;
    TL eta, phi;
};

// Bytes of one wavefront's list of cap candidates.  Its space first holds the
// prefix counts of step 3: candidates (low 16 bits) and, extended schema,
// b-tagged candidates (high 16 bits) before every tile jet.
template <typename T, int EVPL, bool EXT, bool LK>
constexpr int list_bytes(int cap) {
    const int list = cap * static_cast<int>(sizeof(Cand<lds_t<T, EVPL, EXT>, LK>) + (EXT ? 1 : 0));
    const int pre = (Caps<EVPL, EXT, LK>::JC + 1) * static_cast<int>(sizeof(cpre_t<EXT>));
    return ((list > pre ? list : pre) + 15) & ~15;
}

// One wavefront's LDS.  The selected muons and (extended schema) electrons
// share one pair of arrays in the content's own type, the electrons from
// index EO = MC + 2 on, so one index runs over an event's muons and then its
// electrons.
template <typename T, int EVPL, bool EXT, bool LK, bool MS>
struct WaveLds {
    using C = Caps<EVPL, EXT, LK>;
    using TL = lds_t<T, EVPL, EXT>;
    // selected muons, compacted in tile order (+2 padding), then (EXT) the
    // selected electrons likewise from index EO
    TL seta[C::MC + 2 + (EXT ? C::EC + 2 : 0)], sphi[C::MC + 2 + (EXT ? C::EC + 2 : 0)];
    // jets of the events that can pass, as bits; first candidate of each
    // such event in the dense list, as bits
    uint64_t em[16 + C::JK];  // (JK words of either kind; the second is read 32 lanes wide)
    static constexpr int SM = C::JK;  // the second kind starts here
    union {
        struct {  // steps 2-3: selected leptons before lepton m
            float ssf[LK ? C::MC : 1];  // LK: selected muons' pt, then their scale factors
            uint16_t mpre[C::MC + 1];
            uint16_t epre[EXT ? C::EC + 1 : 1];
        } p;
        struct {  // step 4: selected-lepton ranges (first | count << 16) of the
                  // events with candidates, muons and electrons
            uint32_t mu[C::TW];
            uint32_t el[EXT ? C::TW : 1];
        } r;
        struct {  // step 5, several scales: the listed events, candidate
                  // range (first | end << 16) and weight
            uint32_t evjr[MS ? C::TW : 1];
            float evw[MS ? C::TW : 1];
        } w;
    } u;
};

// A selected energy is above jet_pt, so neither NaN nor -inf, and the leading
// pt and the count are never NaN.  H_T is NaN only if negative energies sum to
// -inf and one of +inf follows; an event's fewer than 2^32 jets above a jet_pt
// of -1e28 do not get there.
__device__ __forceinline__ bool ht_can_be_nan(float jet_pt) { return jet_pt < -1e28f; }

// Adds weight w to the histograms of scales v0 + n / 3 (observable n % 3)
// of the lanes whose pass[n / 3] is set.  No value is NaN (ht_can_be_nan).  With
// several scales and LDS histograms every lane adds, zero where it does not
// fill, at a slot of a scale no later than vlast (the query's last), so no
// value needs its own branch.
template <int N, bool MS, bool LDSH, bool W2, typename QT>
__device__ __forceinline__ void fill_bins(const HistSink<LDSH, W2> &sink, const FillC &F, const QT &Q,
                                          const float *edges, const float (&xs)[N], const bool (&pass)[N / 3], int v0,
                                          double w, int vlast) {
    int sl[N];
    find_bins<N>(F, Q, edges, xs, sl);
    if (MS && LDSH) {
#pragma unroll
        for (int n = 0; n < N; ++n)
            sink.add_if(F.base + min(v0 + n / 3, vlast) * F.per + F.off[n % 3] + sl[n], w,
                        pass[n / 3]);
        return;
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
        if (pass[n / 3]) sink.add(F.base + (v0 + n / 3) * F.per + F.off[n % 3] + sl[n], w);
}

// Scales per lane in the walk over an event's jets when a query has several
// (even: the fills take them two at a time).
constexpr int kG = 4;

// Walks the candidates [j0, j1) of one event in order (pt of each in LDS, NaN
// when removed by the cone test) for G scales at once: per scale the
// left-to-right float32 H_T of the selected jets (ptv > jet_pt), their
// count, b-tag count and maximum.  Adding only selected values keeps the sum
// order of the definition.  ptv = pt * s, or with JM (shifted energies)
// pt * (1 + s * d) with the jet's shift d from LDS.  For ptv = pt * s the
// maximum needs no per-scale work: for s > 0, rounding pt * s is monotone
// in pt, so the selected jets are those above a pt bound and the largest
// selected pt * s is the largest cleaned pt times s (rounded once), whenever
// any jet is selected; with JM the factor differs per jet and the maximum is
// taken per scale.  Branch-free, two jets per step (both LDS reads in
// flight).
template <int G, bool EXT, bool JM, typename CT>
__device__ __forceinline__ void walk_jets(const CT *C, const uint8_t *bt, int j0, int j1, const float (&sc)[G], float jet_pt,
                                          float (&ht)[G], float (&lead)[G], int (&nj)[G], int (&nb)[G]) {
    float pmax = -INFINITY;
    // selected jets (low 16 bits) and selected b-tagged jets (high 16 bits)
    // in one counter per scale: a range holds at most JC < 2^16 jets
    uint32_t cnt[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        ht[g] = 0.0f;
        cnt[g] = 0u;
        lead[g] = -INFINITY;
    }
    auto step = [&](float p, float d, int bt) {
        pmax = fmaxf(pmax, p);  // NaN (removed jet) leaves it unchanged
        const uint32_t inc = EXT ? 1u + (static_cast<uint32_t>(bt) << 16) : 1u;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float f = JM ? 1.0f + sc[g] * d : sc[g];
            const float x = p * f;
            const bool sel = x > jet_pt;
            const float hs = ht[g] + x;
            ht[g] = sel ? hs : ht[g];
            cnt[g] += sel ? inc : 0u;
            if (JM) lead[g] = sel ? fmaxf(lead[g], x) : lead[g];
        }
    };
    int k = j0;
    for (; k + 2 <= j1; k += 2) {
        const float p0 = C[k].pt, p1 = C[k + 1].pt;
        float d0 = 0.0f, d1 = 0.0f;
        if constexpr (JM) {
            d0 = C[k].jd;
            d1 = C[k + 1].jd;
        }
        const int b0 = EXT ? bt[k] : 0, b1 = EXT ? bt[k + 1] : 0;
        step(p0, d0, b0);
        step(p1, d1, b1);
    }
    if (k < j1) {
        float d = 0.0f;
        if constexpr (JM) d = C[k].jd;
        step(C[k].pt, d, EXT ? static_cast<int>(bt[k]) : 0);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        nj[g] = static_cast<int>(cnt[g] & 0xffffu);
        nb[g] = EXT ? static_cast<int>(cnt[g] >> 16) : 0;
        if (!JM) lead[g] = nj[g] > 0 ? pmax * sc[g] : -INFINITY;
    }
}

// The same reductions for one scale s when the cone test already stored
// every selected jet as pt * s and every other candidate as +0 (possible when
// jet_pt >= 0: a selected value exceeds jet_pt >= 0, so it is positive and
// the count is that of positive values).  Adding +0 leaves a float32 sum of
// positive values unchanged, so summing every stored value keeps the sum
// order of the definition.  The b-tag flag is stored already ANDed with the
// selection.
template <bool EXT, typename CT>
__device__ __forceinline__ void walk_selected(const CT *C, const uint8_t *bt, int j0, int j1, float &ht, float &lead, int &nj,
                                              int &nb) {
    float h = 0.0f, m = 0.0f;
    int n = 0, b = 0;
    auto step = [&](float x, int bt) {
        h += x;
        n += x > 0.0f ? 1 : 0;
        m = fmaxf(m, x);
        if (EXT) b += bt;
    };
    int k = j0;
    for (; k + 2 <= j1; k += 2) {
        const float x0 = C[k].pt, x1 = C[k + 1].pt;
        const int b0 = EXT ? bt[k] : 0, b1 = EXT ? bt[k + 1] : 0;
        step(x0, b0);
        step(x1, b1);
    }
    if (k < j1) step(C[k].pt, EXT ? static_cast<int>(bt[k]) : 0);
    ht = h;
    nj = n;
    nb = b;
    lead = n > 0 ? m : -INFINITY;
}

// A tile's first object of each collection and its object counts (32-bit:
// the counts are what the kernel compares and indexes with).
struct TileBounds {
    int64_t J0, M0, L0;
    int32_t nj, nm, nl;
};

template <bool EXT, typename DT>
__device__ __forceinline__ TileBounds tile_bounds(const DT &D, bool has_el, int64_t e0, int ne) {
    TileBounds b;
    b.J0 = as_const(D.joff)[e0];
    b.nj = static_cast<int32_t>(as_const(D.joff)[e0 + ne] - b.J0);
    b.M0 = as_const(D.moff)[e0];
    b.nm = static_cast<int32_t>(as_const(D.moff)[e0 + ne] - b.M0);
    b.L0 = (EXT && has_el) ? as_const(D.eoff)[e0] : 0;
    b.nl = (EXT && has_el) ? static_cast<int32_t>(as_const(D.eoff)[e0 + ne] - b.L0) : 0;
    return b;
}

// Number of set bits of m below this lane, plus base.
__device__ __forceinline__ int bits_below(uint64_t m, int base) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(
        static_cast<uint32_t>(m >> 32),
        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), static_cast<uint32_t>(base))));
}

// The 64-bit word whose halves lanes l and l + 1 hold, in scalar registers.
__device__ __forceinline__ uint64_t lane_u64(uint32_t x, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane(x, l), hi = __builtin_amdgcn_readlane(x, l + 1);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ void or_u64(uint64_t *p, uint64_t v) {
    atomicOr(reinterpret_cast<unsigned long long *>(p), static_cast<unsigned long long>(v));
}

// Compacts the selected objects of a tile (sel per slot k of this lane) into
// (eta, phi) arrays in tile order (and, with V3, a third value into o3);
// pre[m] = number of selected objects before object m, for every m up to
// 64 * K (all selected objects for m at or beyond the tile's count).
// Returns the number of selected objects.
template <int K, bool V3, typename TL>
__device__ __forceinline__ int compact(const bool (&sel)[K], const float (&eta)[K], const float (&phi)[K],
                                       int lane, TL *oeta, TL *ophi, uint16_t *pre, const float *v3 = nullptr,
                                       float *o3 = nullptr) {
    int run = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t bal = __ballot(sel[k]);
        const int before = bits_below(bal, run);
        pre[lane + 64 * k] = static_cast<uint16_t>(before);
        if (sel[k]) {
            oeta[before] = static_cast<TL>(eta[k]);
            ophi[before] = static_cast<TL>(phi[k]);
            if (V3) o3[before] = v3[k];
        }
        run += __popcll(bal);
    }
    pre[64 * K] = static_cast<uint16_t>(run);
    return run;
}

// MS: the plan has queries with several jet-energy scales (every query then
// takes the scale-group walk of step 5; otherwise every query has one scale).
// What bounds it: VALU issue (79% of the issue slots with 20 scales, with or
// without lookups, 67% with eight queries, 59% with one) and, per wavefront,
// the wait for a tile's loads and a dozen dependent LDS round trips; so the
// dense list, which cut the instructions per tile (base 545 -> 468, 20 scales
// 1630 -> 1227), and as many wavefronts as registers and LDS allow.  Asked for
// per SIMD: six in the base schema at one scale and one event per lane (at
// most 80 VGPRs; five took 5% longer per 1e7 events, seven, which 256-thread
// workgroups would get, 24%); four in the extended one, with lookups and in
// the base schema at two events; two with several scales, which the launch
// bound of their default 1024 threads raises to four, and in the extended
// schema at two events (four spills).  Before the list / now: 1e7 base events
// 210 / 200 us, eight queries over 6.25e6 events 764 / 518, 20 scales over 2e7
// float16 events 1031 / 795, 20 shifts with lookup weights over 1e7 1467 /
// 662 (there also two wavefronts per SIMD -> four, and shift and scale-factor
// searches for listed jets and selected muons only).  Loading the next tile
// into the registers while the list is worked on was slower at four
// wavefronts (280 us against 240).
// DBG: also write every event's per-scale record (counts, H_T, leading pt,
// whether the event was walked and whether it passed) to P.rec -- the
// intermediate values of the pass, for checking them one by one.  Product
// launches use DBG = false; the arithmetic is the same in both.
// LK: the lookup corrections of Sec. IV -- event weights from the pileup and
// muon scale-factor lookup histograms, jet energies shifted by an
// interpolated table (jes_mode 1) -- and the sums of squared weights; a
// query without lookups runs exactly as in the kernels without LK.
template <typename T, bool EXT, int WAVES, int EVPL, bool LDSH, bool MS, bool DBG, bool LK>
__global__ __launch_bounds__(64 * WAVES)
    __attribute__((amdgpu_waves_per_eu(MS || (EVPL == 2 && EXT) ? 2 : (EXT || LK || EVPL == 2 ? 4 : 6)))) void
    pipeline_kernel(PipeArgs P) {
    using C = Caps<EVPL, EXT, LK>;
    constexpr int TW = C::TW, JK = C::JK, MK = C::MK, MX = C::MX, EK = C::EK;
    __shared__ WaveLds<T, EVPL, EXT, LK, MS> wl[WAVES];
    using TL = typename WaveLds<T, EVPL, EXT, LK, MS>::TL;
    // per workgroup: [sumw | sumw2 (LK) | counts (u32) | edges | scales | candidate lists]
    extern __shared__ double dyn[];

    const int tid = threadIdx.x;
    int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto &L = wl[wave];
    // this wavefront's list, its b-tags, and the prefix counts in its space
    const int cap = P.list_cap;
    auto *cand = reinterpret_cast<Cand<TL, LK> *>(reinterpret_cast<char *>(dyn) + P.list_at + wave * P.list_bytes);
    uint8_t *cbt = reinterpret_cast<uint8_t *>(cand + cap);
    auto *cpre = reinterpret_cast<cpre_t<EXT> *>(cand);

    double *sw_s = dyn;
    double *sw2_s = dyn + (LDSH ? P.ds_slots : 0);
    uint32_t *c_s = reinterpret_cast<uint32_t *>(sw2_s + ((LDSH && LK) ? P.ds_slots : 0));
    float *e_s = reinterpret_cast<float *>(c_s + (LDSH ? P.ds_slots : 0));
    if (LDSH) {
        for (int i = tid; i < P.ds_slots; i += 64 * WAVES) {
            sw_s[i] = 0.0;
            if (LK) sw2_s[i] = 0.0;
            c_s[i] = 0u;
        }
    }
    float *s_s = e_s + (P.edges_in_lds ? P.n_edges : 0);
    const float *edges = P.edges;
    if (P.edges_in_lds) {
        for (int i = tid; i < P.n_edges; i += 64 * WAVES) e_s[i] = as_const(P.edges)[i];
        edges = e_s;
    }
    if (P.scales_in_lds)
        for (int i = tid; i < P.n_scales; i += 64 * WAVES) s_s[i] = as_const(P.scales)[i];
    __syncthreads();
    // Runs f on the table (edges and lookup tables) where it lives, with a
    // pointer whose address space the compiler can see (LDS reads rather
    // than flat ones).
    auto on_tables = [&](auto &&f) {
        if (P.edges_in_lds)
            f(static_cast<const float *>(e_s));
        else
            f(static_cast<const float *>(P.edges));
    };

    // This workgroup's work: an equal slice [my0, my1) of the concatenated
    // tiles of chunks [chunk_begin, chunk_end); its first chunk is found by a
    // binary search over the chunks' tile prefixes (uniform, scalar loads).
    const auto chs = as_const(P.chunks);
    const int64_t T0 = chs[P.chunk_begin].pre;
    const int64_t nT = chs[P.chunk_end - 1].pre + (chs[P.chunk_end - 1].t1 - chs[P.chunk_end - 1].t0) - T0;
    const int64_t my0 = T0 + nT * blockIdx.x / gridDim.x;
    const int64_t my1 = T0 + nT * (blockIdx.x + 1) / gridDim.x;
    int cfirst = P.chunk_begin;
    for (int hi = P.chunk_end - 1; cfirst < hi;) {  // last chunk with pre <= my0
        const int mid = (cfirst + hi + 1) >> 1;
        if (chs[mid].pre <= my0)
            cfirst = mid;
        else
            hi = mid - 1;
    }
    for (int ci = cfirst; ci < P.chunk_end && my0 < my1; ++ci) {
        const Chunk CH = chs[ci];
        if (CH.pre >= my1) break;
        // this workgroup's tiles of the chunk
        const int64_t c_t0 = CH.t0 + max<int64_t>(my0 - CH.pre, 0);
        const int64_t c_t1 = CH.t0 + min<int64_t>(my1 - CH.pre, CH.t1 - CH.t0);
        if (c_t1 <= c_t0) continue;
        const auto &D = as_const(P.ds)[CH.d];  // read in place, like the query table
        HistSink<LDSH, LK> sink;
        if (LDSH) {
            sink.sw = sw_s;
            sink.c32 = c_s;
            sink.sw2 = (LK && P.sumw2) ? sw2_s : nullptr;
        } else {
            sink.sw = P.sumw + D.hist0;
            sink.c64 = P.counts + D.hist0;
            sink.sw2 = (LK && P.sumw2) ? P.sumw2 + D.hist0 : nullptr;
        }
        const bool has_iso = D.miso != nullptr;
        const bool has_el = EXT && D.eoff != nullptr;
        const bool has_bt = EXT && D.jbt != nullptr;

        // The raw loads of one tile (the offsets as their low 32-bit words:
        // tile-relative differences are exact modulo 2^32).
        // (content as raw bits: float32, or float16 in the low half)
        struct Raw {
            uint32_t j0[EVPL], j1[EVPL], m0[EVPL], m1[EVPL], l0[EVPL], l1[EVPL];
            float w[EVPL];
            float npu[LK ? EVPL : 1];
            uint32_t jpt[JK], jeta[JK], jphi[JK], jbt[EXT ? JK : 1];
            uint32_t mpt[MK], meta[MK], mphi[MK], miso[MK];
            uint32_t lpt[EK], leta[EK], lphi[EK];
        };
        // The chunk's tiles are counted from c_t0 in 32 bits (a workgroup's
        // share of one dataset has far fewer than 2^31 tiles); only the last
        // one can hold fewer than TW events.
        const int nt = static_cast<int>(c_t1 - c_t0);
        const int64_t ebase = c_t0 * TW;
        const int tn_last = static_cast<int>(min<int64_t>(TW, D.n_events - (c_t1 - 1) * TW));
        auto tile_events = [&](int r) { return r == nt - 1 ? tn_last : TW; };
        auto bounds_of = [&](int r) {
            return tile_bounds<EXT>(D, has_el, ebase + static_cast<int64_t>(r) * TW, tile_events(r));
        };
        // (compared unsigned: a count of 2^31 to 2^32 objects, which valid
        // offsets of one tile never give, also goes the per-event way)
        auto oversize = [&](const TileBounds &b) {
            return static_cast<uint32_t>(b.nj) > static_cast<uint32_t>(C::JC) ||
                   static_cast<uint32_t>(b.nm) > static_cast<uint32_t>(C::MC) ||
                   static_cast<uint32_t>(b.nl) > static_cast<uint32_t>(C::EC);
        };
        // ---- 1. all of a tile's loads, without waiting: both offsets of each
        // event lane's event (their low 32-bit words), its weight, and up to
        // JK jets, MK muons and EK electrons per lane (consecutive lanes,
        // consecutive objects).  Buffer loads over exactly the tile's range
        // of each column read 0 past its end, which is the value every
        // unused slot must hold.
        auto issue = [&](int64_t e0, int ne, const TileBounds &b, Raw &R) __attribute__((always_inline)) {
            // the extended schema measured 1.5% faster with nontemporal loads,
            // the base schema 1.3% slower
            constexpr int AUX = EXT ? kBufNt : 0;
            const int nj = b.nj, nm = b.nm, nl = b.nl;
            // offsets: events e0 .. e0 + ne (both ends of each event)
            const uint32_t ob = static_cast<uint32_t>(ne + 1) * 8u;
            const buf_t bjo = buf_span(D.joff + e0, ob), bmo = buf_span(D.moff + e0, ob);
            const buf_t beo = buf_span((EXT && has_el) ? D.eoff + e0 : D.joff + e0, ob);
            const buf_t bw = buf_span(D.w ? static_cast<const void *>(D.w + e0) : D.joff, static_cast<uint32_t>(ne) * 4u);
            const buf_t bpu =
                buf_span(LK && D.npu ? static_cast<const void *>(D.npu + e0) : D.joff, static_cast<uint32_t>(ne) * 4u);
#pragma unroll
            for (int r = 0; r < EVPL; ++r) {
                const int ev = lane + 64 * r;
                R.j0[r] = buf_u32<AUX>(bjo, ev * 8);
                R.j1[r] = buf_u32<AUX>(bjo, ev * 8 + 8);
                R.m0[r] = buf_u32<AUX>(bmo, ev * 8);
                R.m1[r] = buf_u32<AUX>(bmo, ev * 8 + 8);
                R.l0[r] = R.l1[r] = 0;
                if (EXT && has_el) {
                    R.l0[r] = buf_u32<AUX>(beo, ev * 8);
                    R.l1[r] = buf_u32<AUX>(beo, ev * 8 + 8);
                }
                R.w[r] = D.w ? __builtin_bit_cast(float, buf_u32<AUX>(bw, ev * 4)) : 1.0f;
                if (LK) R.npu[LK ? r : 0] = D.npu ? __builtin_bit_cast(float, buf_u32<AUX>(bpu, ev * 4)) : 0.0f;
            }
            const uint32_t es = sizeof(T);
            const buf_t bjpt = buf_span(static_cast<const T *>(D.jpt) + b.J0, nj * es);
            const buf_t bjeta = buf_span(static_cast<const T *>(D.jeta) + b.J0, nj * es);
            const buf_t bjphi = buf_span(static_cast<const T *>(D.jphi) + b.J0, nj * es);
#pragma unroll
            for (int k = 0; k < JK; ++k) {
                const int j = lane + 64 * k;
                R.jpt[k] = buf_raw<T, AUX>(bjpt, j);
                R.jeta[k] = buf_raw<T, AUX>(bjeta, j);
                R.jphi[k] = buf_raw<T, AUX>(bjphi, j);
                if (EXT) R.jbt[EXT ? k : 0] = 0u;
            }
            if (EXT && has_bt) {
                const buf_t bjbt = buf_span(static_cast<const T *>(D.jbt) + b.J0, nj * es);
#pragma unroll
                for (int k = 0; k < JK; ++k) R.jbt[EXT ? k : 0] = buf_raw<T, AUX>(bjbt, lane + 64 * k);
            }
            const buf_t bmpt = buf_span(static_cast<const T *>(D.mpt) + b.M0, nm * es);
            const buf_t bmeta = buf_span(static_cast<const T *>(D.meta) + b.M0, nm * es);
            const buf_t bmphi = buf_span(static_cast<const T *>(D.mphi) + b.M0, nm * es);
#pragma unroll
            for (int k = 0; k < MK; ++k) {
                const int m = lane + 64 * k;
                R.mpt[k] = buf_raw<T, AUX>(bmpt, m);
                R.meta[k] = buf_raw<T, AUX>(bmeta, m);
                R.mphi[k] = buf_raw<T, AUX>(bmphi, m);
                R.miso[k] = 0u;
            }
            if (has_iso) {
                const buf_t bmiso = buf_span(static_cast<const T *>(D.miso) + b.M0, nm * es);
#pragma unroll
                for (int k = 0; k < MK; ++k) R.miso[k] = buf_raw<T, AUX>(bmiso, lane + 64 * k);
            }
#pragma unroll
            for (int k = 0; k < EK; ++k) R.lpt[k] = R.leta[k] = R.lphi[k] = 0u;
            if (EXT && has_el) {
                const buf_t bept = buf_span(static_cast<const T *>(D.ept) + b.L0, nl * es);
                const buf_t beeta = buf_span(static_cast<const T *>(D.eeta) + b.L0, nl * es);
                const buf_t bephi = buf_span(static_cast<const T *>(D.ephi) + b.L0, nl * es);
#pragma unroll
                for (int k = 0; k < EK; ++k) {
                    const int m = lane + 64 * k;
                    R.lpt[k] = buf_raw<T, AUX>(bept, m);
                    R.leta[k] = buf_raw<T, AUX>(beeta, m);
                    R.lphi[k] = buf_raw<T, AUX>(bephi, m);
                }
            }
        };
        // Every value of R is used here, so the compiler waits for the tile's
        // loads at this point (once), not at each value's first use.
        auto settle = [&](Raw &R) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < EVPL; ++r)
                asm volatile("" ::"v"(R.j0[r]), "v"(R.j1[r]), "v"(R.m0[r]), "v"(R.m1[r]), "v"(R.w[r]));
            if (LK) {
#pragma unroll
                for (int r = 0; r < EVPL; ++r) asm volatile("" ::"v"(R.npu[LK ? r : 0]));
            }
#pragma unroll
            for (int k = 0; k < JK; ++k) asm volatile("" ::"v"(R.jpt[k]), "v"(R.jeta[k]), "v"(R.jphi[k]));
#pragma unroll
            for (int k = 0; k < MK; ++k)
                asm volatile("" ::"v"(R.mpt[k]), "v"(R.meta[k]), "v"(R.mphi[k]), "v"(R.miso[k]));
            if (EXT) {
#pragma unroll
                for (int r = 0; r < EVPL; ++r) asm volatile("" ::"v"(R.l0[r]), "v"(R.l1[r]));
#pragma unroll
                for (int k = 0; k < JK; ++k) asm volatile("" ::"v"(R.jbt[EXT ? k : 0]));
#pragma unroll
                for (int k = 0; k < EK; ++k) asm volatile("" ::"v"(R.lpt[k]), "v"(R.leta[k]), "v"(R.lphi[k]));
            }
        };
        // Steps 2-5 for every query on a settled tile.
        auto work = [&](int64_t e0, int ne, const TileBounds &B, Raw &R) __attribute__((always_inline)) {
            const int nj = B.nj, nm = B.nm, nl = B.nl;
            int32_t jb[EVPL], je[EVPL], mb[EVPL], me[EVPL], lb[EVPL], le[EVPL];
            float wv[EVPL];
#pragma unroll
            for (int r = 0; r < EVPL; ++r) {
                const bool in = lane + 64 * r < ne;
                jb[r] = in ? static_cast<int32_t>(R.j0[r] - static_cast<uint32_t>(B.J0)) : 0;
                je[r] = in ? static_cast<int32_t>(R.j1[r] - static_cast<uint32_t>(B.J0)) : 0;
                mb[r] = in ? static_cast<int32_t>(R.m0[r] - static_cast<uint32_t>(B.M0)) : 0;
                me[r] = in ? static_cast<int32_t>(R.m1[r] - static_cast<uint32_t>(B.M0)) : 0;
                lb[r] = (in && EXT && has_el) ? static_cast<int32_t>(R.l0[r] - static_cast<uint32_t>(B.L0)) : 0;
                le[r] = (in && EXT && has_el) ? static_cast<int32_t>(R.l1[r] - static_cast<uint32_t>(B.L0)) : 0;
                wv[r] = R.w[r];
            }
            float jpt[JK], jeta[JK], jphi[JK], jbt[EXT ? JK : 1];
            float mpt[MK], meta[MK], mphi[MK], miso[MK];
            float lpt[EK], leta[EK], lphi[EK];
#pragma unroll
            for (int k = 0; k < JK; ++k) {
                jpt[k] = raw_f<T>(R.jpt[k]);
                jeta[k] = raw_f<T>(R.jeta[k]);
                jphi[k] = raw_f<T>(R.jphi[k]);
                if (EXT) jbt[EXT ? k : 0] = raw_f<T>(R.jbt[EXT ? k : 0]);
            }
#pragma unroll
            for (int k = 0; k < MK; ++k) {
                mpt[k] = raw_f<T>(R.mpt[k]);
                meta[k] = raw_f<T>(R.meta[k]);
                mphi[k] = raw_f<T>(R.mphi[k]);
                miso[k] = raw_f<T>(R.miso[k]);
            }
#pragma unroll
            for (int k = 0; k < EK; ++k) {
                lpt[k] = raw_f<T>(R.lpt[k]);
                leta[k] = raw_f<T>(R.leta[k]);
                lphi[k] = raw_f<T>(R.lphi[k]);
            }
            (void)jbt;
            (void)lpt;
            // Per query, the events [wlo, whi) of the tile: all of them, unless
            // they list more candidates than the dense list holds; then as many
            // as fit, and the others in further passes.
            int wlo = 0;
            for (int q = 0; q < P.n_q;) {
                // (values derived from the lane index and from the events'
                // ranges are recomputed per query rather than held across the
                // query loop, where they would spill)
                asm volatile("" : "+v"(lane));
#pragma unroll
                for (int r = 0; r < EVPL; ++r) {
                    asm volatile("" : "+v"(jb[r]), "+v"(je[r]), "+v"(mb[r]), "+v"(me[r]), "+v"(wv[r]));
                    if (EXT) asm volatile("" : "+v"(lb[r]), "+v"(le[r]));
                }
                // the query's fields are read in place (scalar loads near their
                // uses) rather than copied: a copy would hold ~45 SGPRs for the
                // whole query and spill
                const auto &Q = as_const(P.qs)[q];
                if (!Q.active) {
                    ++q;
                    continue;
                }
                // the query's cut constants, read once and pinned by one
                // statement (loads issued together, one wait; unpinned, the
                // compiler reloads them inside the loops below, a wait each)
                float mu_pt = Q.mu_pt, mu_abseta = Q.mu_abseta, mu_iso = Q.mu_iso;
                float el_pt = EXT ? Q.el_pt : 0.0f, el_abseta = EXT ? Q.el_abseta : 0.0f;
                float jet_pt = Q.jet_pt, thr2 = Q.thr2, jet_abseta = Q.jet_abseta, smax = Q.smax, ptmin = Q.ptmin;
                float btag = EXT ? Q.btag : 0.0f;
                int min_mu = Q.min_mu, min_jet = Q.min_jet, min_b = has_bt ? Q.min_b : 0;
                asm volatile(""
                             : "+s"(mu_pt), "+s"(mu_abseta), "+s"(mu_iso), "+s"(el_pt), "+s"(el_abseta),
                               "+s"(jet_pt), "+s"(thr2), "+s"(jet_abseta), "+s"(smax), "+s"(ptmin), "+s"(btag),
                               "+s"(min_mu), "+s"(min_jet), "+s"(min_b));
                // lookup corrections of this query (LK kernels): which are on,
                // the tables as axes over the edge table
                const bool use_pu = LK && Q.pu_nb > 0 && D.npu != nullptr;
                const bool use_sf = LK && Q.sf_nb > 0;
                const bool shift = LK && Q.jes_mode == 1;
                // ---- 2. lepton selection; selected leptons compacted into LDS
                // (all compares evaluated: no branches per slot)
                {
                    bool sel[MK];
#pragma unroll
                    for (int k = 0; k < MK; ++k)
                        sel[k] = (lane + 64 * k < nm) & (mpt[k] > mu_pt) &
                                 (fabsf(meta[k]) < mu_abseta) &
                                 (!has_iso | (miso[k] < mu_iso));
                    if (use_sf) {
                        // the selected muons' pt, compacted beside them and
                        // then replaced by their scale factors, a lane per
                        // selected muon (one round where the slots take MK)
                        const int ns = compact<MK, true>(sel, meta, mphi, lane, L.seta, L.sphi, L.u.p.mpre,
                                                            mpt, L.u.p.ssf);
                        wave_sync();
                        on_tables([&](const float *E) {
                            const Axis ax = lk_axes(Q, E).sf;
                            for (int i = lane; i < ns; i += 64) {
                                const float x[1] = {L.u.p.ssf[LK ? i : 0]};
                                const bool use[1] = {true};
                                float f[1];
                                lookup_bin_n<1>(ax, E + Q.sf_c, x, use, f, false);
                                L.u.p.ssf[LK ? i : 0] = f[0];
                            }
                        });
                    } else {
                        int ns = compact<MK, false>(sel, meta, mphi, lane, L.seta, L.sphi, L.u.p.mpre);
                        if (MX > 0 && __builtin_expect(nm > 64 * MK, 0)) {
                            // the muons beyond the registers, from memory
                            const uint32_t es = sizeof(T), mb_ = static_cast<uint32_t>(nm) * es;
                            const int m = lane + 64 * MK;
                            const uint32_t rpt = buf_raw<T>(buf_span(static_cast<const T *>(D.mpt) + B.M0, mb_), m);
                            const uint32_t reta = buf_raw<T>(buf_span(static_cast<const T *>(D.meta) + B.M0, mb_), m);
                            const uint32_t rphi = buf_raw<T>(buf_span(static_cast<const T *>(D.mphi) + B.M0, mb_), m);
                            const uint32_t riso =
                                has_iso ? buf_raw<T>(buf_span(static_cast<const T *>(D.miso) + B.M0, mb_), m) : 0u;
                            const float eta = raw_f<T>(reta);
                            const bool s = (m < nm) & (raw_f<T>(rpt) > mu_pt) & (fabsf(eta) < mu_abseta) &
                                           (!has_iso | (raw_f<T>(riso) < mu_iso));
                            const uint64_t bal = __ballot(s);
                            const int before = bits_below(bal, ns);
                            L.u.p.mpre[m] = static_cast<uint16_t>(before);
                            if (s) {
                                L.seta[before] = static_cast<TL>(eta);
                                L.sphi[before] = static_cast<TL>(raw_f<T>(rphi));
                            }
                            ns += __popcll(bal);
                            L.u.p.mpre[64 * (MK + 1)] = static_cast<uint16_t>(ns);
                        }
                    }
                }
                if (EXT) {
                    bool sel[EK];
#pragma unroll
                    for (int k = 0; k < EK; ++k)
                        sel[k] = (lane + 64 * k < nl) & (lpt[k] > el_pt) &
                                 (fabsf(leta[k]) < el_abseta);
                    compact<EK, false>(sel, leta, lphi, lane, L.seta + (C::MC + 2), L.sphi + (C::MC + 2),
                                          L.u.p.epre);
                }
                // ---- 3. candidate jets -- inside |eta| and, by ptmin, able to
                // pass jet_pt at some scale -- as one mask per slot, and the
                // number of candidates (b-tagged candidates) before every jet
                uint64_t okm[JK];
                {
                    int runc = 0, runt = 0;
#pragma unroll
                    for (int k = 0; k < JK; ++k) {
                        const int j = lane + 64 * k;
                        const bool ok = (j < nj) & (fabsf(jeta[k]) < jet_abseta) &
                                        (jpt[k] >= ptmin);
                        okm[k] = __ballot(ok);
                        uint32_t before = static_cast<uint32_t>(bits_below(okm[k], runc));
                        runc += __popcll(okm[k]);
                        if (EXT) {
                            const uint64_t tg = __ballot(ok & has_bt & (jbt[EXT ? k : 0] > btag));
                            before |= static_cast<uint32_t>(bits_below(tg, runt)) << 16;
                            runt += __popcll(tg);
                        }
                        cpre[j] = static_cast<cpre_t<EXT>>(before);
                    }
                    cpre[C::JC] = static_cast<cpre_t<EXT>>(static_cast<uint32_t>(runc) |
                                                             (EXT ? static_cast<uint32_t>(runt) << 16 : 0u));
                }
                if (lane < 4 * JK) reinterpret_cast<uint32_t *>(L.em)[lane] = 0u;
                wave_sync();
                // each event's selected-lepton ranges (first | count << 16) and
                // (below) its weight
                int nmu[EVPL];
                uint32_t rmu[EVPL], rel[EVPL];
                float wq[EVPL];
#pragma unroll
                for (int r = 0; r < EVPL; ++r) {
                    const int s0 = L.u.p.mpre[mb[r]];
                    nmu[r] = L.u.p.mpre[me[r]] - s0;
                    rmu[r] = static_cast<uint32_t>(s0) | (static_cast<uint32_t>(nmu[r]) << 16);
                    rel[r] = 0u;
                    if (EXT) {
                        const int u0 = L.u.p.epre[EXT ? lb[r] : 0];
                        rel[r] = static_cast<uint32_t>(u0) |
                                 (static_cast<uint32_t>(L.u.p.epre[EXT ? le[r] : 0] - u0) << 16);
                    }
                }
                // the events that can still pass: every jet selected at any
                // scale is a candidate, and the cone test only removes jets.
                // Their candidates get consecutive places of the dense list.
                // (The record kernels keep to the documented skip reasons.)
                bool elig[EVPL];
                int cnt[EVPL], start[EVPL];
                int total = 0;
                bool some = false;
#pragma unroll
                for (int r = 0; r < EVPL; ++r) {
                    const uint32_t cw0 = cpre[jb[r]], cw1 = cpre[je[r]];
                    const int nc = static_cast<int>((cw1 & 0xffffu) - (cw0 & 0xffffu));
                    elig[r] = (lane + 64 * r < ne) & (nmu[r] >= min_mu) & (je[r] - jb[r] >= min_jet) &
                              (lane + 64 * r >= wlo);
                    if (!DBG)
                        elig[r] = elig[r] & (nc >= min_jet) &
                                  (!EXT | (static_cast<int>((cw1 >> 16) - (cw0 >> 16)) >= min_b));
                    wq[r] = wv[r];
                    if (LK && (DBG || elig[r])) {
                        if (use_pu)
                            on_tables([&](const float *E) {
                                wq[r] = wq[r] * lookup_bin(lk_axes(Q, E).pu, E + Q.pu_c, R.npu[LK ? r : 0]);
                            });
                        if (use_sf) {
                            // product of the selected muons' scale factors, in order from 1
                            float prod = 1.0f;
                            const int s0 = static_cast<int>(rmu[r] & 0xffffu);
                            for (int i = s0; i < s0 + nmu[r]; ++i) prod = prod * L.u.p.ssf[LK ? i : 0];
                            wq[r] = wq[r] * prod;
                        }
                    }
                    cnt[r] = elig[r] ? nc : 0;
                    const int incl = wave_prefix_sum(cnt[r]);
                    start[r] = total + incl - cnt[r];
                    total += __builtin_amdgcn_readlane(incl, 63);
                    some |= elig[r];
                    if (DBG && lane + 64 * r < ne && lane + 64 * r >= wlo) {
                        // the muon count and weight of every event; the rest
                        // only of events that are not walked (the walk writes
                        // the other fields of walked events' records)
                        for (int v = 0; v < Q.n_scale; ++v) {
                            hepk_event_record *o = rec_at(P, Q.scale0 + v, D.ev0 + e0 + lane + 64 * r);
                            o->n_mu = nmu[r];
                            o->w = wq[r];
                            o->reserved = 0;
                            if (!elig[r]) {
                                o->n_jet = 0;
                                o->n_b = 0;
                                o->state = 1;
                                o->ht = 0.0f;
                                o->lead = -INFINITY;
                            }
                        }
                    }
                }
                int whi = TW;
                if (total > cap) {
                    // the events up to the first that does not fit (every event
                    // lists at most cap, so the first one always fits)
                    int fit_total = total;
                    some = false;
#pragma unroll
                    for (int r = EVPL - 1; r >= 0; --r) {
                        const bool fit = start[r] + cnt[r] <= cap;
                        const int nf = __popcll(__ballot(fit));
                        if (nf < 64) {
                            whi = 64 * r + nf;
                            fit_total = __builtin_amdgcn_readlane(start[r], nf);
                        }
                        elig[r] = elig[r] & fit;
                        cnt[r] = fit ? cnt[r] : 0;
                        some |= elig[r];
                    }
                    total = fit_total;
                }
                // their jets' bits
#pragma unroll
                for (int r = 0; r < EVPL; ++r)
                    if (cnt[r] > 0) {
                        const int ja = jb[r], jz = je[r] - 1;
                        const int wa = ja >> 6, wz = jz >> 6;
                        const uint64_t lo = ~uint64_t(0) << (ja & 63), hi = ~uint64_t(0) >> (63 - (jz & 63));
                        or_u64(&L.em[wa], wa == wz ? lo & hi : lo);
                        if (wa != wz) {
                            for (int w = wa + 1; w < wz; ++w) or_u64(&L.em[w], ~uint64_t(0));
                            or_u64(&L.em[wz], hi);
                        }
                    }
                const bool any_ev = __ballot(some) != 0;
                const bool last_pass = whi >= ne;
                // With one scale and jet_pt >= 0 (zsel) the cone test decides
                // the whole jet selection, so a kept jet is stored as pt * s
                // and a removed one as +0, for walk_selected.
                const bool zsel = !MS && jet_pt >= 0.0f;
                if (any_ev) {
                    // ---- 4. the lepton ranges of the events with candidates, in
                    // order, and the first candidate of each as a bit
                    int nrec = 0;
#pragma unroll
                    for (int r = 0; r < EVPL; ++r) {
                        const bool has = cnt[r] > 0;
                        const uint64_t b = __ballot(has);
                        const int o = bits_below(b, nrec);
                        if (has) {
                            L.u.r.mu[o] = rmu[r];
                            if (EXT) L.u.r.el[EXT ? o : 0] = rel[r];
                            or_u64(&L.em[L.SM + (start[r] >> 6)], uint64_t(1) << (start[r] & 63));
                        }
                        nrec += __popcll(b);
                    }
                    // their candidates, in tile order (the bits below were set
                    // by other lanes, and the list takes the place of cpre)
                    wave_sync();
                    int run = 0;
                    // (the bits of all slots in one read, a 32-bit word per lane)
                    const uint32_t ew = reinterpret_cast<const uint32_t *>(L.em)[lane & 31];
                    const float f = (zsel && !shift) ? smax : 1.0f;
#pragma unroll
                    for (int k = 0; k < JK; ++k) {
                        const uint64_t d = okm[k] & lane_u64(ew, 2 * k);
                        const int dst = bits_below(d, run);
                        if (__builtin_amdgcn_inverse_ballot_w64(d)) {
                            cand[dst].pt = jpt[k] * f;
                            cand[dst].eta = static_cast<TL>(jeta[k]);
                            cand[dst].phi = static_cast<TL>(jphi[k]);
                            if (EXT) cbt[dst] = (has_bt & (jbt[EXT ? k : 0] > btag)) ? 1 : 0;
                        }
                        run += __popcll(d);
                    }
                    wave_sync();
                    // the cone test, a lane per candidate, CB groups of 64 at a
                    // time (each step's LDS reads of all groups in flight
                    // together): the candidate's event is the number of first-
                    // candidate bits up to its own; its leptons are the
                    // event's selected muons, then (EXT) its selected
                    // electrons: lepton i is seta[s0 + i] for i < nmu, else
                    // seta[EO + u0 + i - nmu].  The first two are tested
                    // without a branch (reads past a range's end land on other
                    // leptons or on the padding entries and are unused); only
                    // events with more loop over the rest.
                    constexpr int EO = C::MC + 2;
                    const uint32_t sv = reinterpret_cast<const uint32_t *>(L.em + L.SM)[lane & 31];
                    int ord0 = -1;  // events that start before the group, minus one
                    auto cone = [&](auto cb, int p0) __attribute__((always_inline)) {
                        constexpr int CB = decltype(cb)::value;
                        uint32_t wm[CB], we[CB];
                        float eta[CB], phi[CB], pt[CB], dsh[CB];
#pragma unroll
                        for (int b = 0; b < CB; ++b) {
                            const uint64_t sw = lane_u64(sv, 2 * ((p0 >> 6) + b));
                            const int o = bits_below(sw >> 1, ord0 + static_cast<int>(sw & 1u));
                            ord0 += __popcll(sw);
                            const int p = p0 + 64 * b + lane;
                            wm[b] = L.u.r.mu[o];
                            we[b] = EXT ? L.u.r.el[EXT ? o : 0] : 0u;
                            eta[b] = static_cast<float>(cand[p].eta);
                            phi[b] = static_cast<float>(cand[p].phi);
                            pt[b] = LK ? cand[p].pt : 0.0f;
                            dsh[b] = 0.0f;
                        }
                        if constexpr (LK) {  // (before the leptons are read: fewer registers live)
                            if (shift)
                                on_tables([&](const float *E) {
                                    if (Q.jseg >= 0)
                                        jes_lut_n<CB>(Q, E, pt, eta, dsh);
                                    else
                                        jes_shift_n<CB>(lk_axes(Q, E), E, Q.jd, pt, eta, dsh);
                                });
                        }
                        int s0[CB], nm_[CB], ofe[CB], nlep[CB];
                        float e0[CB], f0[CB], e1[CB], f1[CB];
#pragma unroll
                        for (int b = 0; b < CB; ++b) {
                            s0[b] = static_cast<int>(wm[b] & 0xffffu);
                            nm_[b] = static_cast<int>(wm[b] >> 16);
                            ofe[b] = EXT ? EO + static_cast<int>(we[b] & 0xffffu) - nm_[b] : s0[b];
                            nlep[b] = nm_[b] + static_cast<int>(we[b] >> 16);
                            const int i0 = (!EXT || nm_[b] >= 1) ? s0[b] : ofe[b];
                            const int i1 = (!EXT || nm_[b] >= 2) ? s0[b] + 1 : ofe[b] + 1;
                            e0[b] = ldf(L.seta, i0);
                            f0[b] = ldf(L.sphi, i0);
                            e1[b] = ldf(L.seta, i1);
                            f1[b] = ldf(L.sphi, i1);
                        }
#pragma unroll
                        for (int b = 0; b < CB; ++b) {
                            const int p = p0 + 64 * b + lane;
                            const bool live = p < total;
                            const int cn = live ? nlep[b] : 0;
                            bool hit = ((cn >= 1) & (delta_r2(eta[b], phi[b], e0[b], f0[b]) <= thr2)) |
                                       ((cn >= 2) & (delta_r2(eta[b], phi[b], e1[b], f1[b]) <= thr2));
                            const int sm = s0[b], nm2 = nm_[b], oe = ofe[b];
                            auto lidx = [&](int i) { return (!EXT || i < nm2) ? sm + i : oe + i; };
                            int i = 2;
                            // two leptons per step: both LDS reads in flight before the math
                            for (; i + 2 <= cn; i += 2) {
                                const int ia = lidx(i), ib = lidx(i + 1);
                                const float ea = ldf(L.seta, ia), pa = ldf(L.sphi, ia), eb = ldf(L.seta, ib),
                                            pb = ldf(L.sphi, ib);
                                hit |= delta_r2(eta[b], phi[b], ea, pa) <= thr2;
                                hit |= delta_r2(eta[b], phi[b], eb, pb) <= thr2;
                            }
                            if (i < cn) {
                                const int ia = lidx(i);
                                hit |= delta_r2(eta[b], phi[b], ldf(L.seta, ia), ldf(L.sphi, ia)) <= thr2;
                            }
                            if (LK && shift) {
                                if (!live) continue;
                                if (zsel) {
                                    // one scale s (= smax): the jet's energy pt * (1 + s * d)
                                    const float x = pt[b] * (1.0f + smax * dsh[b]);
                                    const bool sel = !hit & (x > jet_pt);
                                    cand[p].pt = sel ? x : 0.0f;
                                    if (EXT && !sel) cbt[p] = 0;
                                } else {
                                    // (an energy not above jet_pt at any scale is
                                    // removed too: the records count it so)
                                    if (DBG && jet_pt >= 0.0f)
                                        hit |= !(shifted_pt_bound(pt[b], dsh[b], Q.smin, smax) > jet_pt);
                                    if constexpr (LK) cand[p].jd = dsh[b];
                                    if (hit) cand[p].pt = __builtin_nanf("");
                                }
                            } else if (live & hit) {
                                cand[p].pt = zsel ? 0.0f : __builtin_nanf("");
                                if (EXT) cbt[p] = 0;
                            }
                        }
                    };
                    for (int p0 = 0; p0 < total; p0 += 128) {
                        if (total - p0 > 64)
                            cone(std::integral_constant<int, 2>{}, p0);
                        else
                            cone(std::integral_constant<int, 1>{}, p0);
                    }
                    wave_sync();
                    // ---- 5. per-event reductions, event cut, fills
                    if (ht_can_be_nan(jet_pt)) {
                        // a lane per event, scale by scale, fills that test for
                        // NaN (tests in the fills below cost 20 scales 4%); an
                        // index of its own, so the fields are not held here
                        // for the fills below
                        int qn = q;
                        asm volatile("" : "+s"(qn));
                        const auto &N = as_const(P.qs)[qn];
#pragma unroll
                        for (int r = 0; r < EVPL; ++r) {
                            if (!elig[r]) continue;
                            for (int v = 0; v < N.n_scale; ++v) {
                                const float sc[1] = {as_const(P.scales)[N.scale0 + v]};
                                float ht[1], lead[1];
                                int njs[1], nbt[1];
                                if (shift)
                                    walk_jets<1, EXT, LK>(cand, cbt, start[r], start[r] + cnt[r], sc, jet_pt, ht, lead, njs, nbt);
                                else
                                    walk_jets<1, EXT, false>(cand, cbt, start[r], start[r] + cnt[r], sc, jet_pt, ht, lead, njs, nbt);
                                const bool pass = njs[0] >= min_jet && nbt[0] >= min_b;
                                if (DBG)
                                    *rec_at(P, N.scale0 + v, D.ev0 + e0 + lane + 64 * r) = hepk_event_record{
                                        nmu[r], njs[0], nbt[0], pass ? 3 : 2, ht[0], lead[0], wq[r], 0};
                                if (pass) fill3(sink, N, P.edges, v, ht[0], lead[0], njs[0], static_cast<double>(wq[r]));
                            }
                        }
                    }
                    const FillC F = fill_consts<LDSH>(Q);
                    // separate calls for the two places the edges live, so each
                    // knows its address space (no flat loads)
                    const int vlast = Q.n_scale - 1;
                    auto fill = [&](const auto &xs, const auto &pass, int v0, double w) __attribute__((always_inline)) {
                        constexpr int N = std::extent<std::remove_reference_t<decltype(xs)>>::value;
                        if (P.edges_in_lds)
                            fill_bins<N, MS>(sink, F, Q, e_s, xs, pass, v0, w, vlast);
                        else
                            fill_bins<N, MS>(sink, F, Q, P.edges, xs, pass, v0, w, vlast);
                    };
                    if (ht_can_be_nan(jet_pt)) {
                        // (filled above)
                    } else if (!MS) {
                        const float sc[1] = {pin<float>(as_const(P.scales)[Q.scale0])};
#pragma unroll
                        for (int r = 0; r < EVPL; ++r) {
                            float ht[1], lead[1];
                            int njs[1], nbt[1];
                            const int k0 = start[r], k1 = k0 + cnt[r];  // (empty unless elig)
                            if (zsel)
                                walk_selected<EXT>(cand, cbt, k0, k1, ht[0], lead[0], njs[0], nbt[0]);
                            else if (shift)
                                walk_jets<1, EXT, LK>(cand, cbt, k0, k1, sc, jet_pt, ht, lead, njs, nbt);
                            else
                                walk_jets<1, EXT, false>(cand, cbt, k0, k1, sc, jet_pt, ht, lead, njs, nbt);
                            const bool pass[1] = {elig[r] && njs[0] >= min_jet && nbt[0] >= min_b};
                            if (DBG && elig[r])
                                *rec_at(P, Q.scale0, D.ev0 + e0 + lane + 64 * r) = hepk_event_record{
                                    nmu[r], njs[0], nbt[0], pass[0] ? 3 : 2, ht[0], lead[0], wq[r], 0};
                            if (pass[0]) {
                                const float xs[3] = {ht[0], lead[0], static_cast<float>(njs[0])};
                                fill(xs, pass, 0, static_cast<double>(wq[r]));
                            }
                        }
                    } else {
                        // Several scales: the events that can pass are compacted, and
                        // lanes take (event, group of kG scales) pairs of them,
                        // event-major.  One walk over an event's candidates
                        // serves the kG scales of its group (kG independent
                        // chains), and one pass of the lanes covers a few
                        // events, so the walks diverge little.
                        int nel = 0;
#pragma unroll
                        for (int r = 0; r < EVPL; ++r) {
                            bool in = elig[r];
                            const int k0 = start[r], k1 = k0 + cnt[r];
                            if (DBG && jet_pt >= 0.0f && in) {
                                // the records tell the events short of jets or
                                // b-tagged jets at the largest scale apart
                                int kj = 0, kb = 0;
                                for (int k = k0; k < k1; ++k) {
                                    const bool kept = cand[k].pt == cand[k].pt;
                                    kj += kept ? 1 : 0;
                                    kb += (EXT && kept) ? cbt[k] : 0;
                                }
                                in = kj >= min_jet && kb >= min_b;
                                for (int v = 0; v < Q.n_scale && !in; ++v) {
                                    hepk_event_record *o = rec_at(P, Q.scale0 + v, D.ev0 + e0 + lane + 64 * r);
                                    o->n_jet = 0;
                                    o->n_b = 0;
                                    o->state = 1;
                                    o->ht = 0.0f;
                                    o->lead = -INFINITY;
                                }
                            }
                            const uint64_t bal = __ballot(in);
                            const int at = bits_below(bal, nel);
                            if (in) {
                                // candidate range: first in bits 0-9, end in bits
                                // 16-25 (both at most JC < 2^10); DBG kernels
                                // keep the event's place in the tile in the bits
                                // between
                                const uint32_t ev = static_cast<uint32_t>(lane + 64 * r);
                                L.u.w.evjr[at] = static_cast<uint32_t>(k0) | (static_cast<uint32_t>(k1) << 16) |
                                                 (DBG ? (((ev & 63u) << 10) | ((ev >> 6) << 26)) : 0u);
                                L.u.w.evw[at] = wq[r];
                            }
                            nel += __popcll(bal);
                        }
                        wave_sync();
                        int V = Q.n_scale, scale0 = Q.scale0;
                        asm volatile("" : "+s"(V), "+s"(scale0));
                        const float *scl = (P.scales_in_lds ? s_s : P.scales) + scale0;
                        const int NG = (V + kG - 1) / kG;
                        const int npairs = nel * NG;
                        int e = lane / NG, g = lane - (lane / NG) * NG;
                        const int de = 64 / NG, dg = 64 - (64 / NG) * NG;
                        for (int i = lane; i < npairs; i += 64) {
                            const uint32_t jr = L.u.w.evjr[e];
                            float sc[kG];
#pragma unroll
                            for (int u = 0; u < kG; ++u) sc[u] = scl[min(g * kG + u, V - 1)];
                            float ht[kG], lead[kG];
                            int njs[kG], nbt[kG];
                            const int wj0 = static_cast<int>(jr & 0x3ffu), wj1 = static_cast<int>((jr >> 16) & 0x3ffu);
                            if (shift)
                                walk_jets<kG, EXT, LK>(cand, cbt, wj0, wj1, sc, jet_pt, ht, lead, njs, nbt);
                            else
                                walk_jets<kG, EXT, false>(cand, cbt, wj0, wj1, sc, jet_pt, ht, lead, njs, nbt);
                            bool pass[kG], any = false;
#pragma unroll
                            for (int u = 0; u < kG; ++u) {
                                pass[u] = g * kG + u < V && njs[u] >= min_jet && nbt[u] >= min_b;
                                any |= pass[u];
                            }
                            if (DBG) {
                                const int64_t ge = D.ev0 + e0 + (((jr >> 10) & 63u) | ((jr >> 26) << 6));
#pragma unroll
                                for (int u = 0; u < kG; ++u) {
                                    if (g * kG + u >= V) continue;
                                    hepk_event_record *o = rec_at(P, scale0 + g * kG + u, ge);
                                    o->n_jet = njs[u];
                                    o->n_b = nbt[u];
                                    o->state = pass[u] ? 3 : 2;
                                    o->ht = ht[u];
                                    o->lead = lead[u];
                                }
                            }
                            if (any) {
                                // FS scales' bins per search: the batch that fits
                                // the registers without spilling
                                constexpr int FS = 2;
                                const double w = static_cast<double>(L.u.w.evw[e]);
#pragma unroll
                                for (int u = 0; u < kG; u += FS) {
                                    float xs[3 * FS];
                                    bool pu[FS], anyu = false;
#pragma unroll
                                    for (int t = 0; t < FS; ++t) {
                                        xs[3 * t] = ht[u + t];
                                        xs[3 * t + 1] = lead[u + t];
                                        xs[3 * t + 2] = static_cast<float>(njs[u + t]);
                                        pu[t] = pass[u + t];
                                        anyu |= pu[t];
                                    }
                                    if (anyu) fill(xs, pu, g * kG + u, w);
                                }
                            }
                            e += de;
                            g += dg;
                            if (g >= NG) {
                                g -= NG;
                                e += 1;
                            }
                        }
                    }
                }
                if (last_pass) {
                    wlo = 0;
                    ++q;
                } else {
                    wlo = whi;
                }
                wave_sync();
            }
        };
        // Tile bounds are fetched one tile ahead (scalar loads that overlap
        // the current tile's vector loads).  A tile whose objects exceed the
        // register capacity runs as consecutive sub-tiles: from its first
        // event not yet run, the event count is halved until the objects fit
        // (a few scalar loads), that sub-tile runs like a tile, and the rest
        // of the tile follows.  Only a single event beyond the capacity, or
        // with more candidates than the dense list holds, goes straight from
        // HBM.
        int r = wave;  // this wavefront's tile (relative to c_t0)
        int eo = 0;    // events of tile r already run
        TileBounds nb{};
        if (r < nt) nb = bounds_of(r);
        while (r < nt) {
            // the lane index is re-read here so that values derived from it
            // are recomputed per tile instead of held (and spilled) across it
            asm volatile("" : "+v"(lane));
            const int tn = tile_events(r);
            const int64_t e = ebase + static_cast<int64_t>(r) * TW + eo;
            int n = tn - eo;
            TileBounds B;
            if (eo == 0) {
                B = nb;
                if (r + WAVES < nt) nb = bounds_of(r + WAVES);
            } else {
                B = tile_bounds<EXT>(D, has_el, e, n);
            }
            while (n > 1 && oversize(B)) {
                n = (n + 1) >> 1;
                B = tile_bounds<EXT>(D, has_el, e, n);
            }
            // (the loads are issued also of a single event beyond the
            // registers -- of no object -- so that one path defines R)
            const bool over = oversize(B);
            if (over) B.nj = B.nm = B.nl = 0;
            Raw R;
            issue(e, n, B, R);
            settle(R);
            // of the events with more jets than the dense list holds, the first
            // that lists too many for some query ends the sub-tile or, as its
            // first event, goes alone
            bool direct = over;
#pragma unroll
            for (int i = 0; i < EVPL; ++i) {
                uint64_t lb = __ballot((lane + 64 * i < n) & (R.j1[i] - R.j0[i] > static_cast<uint32_t>(cap)));
                for (; lb != 0 && !over; lb &= lb - 1) {
                    const int l = __builtin_ctzll(lb);
                    const int ja = static_cast<int>(__builtin_amdgcn_readlane(R.j0[i], l) - static_cast<uint32_t>(B.J0));
                    const int jz = static_cast<int>(__builtin_amdgcn_readlane(R.j1[i], l) - static_cast<uint32_t>(B.J0));
                    bool beyond = false;
                    for (int q = 0; q < P.n_q; ++q) {
                        const auto &Q = as_const(P.qs)[q];
                        int nc = 0;
#pragma unroll
                        for (int k = 0; k < JK; ++k) {
                            const int j = lane + 64 * k;
                            nc += __popcll(__ballot((j >= ja) & (j < jz) & (fabsf(raw_f<T>(R.jeta[k])) < Q.jet_abseta) &
                                                    (raw_f<T>(R.jpt[k]) >= Q.ptmin)));
                        }
                        beyond |= (nc > cap) & (Q.active != 0);
                    }
                    if (beyond) {
                        direct = 64 * i + l == 0;
                        n = direct ? 1 : 64 * i + l;
                        break;
                    }
                }
            }
            if (direct) {
                const DsDev Dc = D;
                event_direct<T, EXT, LDSH, DBG, LK>(P, Dc, e, lane, edges, sink);
            } else {
                work(e, n, B, R);
            }
            // the next (sub-)tile; nb holds the bounds of tile r + WAVES
            // whenever it starts a tile
            eo += n;
            if (eo >= tn) {
                r += WAVES;
                eo = 0;
            }
        }
        // merge the LDS histograms into the dataset's block in HBM (the next
        // chunk, if any, is another dataset)
        if (LDSH) {
            __syncthreads();
            for (int q = 0; q < P.n_q; ++q) {
                const QDev Q = as_const(P.qs)[q];
                if (!Q.active) continue;
                // all of the query's histograms as one run of LDS slots (a loop
                // over 60 short histograms was 60 dependent LDS round trips:
                // 1e4 events with 20 scales 26 -> 19 us, with lookups 42 -> 33);
                // the place in HBM from the slot's scale and observable
                const int per = Q.lper_scale, n = per * Q.n_scale;
                for (int i = tid; i < n; i += 64 * WAVES) {
                    const int ls = Q.lslot0 + i;
                    const uint32_t c = c_s[ls];
                    if (c) {
                        const int v = i / per, k = i - v * per;
                        const int h = (k >= Q.lhoff[1] ? 1 : 0) + (k >= Q.lhoff[2] ? 1 : 0);
                        const int lh = h == 0 ? Q.lhoff[0] : (h == 1 ? Q.lhoff[1] : Q.lhoff[2]);
                        const int gh = h == 0 ? Q.ghoff[0] : (h == 1 ? Q.ghoff[1] : Q.ghoff[2]);
                        const int64_t gs = D.hist0 + Q.gslot0 + v * Q.gper_scale + gh + (k - lh);
                        atomic_add_u64(&P.counts[gs], c);
                        atomic_add_f64(&P.sumw[gs], sw_s[ls]);
                        if (LK && P.sumw2) atomic_add_f64(&P.sumw2[gs], sw2_s[ls]);
                        c_s[ls] = 0u;
                        sw_s[ls] = 0.0;
                        if (LK) sw2_s[ls] = 0.0;
                    }
                }
            }
            __syncthreads();
        }
    }
}

using KernelFn = void (*)(PipeArgs);

template <typename T, bool EXT, int WAVES, int EVPL, bool LDSH, bool MS, bool DBG, bool LK>
static KernelFn kfn() {
    return reinterpret_cast<KernelFn>(&pipeline_kernel<T, EXT, WAVES, EVPL, LDSH, MS, DBG, LK>);
}

template <typename T, bool EXT, int WAVES, int EVPL, bool MS, bool DBG, bool LK>
static KernelFn pick_h(bool ldsh) {
    return ldsh ? kfn<T, EXT, WAVES, EVPL, true, MS, DBG, LK>() : kfn<T, EXT, WAVES, EVPL, false, MS, DBG, LK>();
}

// LK kernels exist for one event per thread only (the plan takes that shape
// for queries with lookups).
template <typename T, bool EXT, bool MS, bool DBG, bool LK>
static KernelFn pick_shape(int block, int evpt, bool ldsh) {
    if (block == 1024) return pick_h<T, EXT, 16, 1, MS, DBG, LK>(ldsh);  // one event per thread only
    if constexpr (!LK) {
        if (evpt == 2) return block == 512 ? pick_h<T, EXT, 8, 2, MS, DBG, LK>(ldsh) : pick_h<T, EXT, 4, 2, MS, DBG, LK>(ldsh);
    }
    return block == 512 ? pick_h<T, EXT, 8, 1, MS, DBG, LK>(ldsh) : pick_h<T, EXT, 4, 1, MS, DBG, LK>(ldsh);
}

// The kernel for a launch shape; each (MS, DBG, LK) triple is instantiated
// in its own translation unit (they compile in parallel).
template <bool MS, bool DBG, bool LK>
KernelFn pick_kernel(int dtype, bool ext, int block, int evpt, bool ldsh) {
    if (dtype == HEPK_F16) return ext ? pick_shape<_Float16, true, MS, DBG, LK>(block, evpt, ldsh)
                                      : pick_shape<_Float16, false, MS, DBG, LK>(block, evpt, ldsh);
    return ext ? pick_shape<float, true, MS, DBG, LK>(block, evpt, ldsh)
               : pick_shape<float, false, MS, DBG, LK>(block, evpt, ldsh);
}

// LDS for the workgroup's private histograms: up to 144 KiB (60 histograms of
// 100 bins with squared weights fit), as long as the workgroup's total fits
// the device; larger sets go to global atomics.  More LDS lowers occupancy,
// which the launch-configuration search weighs against atomic contention.
constexpr int kMaxLdsHistBytes = 144 * 1024;
constexpr int kMaxLdsEdgeBytes = 4 * 1024;
constexpr int kMaxLdsLookupBytes = 8 * 1024;  // with lookup tables
constexpr int kMaxLdsScaleBytes = 1024;

}  // namespace hepk
