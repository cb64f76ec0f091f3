// Positional kernels over jagged collections (Sec. III): get_in_offsets and
// set_in_offsets retrieve or set the n-th selected element of every event,
// select_opposite_sign_muons keeps per event the first two objects in pT
// order with opposite charges, and compaction gathers the selected objects
// into a contiguous collection laid out by the offsets of their counts.
//
// get/set touch a few bytes per event: one lane per event walks its objects
// (consecutive lanes read consecutive events' bytes, so the loads of a
// wavefront share cache lines).  The opposite-sign selection stages tiles of
// 64 events.  Compaction moves every selected element: each wavefront owns tiles of 64
// consecutive events, takes their objects 64 at a time in order, and places
// the kept ones by a wavefront ballot and prefix count, so both its reads and
// its writes are contiguous runs.
#include "common.hpp"

namespace hepk {

// Workgroups per CU, at most: a sweep of 8-64 put the best at 64 (get/set 7%,
// opposite-sign pairs 4% faster than 16).
constexpr int kTileWgPerCu = 64;

constexpr int PB = 256;

// Content index of the n-th (from 0) object of [i0, i1) with m set (every
// object when m is NULL); -1 when there are fewer.
// The first kNthBatch mask bytes are read in one batch (indices clamped
// into the range, so no read waits on another); only a range whose n-th
// selected object lies beyond them goes on byte by byte.
constexpr int kNthBatch = 8;
__device__ __forceinline__ int64_t nth_selected(int64_t i0, int64_t i1, const uint8_t *m, int32_t n) {
    if (n < 0) return -1;
    if (!m) return (n < i1 - i0) ? i0 + n : -1;
    const int64_t len = i1 - i0;
    if (len <= 0) return -1;
    uint32_t b[kNthBatch];
#pragma unroll
    for (int k = 0; k < kNthBatch; ++k) b[k] = m[i0 + min<int64_t>(k, len - 1)];
    int32_t seen = 0;
    int64_t found = -1;
#pragma unroll
    for (int k = 0; k < kNthBatch; ++k) {
        const bool hit = k < len && b[k] != 0u;
        found = (hit && seen == n && found < 0) ? i0 + k : found;
        seen += hit ? 1 : 0;
    }
    if (found >= 0 || len <= kNthBatch) return found;
    for (int64_t i = i0 + kNthBatch; i < i1; ++i) {
        if (!m[i]) continue;
        if (seen == n) return i;
        ++seen;
    }
    return -1;
}

template <typename T>
__global__ __launch_bounds__(PB) void get_in_offsets_kernel(const int64_t *__restrict__ off, int64_t n_events,
                                                            const T *__restrict__ content,
                                                            const uint8_t *__restrict__ om,
                                                            const uint8_t *__restrict__ em,
                                                            const int32_t *__restrict__ idx, int32_t n, float fill,
                                                            float *__restrict__ out, int32_t *__restrict__ out_index) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * PB;
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * PB + threadIdx.x; e < n_events; e += stride) {
        const int64_t i0 = off[e], i1 = off[e + 1];
        int64_t i = -1;
        if (!em || em[e]) i = nth_selected(i0, i1, om, idx ? idx[e] : n);
        out[e] = i >= 0 ? ldf(content, i) : fill;
        if (out_index) out_index[e] = i >= 0 ? static_cast<int32_t>(i - i0) : -1;
    }
}

template <typename T>
__global__ __launch_bounds__(PB) void set_in_offsets_kernel(const int64_t *__restrict__ off, int64_t n_events,
                                                            T *__restrict__ content, const uint8_t *__restrict__ om,
                                                            const uint8_t *__restrict__ em,
                                                            const int32_t *__restrict__ idx, int32_t n, T value) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * PB;
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * PB + threadIdx.x; e < n_events; e += stride) {
        if (em && !em[e]) continue;
        const int64_t i = nth_selected(off[e], off[e + 1], om, idx ? idx[e] : n);
        if (i >= 0) content[i] = value;
    }
}

// Per event, the first pair (p, r), p before r in pT order, of selected
// objects with charges of opposite sign -- which is always the highest-pT
// object of positive charge and the highest-pT object of negative charge:
// with both present, say the positive one P first, every selected object
// before P has charge 0 (P is the first positive and the first negative
// comes after it), so P is the first object with a partner after it and
// its first partner is the first negative; with either absent there is no
// pair.  So one pass keeps the best (in pT order: larger pt first, NaN after
// every number, equal pt by lower index) positive and negative object.  Both
// get mask 1, every other object of the event 0.
struct OsBest {
    int32_t bp = -1, bn = -1;  // best positive and negative object so far
    float pp = 0.0f, pn = 0.0f;
    // objects come in index order, so a later one replaces the best only with
    // a larger pt, or a number a NaN
    __device__ __forceinline__ void take(uint32_t code, float p, int32_t i) {
        const bool up = (code == 1u) & ((bp < 0) | (p > pp) | ((pp != pp) & (p == p)));
        const bool dn = (code == 2u) & ((bn < 0) | (p > pn) | ((pn != pn) & (p == p)));
        bp = up ? i : bp;
        pp = up ? p : pp;
        bn = dn ? i : bn;
        pn = dn ? p : pn;
    }
};

// 1: selected, positive; 2: selected, negative; 0: neither
__device__ __forceinline__ uint32_t os_code(uint32_t m, int32_t q) { return m == 0u ? 0u : (q > 0 ? 1u : (q < 0 ? 2u : 0u)); }

// A pt's place in pT order as an integer: 1 for NaN, above it the numbers
// ascending, -0 as +0 (0 is left for "no object").
__device__ __forceinline__ uint32_t os_key(float p) {
    const uint32_t u = __builtin_bit_cast(uint32_t, p + 0.0f);
    return p != p ? 1u : ((u & 0x80000000u) ? ~u : u | 0x80000000u);
}

// The pair of one event of n objects by the whole wavefront: get(i, code, pt)
// reads object i.  The best object of a sign is the lowest index among the
// largest keys.
struct OsPair {
    int64_t p, n;  // -1: none
};
template <typename G>
__device__ __forceinline__ OsPair os_pair(int lane, int64_t n, G &&get) {
    uint32_t kp = 0, kn = 0, ip = 0, in = 0;
#pragma unroll 1
    for (int64_t i = lane; i < n; i += 64) {
        uint32_t code;
        float pt;
        get(i, code, pt);
        const uint32_t k = os_key(pt);
        const bool up = (code == 1u) & (k > kp), dn = (code == 2u) & (k > kn);
        kp = up ? k : kp;
        ip = up ? static_cast<uint32_t>(i) : ip;
        kn = dn ? k : kn;
        in = dn ? static_cast<uint32_t>(i) : in;
    }
    const uint32_t mp = wave_max(kp), mn = wave_max(kn);
    const uint32_t bp = ~wave_max(kp == mp ? ~ip : 0u), bn = ~wave_max(kn == mn ? ~in : 0u);
    if (mp == 0u || mn == 0u) return {-1, -1};
    return {static_cast<int64_t>(bp), static_cast<int64_t>(bn)};
}

// Each wavefront takes tiles of 64 consecutive events: the tile's objects as
// coalesced buffer loads over exactly its range, waited for once, staged in
// LDS with their code; one lane per event walks its objects there and marks
// the pair; then the mask bytes are written as one contiguous run.  A lane
// per event reading its objects itself took 24 gathers of 64 scattered
// addresses per tile and was bound by their address rate: 76 -> 37 us on
// 7.5e6 muons in 5e6 events (115 MB; floor 17 us).  Tiles with more objects
// than the staging holds run in parts.  Parts of few events, which would leave
// most lanes idle, are taken event by event by the whole wavefront, straight
// from HBM (events of 300 objects 2500 -> 208 us per 1.5e7 objects, of 2000
// 20 -> 0.87 ms per 2e7).
constexpr int kOsSlots = 8;   // objects per lane staged for one tile
constexpr int kOsFew = 8;     // events of a part that go one by one

template <typename T>
__global__ __launch_bounds__(PB) void opposite_sign_kernel(const int64_t *__restrict__ off, int64_t n_events,
                                                           const T *__restrict__ pt, const int32_t *__restrict__ q,
                                                           const uint8_t *__restrict__ om,
                                                           uint8_t *__restrict__ out) {
    struct Obj {
        float pt;
        uint32_t code;  // os_code, then 3 for the two objects of the pair
    };
    __shared__ Obj obj_s[PB / 64][64 * kOsSlots];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Obj *ob = obj_s[wave];
    const int64_t n_tiles = ceil_div(n_events, 64);
    const int64_t step = static_cast<int64_t>(gridDim.x) * (PB / 64);
    // the part [e0, e1) of a tile that ends at t1: its events (at least one),
    // and its objects [A, B)
    auto part = [&](int64_t e0, int64_t t1, int64_t &A, int64_t &B) {
        int ne = static_cast<int>(t1 - e0);
        A = as_const(off)[e0];
        B = as_const(off)[t1];
        while (ne > 1 && B - A > 64 * kOsSlots) {
            ne = (ne + 1) / 2;
            B = as_const(off)[e0 + ne];
        }
        return ne;
    };
    bool few = false;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (PB / 64) + wave; t < n_tiles; t += step) {
        const int64_t t1 = min<int64_t>(t * 64 + 64, n_events);
        for (int64_t e0 = t * 64, e1; e0 < t1; e0 = e1) {
            int64_t A, B;
            const int ne = part(e0, t1, A, B);
            e1 = e0 + ne;
            if (__builtin_expect(ne <= kOsFew, 0)) {
                few = true;  // below
                continue;
            }
            const int n = static_cast<int>(B - A);
            const buf_t bo = buf_span(off + e0, static_cast<uint32_t>(ne + 1) * 8u);
            const uint32_t o0 = buf_u32<kBufNt>(bo, lane * 8), o1 = buf_u32<kBufNt>(bo, lane * 8 + 8);
            const buf_t bp = buf_span(pt + A, static_cast<uint32_t>(n) * sizeof(T));
            const buf_t bq = buf_span(q + A, static_cast<uint32_t>(n) * 4u);
            const buf_t bm = buf_span(om ? static_cast<const void *>(om + A) : static_cast<const void *>(q),
                                      om ? static_cast<uint32_t>(n) : 0u);
            // half of the slots at a time: most tiles need the first half only
            constexpr int H = kOsSlots / 2;
            for (int h = 0; h < 2 && 64 * H * h < n; ++h) {
                uint32_t p[H], c[H], m[H];
#pragma unroll
                for (int k = 0; k < H; ++k) {
                    const int i = lane + 64 * (k + H * h);
                    p[k] = buf_raw<T, kBufNt>(bp, i);
                    c[k] = buf_u32<kBufNt>(bq, i * 4);
                    m[k] = om ? __builtin_amdgcn_raw_buffer_load_b8(bm, i, 0, kBufNt) : 1u;
                }
                asm volatile("" ::"v"(o0), "v"(o1));
#pragma unroll
                for (int k = 0; k < H; ++k) asm volatile("" ::"v"(p[k]), "v"(c[k]), "v"(m[k]));
#pragma unroll
                for (int k = 0; k < H; ++k)
                    ob[lane + 64 * (k + H * h)] = Obj{raw_f<T>(p[k]), os_code(m[k], static_cast<int32_t>(c[k]))};
            }
            wave_sync();
            if (lane < ne) {
                const int a0 = static_cast<int32_t>(o0 - static_cast<uint32_t>(A));
                const int a1 = static_cast<int32_t>(o1 - static_cast<uint32_t>(A));
                OsBest b;
                int i = a0;
                // two objects per step (both LDS reads in flight)
                for (; i + 2 <= a1; i += 2) {
                    const Obj x = ob[i], y = ob[i + 1];
                    b.take(x.code, x.pt, i);
                    b.take(y.code, y.pt, i + 1);
                }
                if (i < a1) b.take(ob[i].code, ob[i].pt, i);
                if (b.bp >= 0 && b.bn >= 0) {
                    ob[b.bp].code = 3u;
                    ob[b.bn].code = 3u;
                }
            }
            wave_sync();
            for (int i = lane; i < n; i += 64) out[A + i] = ob[i].code == 3u ? 1 : 0;
            wave_sync();  // the next (part of a) tile overwrites the staging
        }
    }
    if (!few) return;
    // the parts of few events (a loop of their own: beside the tiles their
    // registers and addresses cost 5e6 ordinary events 4%)
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (PB / 64) + wave; t < n_tiles; t += step) {
        const int64_t t1 = min<int64_t>(t * 64 + 64, n_events);
        for (int64_t e0 = t * 64, e1; e0 < t1; e0 = e1) {
            int64_t A, B;
            const int ne = part(e0, t1, A, B);
            e1 = e0 + ne;
            if (ne > kOsFew) continue;
            for (int64_t e = e0; e < e1; ++e) {
                const int64_t a0 = as_const(off)[e], m = as_const(off)[e + 1] - a0;
                const OsPair b = os_pair(lane, m, [&](int64_t i, uint32_t &code, float &p) {
                    code = os_code(om ? om[a0 + i] : 1u, q[a0 + i]);
                    p = ldf(pt, a0 + i);
                });
#pragma unroll 1
                for (int64_t i = lane; i < m; i += 64) out[a0 + i] = (b.p >= 0 && (i == b.p || i == b.n)) ? 1 : 0;
            }
        }
    }
}

// Compaction: each wavefront a tile of 64 events; the tile's objects 64 at a
// time, kept ones placed at base + (kept objects of the tile before them),
// base = offsets_out[first event of the tile].  ES: element size in bytes.
template <int ES>
struct Elem;
template <>
struct Elem<1> {
    using T = uint8_t;
};
template <>
struct Elem<2> {
    using T = uint16_t;
};
template <>
struct Elem<4> {
    using T = uint32_t;
};

constexpr int kCompactChunks = 8;  // chunks of 64 objects a tile reads in one batch

template <int ES>
__global__ __launch_bounds__(PB) void compact_kernel(const int64_t *__restrict__ off, int64_t n_events,
                                                     const typename Elem<ES>::T *__restrict__ content,
                                                     const uint8_t *__restrict__ om,
                                                     const int64_t *__restrict__ offsets_out, int64_t n_out,
                                                     typename Elem<ES>::T *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = static_cast<int64_t>(blockIdx.x) * (PB / 64) + (threadIdx.x >> 6);
    const int64_t n_waves = static_cast<int64_t>(gridDim.x) * (PB / 64);
    const int64_t n_tiles = ceil_div(n_events, 64);
    for (int64_t t = wave; t < n_tiles; t += n_waves) {
        const int64_t e0 = t * 64;
        const int64_t e1 = min<int64_t>(e0 + 64, n_events);
        const int64_t A = as_const(off)[e0], B = as_const(off)[e1];
        int64_t base = as_const(offsets_out)[e0];
        if (B - A <= 64 * kCompactChunks) {
            // the whole tile: every chunk's mask bytes and elements as
            // buffer loads over exactly [A, B) (0 past the end), all in
            // flight and waited for once
            const int nobj = static_cast<int>(B - A);
            const buf_t bc = buf_span(content + A, static_cast<uint32_t>(nobj) * ES);
            const buf_t bm = buf_span(om ? static_cast<const void *>(om + A) : static_cast<const void *>(content),
                                      om ? static_cast<uint32_t>(nobj) : 0u);
            uint32_t mk[kCompactChunks], v[kCompactChunks];
#pragma unroll
            for (int c = 0; c < kCompactChunks; ++c) {
                const int i = lane + 64 * c;
                mk[c] = om ? __builtin_amdgcn_raw_buffer_load_b8(bm, i, 0, kBufNt) : 1u;
                if constexpr (ES == 4)
                    v[c] = __builtin_amdgcn_raw_buffer_load_b32(bc, i * 4, 0, kBufNt);
                else if constexpr (ES == 2)
                    v[c] = __builtin_amdgcn_raw_buffer_load_b16(bc, i * 2, 0, kBufNt);
                else
                    v[c] = __builtin_amdgcn_raw_buffer_load_b8(bc, i, 0, kBufNt);
            }
#pragma unroll
            for (int c = 0; c < kCompactChunks; ++c) asm volatile("" ::"v"(mk[c]), "v"(v[c]));
#pragma unroll
            for (int c = 0; c < kCompactChunks; ++c) {
                if (64 * c >= nobj) break;
                const bool keep = (lane + 64 * c < nobj) & (mk[c] != 0u);
                const uint64_t bal = __ballot(keep);
                const int before = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                    static_cast<uint32_t>(bal >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(bal), 0u)));
                const int64_t dst = base + before;
                if (keep && dst < n_out) out[dst] = static_cast<typename Elem<ES>::T>(v[c]);
                base += __popcll(bal);
            }
            continue;
        }
        for (int64_t k0 = A; k0 < B; k0 += 64) {
            const int64_t i = k0 + lane;
            const bool in = i < B;
            const bool keep = in && (!om || om[i] != 0);
            typename Elem<ES>::T v{};
            if (keep) v = content[i];
            const uint64_t bal = __ballot(keep);
            const int before = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                static_cast<uint32_t>(bal >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(bal), 0u)));
            const int64_t dst = base + before;
            if (keep && dst < n_out) out[dst] = v;
            base += __popcll(bal);
        }
    }
}

static int grid_for(int64_t rows, int per_thread = 1) {
    return static_cast<int>(
        std::max<int64_t>(1, std::min<int64_t>(ceil_div(ceil_div(rows, per_thread), PB), kTileWgPerCu * device_cus())));
}

}  // namespace hepk

extern "C" int hepk_get_in_offsets(const int64_t *offsets, int64_t n_events, const void *content, int32_t dtype,
                                   const uint8_t *obj_mask, const uint8_t *evt_mask, const int32_t *idx, int32_t n,
                                   float fill, float *out, int32_t *out_index, hipStream_t stream) {
    using namespace hepk;
    clear_error();
    HEPK_REQUIRE(n_events >= 0 && offsets, "hepk_get_in_offsets: bad offsets or n_events");
    HEPK_REQUIRE(n_events == 0 || (content && out), "hepk_get_in_offsets: content or out is NULL");
    HEPK_REQUIRE(dtype == HEPK_F32 || dtype == HEPK_F16, "hepk_get_in_offsets: dtype %d not F32 or F16", dtype);
    if (n_events == 0) return HEPK_OK;
    const int g = grid_for(n_events);
    if (dtype == HEPK_F16)
        get_in_offsets_kernel<_Float16><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const _Float16 *>(content),
                                                               obj_mask, evt_mask, idx, n, fill, out, out_index);
    else
        get_in_offsets_kernel<float><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const float *>(content),
                                                            obj_mask, evt_mask, idx, n, fill, out, out_index);
    return check_launch("hepk_get_in_offsets");
}

extern "C" int hepk_set_in_offsets(const int64_t *offsets, int64_t n_events, void *content, int32_t dtype,
                                   const uint8_t *obj_mask, const uint8_t *evt_mask, const int32_t *idx, int32_t n,
                                   float value, hipStream_t stream) {
    using namespace hepk;
    clear_error();
    HEPK_REQUIRE(n_events >= 0 && offsets, "hepk_set_in_offsets: bad offsets or n_events");
    HEPK_REQUIRE(n_events == 0 || content, "hepk_set_in_offsets: content is NULL");
    HEPK_REQUIRE(dtype == HEPK_F32 || dtype == HEPK_U8, "hepk_set_in_offsets: dtype %d not F32 or U8", dtype);
    if (n_events == 0) return HEPK_OK;
    const int g = grid_for(n_events);
    if (dtype == HEPK_U8)
        set_in_offsets_kernel<uint8_t><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<uint8_t *>(content),
                                                              obj_mask, evt_mask, idx, n,
                                                              static_cast<uint8_t>(value != 0.0f ? 1 : 0));
    else
        set_in_offsets_kernel<float><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<float *>(content), obj_mask,
                                                            evt_mask, idx, n, value);
    return check_launch("hepk_set_in_offsets");
}

extern "C" int hepk_select_opposite_sign(const int64_t *offsets, int64_t n_events, const void *pt, int32_t dtype,
                                         const int32_t *charge, const uint8_t *obj_mask, uint8_t *mask_out,
                                         hipStream_t stream) {
    using namespace hepk;
    clear_error();
    HEPK_REQUIRE(n_events >= 0 && offsets, "hepk_select_opposite_sign: bad offsets or n_events");
    HEPK_REQUIRE(n_events == 0 || (pt && charge && mask_out), "hepk_select_opposite_sign: NULL column or output");
    HEPK_REQUIRE(dtype == HEPK_F32 || dtype == HEPK_F16, "hepk_select_opposite_sign: dtype %d not F32 or F16", dtype);
    if (n_events == 0) return HEPK_OK;
    const int g = grid_for(n_events);  // a tile of 64 events per wavefront
    if (dtype == HEPK_F16)
        opposite_sign_kernel<_Float16><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const _Float16 *>(pt),
                                                              charge, obj_mask, mask_out);
    else
        opposite_sign_kernel<float><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const float *>(pt), charge,
                                                           obj_mask, mask_out);
    return check_launch("hepk_select_opposite_sign");
}

extern "C" int hepk_compact(const int64_t *offsets, int64_t n_events, const void *content, int32_t dtype,
                            const uint8_t *obj_mask, const int64_t *offsets_out, int64_t n_out, void *out,
                            hipStream_t stream) {
    using namespace hepk;
    clear_error();
    HEPK_REQUIRE(n_events >= 0 && offsets && offsets_out, "hepk_compact: bad offsets or n_events");
    HEPK_REQUIRE(n_out >= 0 && (n_out == 0 || out), "hepk_compact: bad output");
    HEPK_REQUIRE(n_events == 0 || content, "hepk_compact: content is NULL");
    HEPK_REQUIRE(dtype >= HEPK_F32 && dtype <= HEPK_U8, "hepk_compact: bad dtype %d", dtype);
    if (n_events == 0 || n_out == 0) return HEPK_OK;
    const int g = static_cast<int>(
        std::max<int64_t>(1, std::min<int64_t>(ceil_div(ceil_div(n_events, 64), PB / 64), kTileWgPerCu * device_cus())));
    if (dtype == HEPK_U8)
        compact_kernel<1><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const uint8_t *>(content), obj_mask,
                                                offsets_out, n_out, static_cast<uint8_t *>(out));
    else if (dtype == HEPK_F16)
        compact_kernel<2><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const uint16_t *>(content), obj_mask,
                                                offsets_out, n_out, static_cast<uint16_t *>(out));
    else
        compact_kernel<4><<<g, PB, 0, stream>>>(offsets, n_events, static_cast<const uint32_t *>(content), obj_mask,
                                                offsets_out, n_out, static_cast<uint32_t *>(out));
    return check_launch("hepk_compact");
}
