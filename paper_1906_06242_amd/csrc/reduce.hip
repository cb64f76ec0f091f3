// hepk_reduce: per-event segmented reductions over jagged content
// (Sec. III: the H_T kernel of Listing 1, the count/sum/max/min-within-
// offsets kernels, and the generic pairwise operator taken as the product).
//
// Each wavefront owns tiles of 64 consecutive events and works through them
// without waiting for the rest of its workgroup.  For one tile it reads the
// tile's object range with two scalar loads, then issues every load of the
// tile at once -- both offsets and the event mask of each event lane, and up
// to RK objects (content and object mask) per lane, consecutive lanes on
// consecutive objects -- stages the objects in its own LDS region, and lets
// one lane per event walk its objects in order.  Walking in order keeps the
// float32 sum identical to the left-to-right sum of Listing 1's inner loop (a
// tree would round differently), and gives the lowest index on max/min ties.
// A tile with more than 64 * RK objects is walked straight from HBM, one lane
// per event, with the same arithmetic.  Counts can feed an exclusive scan
// that yields the offsets of the selected sub-collection.
#include "common.hpp"

namespace hepk {

constexpr int RB = 256;  // threads per workgroup
constexpr int RW = RB / 64;
constexpr int RK = 8;    // objects per lane staged for one tile (512 per tile)

enum { R_COUNT = 0, R_SUM = 1, R_MAX = 2, R_MIN = 3, R_PROD = 4 };

// Inclusive prefix sum over the wavefront (every lane active).
__device__ __forceinline__ int64_t wave_scan(int64_t v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t u = __shfl_up(v, d);
        v += static_cast<int>(threadIdx.x & 63) >= d ? u : 0;
    }
    return v;
}

// Running reduction of one event.
template <int OP>
struct Acc {
    int32_t cnt = 0;
    float sum = 0.0f;
    float prod = 1.0f;
    float best = (OP == R_MAX) ? -INFINITY : INFINITY;
    int32_t bi = -1;
    __device__ __forceinline__ void add(float v, bool keep, int32_t k) {
        if (!keep) return;
        if (OP == R_COUNT) {
            ++cnt;
        } else if (OP == R_SUM) {
            sum = sum + v;
        } else if (OP == R_PROD) {
            prod = prod * v;
        } else {
            const bool better = (OP == R_MAX) ? (v > best) : (v < best);
            if (bi < 0 || better) {
                best = v;
                bi = k;
            }
        }
    }
};

// SUMS (COUNT with offsets_out): a workgroup takes `span` consecutive events
// (a multiple of RB) instead of every gridDim-th group of tiles and leaves
// their total at offsets_out[min((blockIdx + 1) * span, N)] for the scan below.
template <typename T, int OP, bool SUMS = false>
__global__ __launch_bounds__(RB) void reduce_kernel(const int64_t *__restrict__ off, int64_t n_events,
                                                    const T *__restrict__ content,
                                                    const uint8_t *__restrict__ obj_mask,
                                                    const uint8_t *__restrict__ evt_mask, void *out,
                                                    int32_t *out_arg, int index_only, int64_t span,
                                                    int64_t *offsets_out) {
    static_assert(__is_same(T, float) || __is_same(T, _Float16), "content is float32 or float16 (raw_f)");
    __shared__ float val_s[RW][(OP == R_COUNT) ? 1 : 64 * RK];
    // the tile's mask bytes as the 4-byte words that hold them (the first
    // byte of the range at byte s of the first word)
    constexpr int RMW = (64 * RK + 3 + 255) / 256;  // words per lane
    __shared__ uint32_t msk_s[RW][64 * RMW];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *vs = val_s[wave];
    uint32_t *msw = msk_s[wave];
    const int64_t n_tiles = SUMS ? min<int64_t>(ceil_div(n_events, 64), (blockIdx.x + 1) * (span / 64)) : ceil_div(n_events, 64);
    int64_t sum64 = 0;  // SUMS: objects counted by this lane
    const bool walk_objects = !(OP == R_COUNT && !obj_mask);
    const int64_t step = SUMS ? RW : static_cast<int64_t>(gridDim.x) * RW;
    // the object range of a tile is fetched one tile ahead (scalar loads that
    // overlap the current tile's work)
    auto bounds = [&](int64_t t, int64_t &lo, int64_t &hi) {
        const int64_t e0 = t * 64;
        lo = as_const(off)[e0];
        hi = as_const(off)[e0 + min<int64_t>(64, n_events - e0)];
    };
    int64_t t = static_cast<int64_t>(blockIdx.x) * (SUMS ? span / 64 : RW) + wave;
    int64_t nA = 0, nB = 0;
    if (t < n_tiles) bounds(t, nA, nB);
    for (; t < n_tiles; t += step) {
        const int64_t e0 = t * 64;
        const int ne = static_cast<int>(min<int64_t>(64, n_events - e0));
        const int64_t A = nA;
        const int64_t tot = nB - nA;
        if (t + step < n_tiles) bounds(t + step, nA, nB);
        const int64_t e = e0 + lane;
        const bool act = lane < ne;
        // the tile's loads are buffer loads over exactly its ranges (0 past
        // their ends: no per-lane or per-slot branch), waited for together:
        // both offsets of each event lane's event (their low 32-bit words:
        // tile-relative differences are exact modulo 2^32), its event mask
        // byte, and below the objects and their mask words
        const buf_t bo = buf_span(off + e0, static_cast<uint32_t>(ne + 1) * 8u);
        const uint32_t o0 = buf_u32(bo, lane * 8), o1 = buf_u32(bo, lane * 8 + 8);
        const buf_t bev = buf_span(evt_mask ? static_cast<const void *>(evt_mask + e0) : static_cast<const void *>(off),
                                   evt_mask ? static_cast<uint32_t>(ne) : 0u);
        const uint32_t evb = evt_mask ? __builtin_amdgcn_raw_buffer_load_b8(bev, lane, 0, 0) : 1u;
        int64_t a0 = 0, a1 = 0;  // the event's objects, relative to the tile's first
        bool take = false;
        auto event_range = [&]() {
            a0 = act ? static_cast<int32_t>(o0 - static_cast<uint32_t>(A)) : 0;
            a1 = act ? static_cast<int32_t>(o1 - static_cast<uint32_t>(A)) : 0;
            take = act && evb != 0u;
        };
        Acc<OP> r;
        if (!walk_objects) {
            event_range();
            r.cnt = take ? static_cast<int32_t>(a1 - a0) : 0;
        } else if (tot <= 64 * RK) {
            const int n = static_cast<int>(tot);
            const buf_t bc = buf_span(content + A, static_cast<uint32_t>(n) * sizeof(T));
            uint32_t rv[RK];
#pragma unroll
            for (int k = 0; k < RK; ++k) rv[k] = OP != R_COUNT ? buf_raw<T>(bc, lane + 64 * k) : 0u;
            // mask bytes in 4-byte loads: the aligned words that hold bytes
            // [A, A + n)
            int s = 0, nw = 0;
            uint32_t mw[RMW];
#pragma unroll
            for (int k = 0; k < RMW; ++k) mw[k] = 0u;
            if (obj_mask) {
                const uint8_t *p = obj_mask + A;
                s = static_cast<int>(reinterpret_cast<uintptr_t>(p) & 3u);
                nw = n > 0 ? (n + s + 3) >> 2 : 0;
                const buf_t bw = buf_span(p - s, static_cast<uint32_t>(nw) * 4u);
#pragma unroll
                for (int k = 0; k < RMW; ++k) mw[k] = buf_u32(bw, (lane + 64 * k) * 4);
            }
            asm volatile("" ::"v"(o0), "v"(o1), "v"(evb));
#pragma unroll
            for (int k = 0; k < RK; ++k) asm volatile("" ::"v"(rv[k]));
#pragma unroll
            for (int k = 0; k < RMW; ++k) asm volatile("" ::"v"(mw[k]));
            event_range();
            float v[RK];
#pragma unroll
            for (int k = 0; k < RK; ++k) v[k] = raw_f<T>(rv[k]);
#pragma unroll
            for (int k = 0; k < RK; ++k) {
                const int i = lane + 64 * k;
                if (OP != R_COUNT && i < n) vs[i] = v[k];
            }
            if (obj_mask) {
#pragma unroll
                for (int k = 0; k < RMW; ++k) {
                    const int w = lane + 64 * k;
                    if (w < nw) msw[w] = mw[k];
                }
            }
            const uint8_t *ms = reinterpret_cast<const uint8_t *>(msw) + s;
            const bool all = obj_mask == nullptr;
            wave_sync();
            const int b0 = static_cast<int>(a0), b1 = static_cast<int>(a1);  // within the tile's 512
            if (take) {
                // two objects per step (both LDS reads in flight), in order
                int k = b0;
                for (; k + 2 <= b1; k += 2) {
                    const float v0 = OP != R_COUNT ? vs[k] : 0.0f, v1 = OP != R_COUNT ? vs[k + 1] : 0.0f;
                    const bool m0 = all || ms[k] != 0, m1 = all || ms[k + 1] != 0;
                    r.add(v0, m0, k - b0);
                    r.add(v1, m1, k + 1 - b0);
                }
                if (k < b1) r.add(OP != R_COUNT ? vs[k] : 0.0f, all || ms[k] != 0, k - b0);
            }
            wave_sync();  // the next tile overwrites the staging
        } else if (event_range(), take) {
            for (int64_t k = a0; k < a1; ++k)
                r.add(OP != R_COUNT ? ldf(content, A + k) : 0.0f, !obj_mask || obj_mask[A + k] != 0,
                      static_cast<int32_t>(k - a0));
        }
        if (act) {
            if (OP == R_COUNT) {
                static_cast<int32_t *>(out)[e] = r.cnt;
                if (SUMS) sum64 += r.cnt;
            } else if (OP == R_SUM) {
                static_cast<float *>(out)[e] = r.sum;
            } else if (OP == R_PROD) {
                static_cast<float *>(out)[e] = r.prod;
            } else if (index_only) {
                static_cast<int32_t *>(out)[e] = r.bi;
            } else {
                static_cast<float *>(out)[e] = r.best;
                if (out_arg) out_arg[e] = r.bi;
            }
        }
    }
    if constexpr (SUMS) {
        __shared__ int64_t tot_s[RW];
        sum64 = wave_scan(sum64);
        if (lane == 63) tot_s[wave] = sum64;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t s = 0;
            for (int w = 0; w < RW; ++w) s += tot_s[w];
            offsets_out[min<int64_t>((blockIdx.x + 1) * span, n_events)] = s;
        }
    }
}

// Prefix offsets of the selected sub-collection without a temporary, in three
// launches: the counting kernel above leaves the total of every span of
// events at the entry whose final value is the sum up to that span's end;
// one workgroup scans those entries in place; then every span reads its base
// from the entry of its first event and writes its other entries.  The span
// grows with the events so that at most kMaxSpans totals are scanned -- by
// one workgroup in one step, each total a 64-bit load on a line of its own:
// 5e6 events took 117 us counting included with 256-event spans (61 us of it
// that scan), 47 us now; floor 25 us (145 MB).
//
// Where offsets_out overlaps offsets (a collection's offsets replaced by its
// selection's), no total may be written while another workgroup still reads
// its ranges: the counts are made by a launch of their own and the totals from
// them by span_sums_kernel.
constexpr int kMaxSpans = 4096;

__global__ __launch_bounds__(RB) void span_sums_kernel(const int32_t *counts, int64_t n_events, int64_t *offsets_out,
                                                       int64_t span) {
    __shared__ int64_t tot_s[RW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e1 = min<int64_t>((blockIdx.x + 1) * span, n_events);
    int64_t sum = 0;
    for (int64_t e = blockIdx.x * span + threadIdx.x; e < e1; e += RB) sum += counts[e];
    sum = wave_scan(sum);
    if (lane == 63) tot_s[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t s = 0;
        for (int w = 0; w < RW; ++w) s += tot_s[w];
        offsets_out[e1] = s;
    }
}

static int64_t span_of(int64_t n_events) {
    int64_t s = RB;
    while (ceil_div(n_events, s) > kMaxSpans) s *= 2;
    return s;
}

// Inclusive scan, in place, of the (at most kMaxSpans) totals.
__global__ __launch_bounds__(1024) void scan_spans_kernel(int64_t *offsets_out, int64_t n_events, int64_t span) {
    constexpr int K = kMaxSpans / 1024;
    __shared__ int64_t wave_s[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = ceil_div(n_events, span);
    int64_t v[K];
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t t = static_cast<int64_t>(tid) * K + k;
        v[k] = t < n ? offsets_out[min<int64_t>((t + 1) * span, n_events)] : 0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) sum += v[k];
    int64_t incl = wave_scan(sum);
    if (lane == 63) wave_s[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wave_s[w];
    int64_t run = incl - sum;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t t = static_cast<int64_t>(tid) * K + k;
        run += v[k];
        if (t < n) offsets_out[min<int64_t>((t + 1) * span, n_events)] = run;
    }
}

// offsets_out[e] = sum of counts[0..e) for the events of one span per
// workgroup (the entry N is final already; a span's first entry is read as
// its base and written back).  Four events per thread and step, one 16-byte
// load and two 16-byte stores when the arrays allow (VEC).
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef long long i64x2 __attribute__((ext_vector_type(2)));

template <bool VEC>
__global__ __launch_bounds__(RB) void offsets_from_counts_kernel(const int32_t *counts, int64_t n_events,
                                                                 int64_t *offsets_out, int64_t span) {
    __shared__ int64_t wave_s[2][RW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t e0 = static_cast<int64_t>(blockIdx.x) * span;
    const int64_t e1 = min<int64_t>(e0 + span, n_events);
    int64_t base = blockIdx.x > 0 ? offsets_out[e0] : 0;
    if (n_events == 0 && tid == 0) offsets_out[0] = 0;
    int buf = 0;
    for (int64_t s = e0; s < e1; s += 4 * RB, buf ^= 1) {
        const int64_t e = s + 4 * tid;
        int32_t c[4] = {0, 0, 0, 0};
        if (VEC && e + 4 <= e1) {
            const i32x4 q = *reinterpret_cast<const i32x4 *>(counts + e);
            c[0] = q.x;
            c[1] = q.y;
            c[2] = q.z;
            c[3] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (e + k < e1) c[k] = counts[e + k];
        }
        const int64_t sum = static_cast<int64_t>(c[0]) + c[1] + c[2] + c[3];
        const int64_t incl = wave_scan(sum);
        if (lane == 63) wave_s[buf][wave] = incl;
        __syncthreads();  // (the other buffer's readers are past it by the next barrier)
        int64_t before = base, all = 0;
#pragma unroll
        for (int w = 0; w < RW; ++w) {
            const int64_t t = wave_s[buf][w];
            before += w < wave ? t : 0;
            all += t;
        }
        base += all;
        int64_t o[4];
        o[0] = before + incl - sum;
#pragma unroll
        for (int k = 1; k < 4; ++k) o[k] = o[k - 1] + c[k - 1];
        if (VEC && e + 4 <= e1) {
            i64x2 *w = reinterpret_cast<i64x2 *>(offsets_out + e);
            w[0] = i64x2{o[0], o[1]};
            w[1] = i64x2{o[2], o[3]};
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (e + k < e1) offsets_out[e + k] = o[k];
        }
    }
}

template <typename T, int OP>
static int launch_reduce(const int64_t *off, int64_t n, const void *content, const uint8_t *om,
                         const uint8_t *em, void *out, int32_t *out_arg, int index_only, hipStream_t stream) {
    const int64_t n_wave_tiles = ceil_div(n, 64);
    const int grid = static_cast<int>(std::min<int64_t>(ceil_div(n_wave_tiles, RW), 16 * device_cus()));
    reduce_kernel<T, OP><<<grid, RB, 0, stream>>>(off, n, static_cast<const T *>(content), om, em, out,
                                                  out_arg, index_only, 0, nullptr);
    return check_launch("hepk_reduce");
}

// Whether the byte ranges [p, p + np) and [q, q + nq) share a byte.
static bool overlap(const void *p, int64_t np, const void *q, int64_t nq) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + static_cast<uintptr_t>(nq) && b < a + static_cast<uintptr_t>(np);
}

// COUNT with offsets_out (three launches, four when it overlaps an input; no
// temporary).
static int launch_count_offsets(const int64_t *off, int64_t n, const uint8_t *om, const uint8_t *em, int32_t *counts,
                                int64_t *offsets_out, hipStream_t stream) {
    const int64_t span = span_of(n);
    const int g = static_cast<int>(std::max<int64_t>(1, ceil_div(n, span)));
    const int64_t bytes = (n + 1) * static_cast<int64_t>(sizeof(int64_t));
    if (n > 0 && (overlap(offsets_out, bytes, off, bytes) || (em && overlap(offsets_out, bytes, em, n)))) {
        if (int rc = launch_reduce<float, R_COUNT>(off, n, nullptr, om, em, counts, nullptr, 0, stream)) return rc;
        span_sums_kernel<<<g, RB, 0, stream>>>(counts, n, offsets_out, span);
        if (int rc = check_launch("hepk_reduce span sums")) return rc;
    } else if (n > 0) {
        reduce_kernel<float, R_COUNT, true><<<g, RB, 0, stream>>>(off, n, nullptr, om, em, counts, nullptr, 0, span,
                                                                  offsets_out);
        if (int rc = check_launch("hepk_reduce count")) return rc;
    }
    if (n > 0) {
        scan_spans_kernel<<<1, 1024, 0, stream>>>(offsets_out, n, span);
        if (int rc = check_launch("hepk_reduce scan")) return rc;
    }
    const bool vec = reinterpret_cast<uintptr_t>(counts) % 16 == 0 && reinterpret_cast<uintptr_t>(offsets_out) % 16 == 0;
    if (vec)
        offsets_from_counts_kernel<true><<<g, RB, 0, stream>>>(counts, n, offsets_out, span);
    else
        offsets_from_counts_kernel<false><<<g, RB, 0, stream>>>(counts, n, offsets_out, span);
    return check_launch("hepk_reduce offsets");
}

}  // namespace hepk

extern "C" int hepk_reduce(int32_t op, const int64_t *offsets, int64_t n_events, const void *content,
                           int32_t dtype, const uint8_t *obj_mask, const uint8_t *evt_mask, void *out,
                           int32_t *out_arg, int64_t *offsets_out, hipStream_t stream) {
    using namespace hepk;
    clear_error();
    HEPK_REQUIRE(op >= HEPK_COUNT && op <= HEPK_PROD, "hepk_reduce: bad op %d", op);
    HEPK_REQUIRE(n_events >= 0, "hepk_reduce: n_events < 0");
    HEPK_REQUIRE(offsets, "hepk_reduce: offsets is NULL");
    HEPK_REQUIRE(n_events == 0 || out, "hepk_reduce: out is NULL");
    HEPK_REQUIRE(!offsets_out || op == HEPK_COUNT, "hepk_reduce: offsets_out is for COUNT only");
    HEPK_REQUIRE(!out_arg || op == HEPK_MAX || op == HEPK_MIN, "hepk_reduce: out_arg is for MAX/MIN only");
    if (op != HEPK_COUNT) {
        if (dtype != HEPK_F32 && dtype != HEPK_F16) {
            set_error("hepk_reduce: content dtype %d unsupported for this op", dtype);
            return HEPK_EUNSUPPORTED;
        }
        HEPK_REQUIRE(content || n_events == 0, "hepk_reduce: content is NULL");
    }
    if (offsets_out)
        return launch_count_offsets(offsets, n_events, obj_mask, evt_mask, static_cast<int32_t *>(out), offsets_out,
                                    stream);
    if (n_events == 0) return HEPK_OK;
    int rc;
    const bool h = dtype == HEPK_F16;
    switch (op) {
    case HEPK_COUNT:
        rc = launch_reduce<float, R_COUNT>(offsets, n_events, nullptr, obj_mask, evt_mask, out, nullptr, 0,
                                           stream);
        break;
    case HEPK_SUM:
        rc = h ? launch_reduce<_Float16, R_SUM>(offsets, n_events, content, obj_mask, evt_mask, out, nullptr, 0,
                                                stream)
               : launch_reduce<float, R_SUM>(offsets, n_events, content, obj_mask, evt_mask, out, nullptr, 0,
                                             stream);
        break;
    case HEPK_PROD:
        rc = h ? launch_reduce<_Float16, R_PROD>(offsets, n_events, content, obj_mask, evt_mask, out, nullptr, 0,
                                                 stream)
               : launch_reduce<float, R_PROD>(offsets, n_events, content, obj_mask, evt_mask, out, nullptr, 0,
                                              stream);
        break;
    case HEPK_MAX:
    case HEPK_ARGMAX:
        rc = h ? launch_reduce<_Float16, R_MAX>(offsets, n_events, content, obj_mask, evt_mask, out, out_arg,
                                                op == HEPK_ARGMAX, stream)
               : launch_reduce<float, R_MAX>(offsets, n_events, content, obj_mask, evt_mask, out, out_arg,
                                             op == HEPK_ARGMAX, stream);
        break;
    default:
        rc = h ? launch_reduce<_Float16, R_MIN>(offsets, n_events, content, obj_mask, evt_mask, out, out_arg,
                                                op == HEPK_ARGMIN, stream)
               : launch_reduce<float, R_MIN>(offsets, n_events, content, obj_mask, evt_mask, out, out_arg,
                                             op == HEPK_ARGMIN, stream);
        break;
    }
    return rc;
}
