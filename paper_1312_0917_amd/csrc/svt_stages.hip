// Stage kernels of libsvt: combine (count, scan, list), plain fit (one lane per listed
// combination), select (cut, best track, kept list); the batched pass shares the kept-list and
// best-track kernels.
//
// Section II-A of the paper splits the serial code into unpack / combine / fit; these are the
// GPU forms of the last two, a few launches each (the unpack stage is k_unit_count and
// k_unit_table in svt_units.hip).
#include "svt_fit.h"

namespace svt {
namespace {

// ---- single-workgroup in-place exclusive scan ---------------------------------------------
// Exclusive scan of col[0 .. n) in place by one workgroup of NT threads; the total goes to *tot
// (nullable).  tmp holds NT / 64 + 1 values.
template <int NT>
__device__ int64_t scan_column(int64_t *col, int64_t n, int64_t *tot, int64_t *tmp) {
    constexpr int kItems = 4;
    int64_t carry = 0;
    for (int64_t base = 0; base < n; base += static_cast<int64_t>(NT) * kItems) {
        const int64_t i0 = base + static_cast<int64_t>(threadIdx.x) * kItems;
        int64_t v[kItems];
        int64_t s = 0;
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            v[e] = (i0 + e < n) ? col[i0 + e] : 0;
            s += v[e];
        }
        int64_t total;
        int64_t ex = block_excl_scan<int64_t, NT>(s, tmp, total);
        int64_t run = carry + ex;
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            if (i0 + e < n) col[i0 + e] = run;
            run += v[e];
        }
        carry += total;
    }
    if (threadIdx.x == 0 && tot) *tot = carry;
    return carry;
}

// The total is checked against cap (class CAPACITY, index cap_index) when cap >= 0.
__global__ __launch_bounds__(kScanThreads) void k_scan(int64_t *data, Sizes n_s, int64_t div,
                                                       int64_t *tot, int64_t cap,
                                                       uint32_t cap_index, uint64_t *err,
                                                       int32_t skip_if_error) {
    __shared__ int64_t tmp[kScanThreads / kWaveSize + 1];
    if (skip_if_error && block_has_error(err)) {
        if (threadIdx.x == 0 && tot) *tot = -1;
        return;
    }
    const int64_t n = (load_size(n_s) + div - 1) / div;
    const int64_t carry = scan_column<kScanThreads>(data, n, tot, tmp);
    if (threadIdx.x == 0 && cap >= 0 && carry > cap) report(err, SVT_ERRCLASS_CAPACITY, cap_index);
}

// ---- combine 1: combinations per road and per-block sums ---------------------------------
__global__ __launch_bounds__(kRoadBlock) void k_combo_count(svt_roads roads, Sizes n_roads_s,
                                                            int64_t *rb_sums, uint64_t *err) {
    __shared__ int64_t tmp[kRoadBlock / kWaveSize + 1];
    if (has_error(err)) return;
    const int64_t nr = load_size(n_roads_s);
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRoadBlock + threadIdx.x;
    if (static_cast<int64_t>(blockIdx.x) * kRoadBlock >= nr) return;
    int64_t c = 0;
    if (r < nr) {
        const uint32_t p = roads.nhits[r];
        c = 1;
        for (int l = 0; l < SVT_N_LAYERS; ++l) c *= nh_of(p, l);
        roads.ncombo[r] = static_cast<int32_t>(c);
    }
    const int64_t s = block_sum<int64_t, kRoadBlock>(c, tmp);
    if (threadIdx.x == 0) rb_sums[blockIdx.x] = s;
}

constexpr int kListTile = 2048;  // combinations a workgroup of k_materialize lists

// ---- combine 2: combo_begin, marks for the listing -----------------------------------------
__global__ __launch_bounds__(kRoadBlock) void k_combo_begin(svt_roads roads, Sizes n_roads_s,
                                                            const int64_t *rb_prefix,
                                                            int32_t *combo_road,
                                                            int64_t combo_cap, uint64_t *err) {
    __shared__ int64_t tmp[kRoadBlock / kWaveSize + 1];
    if (has_error(err)) return;
    const int64_t nr = load_size(n_roads_s);
    if (static_cast<int64_t>(blockIdx.x) * kRoadBlock >= nr) return;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRoadBlock + threadIdx.x;
    const int64_t c = (r < nr) ? roads.ncombo[r] : 0;
    int64_t tot;
    const int64_t begin = block_excl_scan<int64_t, kRoadBlock>(c, tmp, tot) + rb_prefix[blockIdx.x];
    if (r >= nr) return;
    roads.combo_begin[r] = begin;
    if (combo_road && c > 0) {
        // the road of each listing tile's first combination, where the listing will put it
        for (int64_t t = (begin + kListTile - 1) / kListTile; t * kListTile < begin + c; ++t)
            if (t * kListTile < combo_cap) combo_road[t * kListTile] = static_cast<int32_t>(r);
    }
}

// ---- combine 3 (plain path): list every combination --------------------------------------
// A workgroup lists kListTile consecutive combinations, however few or many roads they belong
// to: by blocks of 256 roads, the workgroup with the largest roads took most of the time (190 us
// for 1500 uneven events, now 19; 51 and 20 us for 3000 events of 64 roads, whose list is 49 MB;
// tiles of 4096 and 8192 take 20 and 23).  k_combo_begin has left the road of the tile's first
// combination in combo_road; the tile's roads are staged in LDS, up to kListRoads at a time.
//
// The list's capacity says nothing about its length: up to kListGrid tiles of it get a workgroup each
// (16.8e6 combinations), above that (LOOP) the workgroups take the tiles in turn.  400 roads listed by a
// caller with room for 4e8 combinations take 21 us, with a workgroup per tile of the capacity 52; the
// loop costs 1 us of 20 where a tile each would do.
//
// Where kListRoads roads have fewer than kListSparse combinations, nearly all of them none, the rest of
// the tile is not staged: a lane searches the table for its combinations' roads.  The stage for 1e6 roads
// of which one in N has 32 combinations, staged throughout / so: N = 5000 720 / 27 us, 500 156 / 27,
// 100 47 / 28, 50 37 / 30; 20 has 800 combinations per 512 roads and takes 30 staged.
constexpr int kListRoads = 512;
constexpr int kListThreads = 256;
constexpr int kListSparse = 400;
constexpr int kListGrid = 8192;

// The last road of lo .. hi that starts at or before combination c (lo does).  Seven probes at a time:
// one waits for memory as long as seven do.
__device__ int64_t road_of(const int64_t *__restrict__ begin, int64_t lo, int64_t hi, int64_t c) {
    while (lo < hi) {
        const int64_t step = (hi - lo) / 8 + 1;
        int64_t b[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            const int64_t p = lo + (q + 1) * step;
            b[q] = p <= hi ? begin[p] : INT64_MAX;
        }
        int n = 0;
#pragma unroll
        for (int q = 0; q < 7; ++q) n += b[q] <= c ? 1 : 0;
        lo += n * step;
        hi = lo + step - 1 < hi ? lo + step - 1 : hi;
    }
    return lo;
}

// Combinations c_lo .. c_lo + len - 1 (at most kListTile), which belong to roads r0 .. last.
__device__ __forceinline__ void list_sparse(const svt_roads &roads, int64_t r0, int64_t last,
                                         int64_t c_lo, int len, int32_t *combo_road,
                                         uint32_t *combo_hits) {
    constexpr int kPer = kListTile / kListThreads;
    int i = kPer * static_cast<int>(threadIdx.x);
    const int stop = i + kPer < len ? i + kPer : len;
    while (i < stop) {
        r0 = road_of(roads.combo_begin, r0, last, c_lo + i);
        const uint32_t nh = roads.nhits[r0];
        uint32_t at = static_cast<uint32_t>(c_lo + i - roads.combo_begin[r0]), n = 1;
#pragma unroll
        for (int l = 0; l < SVT_N_LAYERS; ++l) n *= nh_of(nh, l);
        for (; i < stop && at < n; ++i, ++at) {
            uint32_t k = at, digits = 0;
            for (int l = SVT_N_LAYERS - 1; l >= 0; --l) {  // layer 0 most significant
                const uint32_t nl = nh_of(nh, l);
                digits |= (k % nl) << (4 * l);
                k /= nl;
            }
            if (combo_road) combo_road[c_lo + i] = static_cast<int32_t>(r0);
            if (combo_hits) combo_hits[c_lo + i] = digits;
        }
    }
}

template <bool LOOP>
__global__ __launch_bounds__(kListThreads) void k_materialize(svt_roads roads, int64_t n_roads,
                                                              const int64_t *d_n_combos,
                                                              int64_t combo_cap,
                                                              int32_t *combo_road,
                                                              uint32_t *combo_hits,
                                                              uint64_t *err) {
    __shared__ int32_t s_begin[kListRoads];  // first combination, from the tile's first
    __shared__ uint32_t s_nh[kListRoads];
    __shared__ float s_inverse[16];
    __shared__ int64_t s_first;
    __shared__ int32_t s_end;
    if (has_error(err)) return;
    if (threadIdx.x < 16) s_inverse[threadIdx.x] = 1.0f / static_cast<float>(threadIdx.x);
    const bool wide = ((reinterpret_cast<uintptr_t>(combo_road) |
                        reinterpret_cast<uintptr_t>(combo_hits)) & 15) == 0;
    const int64_t total = *d_n_combos;
    if (total > combo_cap) return;
    for (int64_t c_lo = static_cast<int64_t>(blockIdx.x) * kListTile; c_lo < total;
         c_lo += static_cast<int64_t>(gridDim.x) * kListTile) {
        const int len = static_cast<int>(total - c_lo < kListTile ? total - c_lo : kListTile);
        if (threadIdx.x == 0)  // the road of the tile's first combination
            s_first = combo_road ? combo_road[c_lo] : road_of(roads.combo_begin, 0, n_roads - 1, c_lo);
        __syncthreads();
        int64_t r0 = s_first;
        for (int done = 0; done < len; r0 += kListRoads) {
            const int nr = static_cast<int>(n_roads - r0 < kListRoads ? n_roads - r0 : kListRoads);
            if (nr <= 0) break;  // (never on a consistent table)
            for (int j = threadIdx.x; j < nr; j += kListThreads) {
                const int64_t rel = roads.combo_begin[r0 + j] - c_lo;
                const uint32_t nh = roads.nhits[r0 + j];
                s_begin[j] = static_cast<int32_t>(rel < kListTile ? rel : kListTile);
                s_nh[j] = nh;
                if (j == nr - 1) {
                    const int64_t e = rel + roads.ncombo[r0 + j];
                    s_end = static_cast<int32_t>(e < len ? e : len);
                }
            }
            __syncthreads();
            const int end = s_end;
            // four consecutive combinations per lane: one search, then steps
            for (int i0 = (done & ~3) + 4 * static_cast<int>(threadIdx.x); i0 < end;
                 i0 += 4 * kListThreads) {
                const int first = i0 > done ? i0 : done;
                int lo = 0, hi = nr - 1;  // last road with begin <= first (it has combinations)
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (s_begin[mid] <= first) lo = mid; else hi = mid - 1;
                }
                uint32_t nh = s_nh[lo], digits = 0;
                uint32_t k = static_cast<uint32_t>(first - s_begin[lo]);
                // A caller's table may hold up to 15 hits a layer, 15^5 combinations a road.  k is below
                // nl * 15^4, so the quotient is below 2^16, k / nl in float is within 2^-7 of it, and a
                // quotient that is no whole number is at least 1/15 below the next: with 1/32 added it
                // rounds down to floor(k / nl).  (Three instructions; the 24-bit multiplication of
                // div_small holds for k < 2^15 only, a 32-bit one in its place costs 6.2e6
                // combinations 1 us of 31.)
#pragma unroll
                for (int l = SVT_N_LAYERS - 1; l > 0; --l) {  // layer 0 most significant
                    const uint32_t nl = nh_of(nh, l);
                    const uint32_t q = static_cast<uint32_t>(
                        __fmaf_rn(static_cast<float>(k), s_inverse[nl], 0.03125f));
                    digits |= (k - q * nl) << (4 * l);
                    k = q;
                }
                digits |= k;
                int32_t rd[4] = {0, 0, 0, 0};
                uint32_t ht[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = i0 + e;
                    if (i < first || i >= end) continue;
                    rd[e] = static_cast<int32_t>(r0 + lo);
                    ht[e] = digits;
                    // the next combination: carry from layer 4 to layer 0, then the next road that
                    // has combinations
                    digits += 1u << 16;
                    bool past = false;
#pragma unroll
                    for (int l = SVT_N_LAYERS - 1; l >= 0; --l)
                        if (nh_of(digits, l) == nh_of(nh, l)) {
                            digits &= ~(0xFu << (4 * l));
                            if (l > 0) digits += 1u << (4 * (l - 1));
                            past = l == 0;
                        } else {
                            break;
                        }
                    if (past && i + 1 < end) {
                        do ++lo;
                        while (lo < nr - 1 && s_begin[lo + 1] <= i + 1);
                        nh = s_nh[lo];
                        digits = 0;
                    }
                }
                if (wide && i0 >= done && i0 + 4 <= end) {
                    if (combo_road)
                        *reinterpret_cast<int4 *>(combo_road + c_lo + i0) =
                            make_int4(rd[0], rd[1], rd[2], rd[3]);
                    if (combo_hits)
                        *reinterpret_cast<uint4 *>(combo_hits + c_lo + i0) =
                            make_uint4(ht[0], ht[1], ht[2], ht[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (i0 + e >= first && i0 + e < end) {
                            if (combo_road) combo_road[c_lo + i0 + e] = rd[e];
                            if (combo_hits) combo_hits[c_lo + i0 + e] = ht[e];
                        }
                }
            }
            const int more = end > done ? end - done : 0;
            done += more;
            if (done < len && more < kListSparse && r0 + nr < n_roads) {
                list_sparse(roads, r0 + nr, n_roads - 1, c_lo + done, len - done, combo_road,
                            combo_hits);
                break;
            }
            __syncthreads();
        }
        if (!LOOP) break;
        __syncthreads();  // s_first is written again for the next tile
    }
}

// ---- plain fit: one lane per listed combination ------------------------------------------------
// The list may hold any combinations in any order; where it is the combine stage's, a tile of
// 2048 names few roads, whose table entries and coordinates then come from LDS (every lane
// gathering its own from memory took 86 us at 6.2e6 combinations, now 47 for 246 MB: 54 with 256
// threads that take 8 each, 61 with 64-bit indices checked one by one).  The constant bank is packed
// into LDS once per workgroup, in the pairs of the 16-bit dot products; with the offset split as
// q = qh * 2^s + ql every sum of 13-bit coordinates stays inside int32 (svt_fit.h), where 64-bit
// products ran at a quarter of the rate.  A caller's coordinates may be any int16: they are looked at
// when staged, and a tile with one outside 13 bits is summed in 64 bits (3000 events
// of 64 roads 45.5 us before this check and 46.3 with it, 2 more with every tile so).
constexpr int kFitThreads = 512;
constexpr int kFitLane = 4;
constexpr int kFitTile = kFitThreads * kFitLane;
constexpr int kFitRoads = 512;
constexpr int kFitCoords = 4096;

struct alignas(16) PlainSet {  // row j: f0|f1, f2|f3, f4|0, q; 112 bytes spread the LDS banks
    uint4 row[6];
    uint32_t pad[4];
};
// A road of the tile: where its coordinates are staged (-1: not all of them, or its set is not in
// the bank), hits per layer, set.
struct PlainRoad {
    int32_t at;
    uint32_t nh;
    int32_t set;
};

// c ^ (c >> 15) of a 13-bit coordinate is at most this
constexpr int32_t kInt13 = 4095;

__global__ __launch_bounds__(kFitThreads) void k_fit_plain(
    const svt_fconst *__restrict__ bank, svt_config cfg, svt_roads roads, int64_t n_roads,
    const int16_t *__restrict__ hit_coord, int64_t n_hits, const int32_t *__restrict__ combo_road,
    const uint32_t *__restrict__ combo_hits, int64_t n_combos, svt_fitrec out, uint64_t *err) {
    __shared__ PlainSet s_bank[256];
    __shared__ PlainRoad s_road[kFitRoads];
    __shared__ int16_t s_coord[kFitCoords + 1];  // (one past the end is read for a layer without hits)
    __shared__ int32_t s_lo[2], s_hi[2], s_wide[2];  // (s_wide: a staged coordinate needs 64-bit sums)
    const int tid = threadIdx.x;
    const int32_t shift = cfg.shift;
    const uint32_t qlmask = (1u << shift) - 1u;
    for (int i = tid; i < 6 * cfg.n_sets; i += kFitThreads) {
        const int set = i / 6, j = i - 6 * set;
        const int16_t *f = bank[set].f[j];
        s_bank[set].row[j] =
            make_uint4(static_cast<uint32_t>(pack16(f[0], f[1])),
                       static_cast<uint32_t>(pack16(f[2], f[3])),
                       static_cast<uint32_t>(pack16(f[4], 0)),
                       static_cast<uint32_t>(bank[set].q[j]));
    }
    if (tid < 2) {
        s_lo[tid] = INT32_MAX;
        s_hi[tid] = -1;
        s_wide[tid] = 0;
    }
    __syncthreads();
    int par = 0;
    for (int64_t t0 = static_cast<int64_t>(blockIdx.x) * kFitTile; t0 < n_combos;
         t0 += static_cast<int64_t>(gridDim.x) * kFitTile, par ^= 1) {
        int32_t r[kFitLane];
        uint32_t ph[kFitLane];
        int32_t lo = INT32_MAX, hi = -1;
#pragma unroll
        for (int e = 0; e < kFitLane; ++e) {
            const int64_t i = t0 + e * kFitThreads + tid;
            r[e] = i < n_combos ? combo_road[i] : -1;
            ph[e] = i < n_combos ? combo_hits[i] : 0;
            if (r[e] >= 0 && r[e] < n_roads) {
                lo = r[e] < lo ? r[e] : lo;
                hi = r[e] > hi ? r[e] : hi;
            }
        }
#pragma unroll
        for (int d = kWaveSize / 2; d > 0; d >>= 1) {
            const int32_t l2 = __shfl_xor(lo, d), h2 = __shfl_xor(hi, d);
            lo = l2 < lo ? l2 : lo;
            hi = h2 > hi ? h2 : hi;
        }
        if (lane_id() == 0) {
            atomicMin(&s_lo[par], lo);
            atomicMax(&s_hi[par], hi);
        }
        __syncthreads();
        lo = s_lo[par];
        hi = s_hi[par];
        const int span = hi >= lo && hi - lo < kFitRoads ? hi - lo + 1 : 0;
        if (tid == 0) {  // the other tile's bounds, for its next turn
            s_lo[par ^ 1] = INT32_MAX;
            s_hi[par ^ 1] = -1;
            s_wide[par ^ 1] = 0;
        }
        if (span > 0) {
            // coordinates staged: w_lo .. w_lo + wn - 1
            const int64_t w_lo = roads.hit_begin[lo];
            const int64_t w_hi = roads.hit_begin[hi] + SVT_N_LAYERS * SVT_MAX_HITS;
            int wn = 0;
            if (w_lo >= 0 && w_lo < n_hits && w_hi > w_lo) {
                const int64_t stop = w_hi < n_hits ? w_hi : n_hits;
                wn = static_cast<int>(stop - w_lo < kFitCoords ? stop - w_lo : kFitCoords);
                int32_t past = 0;
                for (int j = tid; j < wn; j += kFitThreads) {
                    const int16_t c = hit_coord[w_lo + j];
                    s_coord[j] = c;
                    past |= c ^ (c >> 15);
                }
                if (past > kInt13) s_wide[par] = 1;
            }
            for (int j = tid; j < span; j += kFitThreads) {
                const int64_t q = lo + j, at = roads.hit_begin[q] - w_lo;
                const uint32_t nh = roads.nhits[q];
                const int32_t set = roads.set[q];
                int n = 0;
#pragma unroll
                for (int l = 0; l < SVT_N_LAYERS; ++l) n += static_cast<int>(nh_of(nh, l));
                const bool in = at >= 0 && at + n <= wn && set >= 0 && set < cfg.n_sets;
                s_road[j] = PlainRoad{in ? static_cast<int32_t>(at) : -1, nh, set};
            }
        }
        __syncthreads();
        const bool wide_tile = __builtin_amdgcn_readfirstlane(s_wide[par]) != 0;
#pragma unroll
        for (int e = 0; e < kFitLane; ++e) {
            const int64_t i = t0 + e * kFitThreads + tid;
            if (i >= n_combos) break;
            if (r[e] < 0 || r[e] >= n_roads) { report(err, SVT_ERRCLASS_INDEX, i); continue; }
            PlainRoad rd{-1, 0, 0};
            if (span > 0) rd = s_road[r[e] - lo];
            bool ok = true, wide = wide_tile;
            int32_t x[SVT_N_LAYERS];
            if (rd.at >= 0) {
                int32_t off = rd.at;
#pragma unroll
                for (int l = 0; l < SVT_N_LAYERS; ++l) {
                    const uint32_t d = (ph[e] >> (4 * l)) & 0xFu, nl = nh_of(rd.nh, l);
                    ok &= d < nl;
                    x[l] = s_coord[off + static_cast<int32_t>(d < nl ? d : 0)];
                    off += static_cast<int32_t>(nl);
                }
            } else {
                rd = PlainRoad{0, roads.nhits[r[e]], roads.set[r[e]]};
                ok = rd.set >= 0 && rd.set < cfg.n_sets;
                int64_t off = roads.hit_begin[r[e]];
#pragma unroll
                for (int l = 0; l < SVT_N_LAYERS; ++l) {
                    const uint32_t d = (ph[e] >> (4 * l)) & 0xFu, nl = nh_of(rd.nh, l);
                    const int64_t idx = off + d;
                    ok &= d < nl && idx >= 0 && idx < n_hits;
                    x[l] = ok ? hit_coord[idx] : 0;
                    wide |= (x[l] ^ (x[l] >> 15)) > kInt13;
                    off += nl;
                }
            }
            if (!ok) { report(err, SVT_ERRCLASS_INDEX, i); continue; }
            const PlainSet &F = s_bank[rd.set];
            int32_t v[6];
            if (__builtin_amdgcn_ballot_w64(wide) == 0) {
                const int32_t x01 = pack16(x[0], x[1]), x23 = pack16(x[2], x[3]);
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const uint4 w = F.row[j];
                    int32_t acc = dot2(static_cast<int32_t>(w.x), x01,
                                       static_cast<int32_t>(w.w & qlmask));
                    acc = dot2(static_cast<int32_t>(w.y), x23, acc);
                    acc = dot2(static_cast<int32_t>(w.z), x[4], acc);
                    v[j] = (acc >> shift) + (static_cast<int32_t>(w.w) >> shift);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const uint4 w = F.row[j];
                    int64_t acc = static_cast<int32_t>(w.w);
                    acc += static_cast<int64_t>(static_cast<int16_t>(w.x)) * x[0];
                    acc += static_cast<int64_t>(static_cast<int16_t>(w.x >> 16)) * x[1];
                    acc += static_cast<int64_t>(static_cast<int16_t>(w.y)) * x[2];
                    acc += static_cast<int64_t>(static_cast<int16_t>(w.y >> 16)) * x[3];
                    acc += static_cast<int64_t>(static_cast<int16_t>(w.z)) * x[4];
                    v[j] = static_cast<int32_t>(acc >> shift);
                }
            }
            out.p0[i] = v[0];
            out.p1[i] = v[1];
            out.p2[i] = v[2];
            out.chi2[i] = static_cast<int64_t>(v[3]) * v[3] + static_cast<int64_t>(v[4]) * v[4] +
                          static_cast<int64_t>(v[5]) * v[5];
            if (out.c0) out.c0[i] = v[3];
            if (out.c1) out.c1[i] = v[4];
            if (out.c2) out.c2[i] = v[5];
        }
    }
}

// ---- select: cut, per-road best key (chi2 << 15 | k) and counts, kept-block counts -------
__global__ void k_best_init(svt_best best, int64_t n_roads) {
    for (int64_t r = gtid(); r < n_roads; r += gstride()) {
        reinterpret_cast<uint64_t *>(best.chi2)[r] = UINT64_MAX;
        best.n_accept[r] = 0;
    }
}

__global__ __launch_bounds__(kSegThreads) void k_select_mark(svt_config cfg, svt_roads roads,
                                                             int64_t n_roads,
                                                             const int32_t *__restrict__ combo_road,
                                                             const int64_t *__restrict__ chi2,
                                                             int64_t n_combos, uint8_t *accept,
                                                             svt_best best, int64_t *kb_counts,
                                                             uint64_t *err) {
    // four consecutive combinations per lane and load: each thread taking 16 of them one by one
    // read every line of chi2 from many instructions (93 us at 6.2e6 combinations, now 20)
    constexpr int kPer = kKeptBlock / kSegThreads / 4;
    __shared__ int32_t s_cnt[kSegThreads / kWaveSize];
    const int64_t nb = (n_combos + kKeptBlock - 1) / kKeptBlock;
    uint64_t *key = reinterpret_cast<uint64_t *>(best.chi2);
    const bool wide = (reinterpret_cast<uintptr_t>(chi2) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(accept) & 3) == 0;
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t base = b * kKeptBlock + 4 * static_cast<int64_t>(threadIdx.x);
        const bool full = wide && (b + 1) * kKeptBlock <= n_combos;
        int64_t c2[kPer][4];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = base + q * 4 * kSegThreads;
            if (full) {
                const longlong2 u = *reinterpret_cast<const longlong2 *>(chi2 + i);
                const longlong2 v = *reinterpret_cast<const longlong2 *>(chi2 + i + 2);
                c2[q][0] = u.x;
                c2[q][1] = u.y;
                c2[q][2] = v.x;
                c2[q][3] = v.y;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    c2[q][e] = i + e < n_combos ? chi2[i + e] : INT64_MAX;
            }
        }
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = base + q * 4 * kSegThreads;
            uint32_t bits = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                bits |= c2[q][e] <= cfg.chi2_cut && i + e < n_combos ? 1u << e : 0u;
            if (full) {
                *reinterpret_cast<uint32_t *>(accept + i) = mul_u24(bits, 0x204081u) & 0x01010101u;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < n_combos) accept[i + e] = (bits >> e) & 1u;
            }
            if (bits == 0) continue;
            cnt += __popc(bits);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!((bits >> e) & 1u)) continue;
                const int32_t r = combo_road[i + e];
                if (r < 0 || r >= n_roads) {
                    report(err, SVT_ERRCLASS_INDEX, i + e);
                    continue;
                }
                const int64_t k = i + e - roads.combo_begin[r];
                if (k < 0 || k >= (1 << kKeyKBits) || c2[q][e] < 0) {
                    report(err, SVT_ERRCLASS_INDEX, i + e);
                    continue;
                }
                const uint64_t kv = best_key(c2[q][e], static_cast<uint32_t>(k));
                atomicMin(reinterpret_cast<unsigned long long *>(key + r), kv);
                atomicAdd(best.n_accept + r, 1);
            }
        }
        if (kb_counts) {
            const int s = wave_sum(cnt);
            if (lane_id() == 0) s_cnt[threadIdx.x / kWaveSize] = s;
            __syncthreads();
            if (threadIdx.x == 0) {
                int64_t t = 0;
                for (int w = 0; w < kSegThreads / kWaveSize; ++w) t += s_cnt[w];
                kb_counts[b] = t;
            }
            __syncthreads();
        }
    }
}

// Parameters of combination k of road r, fitted again from the grouped coordinates and the
// road's constant set (the same integer arithmetic as the records, so the same values).
__device__ inline int64_t refit_combo(const svt_fconst *__restrict__ bank,
                                     const int16_t *__restrict__ coords, int32_t shift,
                                     uint32_t nh, int64_t hb, int32_t set, uint32_t k, int32_t *v,
                                     int rows) {
    uint32_t h[SVT_N_LAYERS];
#pragma unroll
    for (int l = SVT_N_LAYERS - 1; l >= 0; --l) {  // layer 0 most significant
        const uint32_t nl = nh_of(nh, l);
        h[l] = k % nl;
        k /= nl;
    }
    int64_t off = hb;
    int32_t x[SVT_N_LAYERS];
#pragma unroll
    for (int l = 0; l < SVT_N_LAYERS; ++l) {
        x[l] = coords[off + h[l]];
        off += nh_of(nh, l);
    }
    const svt_fconst &F = bank[set];
    for (int j = 0; j < rows; ++j) {
        int64_t acc = F.q[j];
#pragma unroll
        for (int l = 0; l < SVT_N_LAYERS; ++l)
            acc += static_cast<int64_t>(F.f[j][l]) * static_cast<int64_t>(x[l]);
        v[j] = static_cast<int32_t>(acc >> shift);
    }
    if (rows < 6) return 0;
    return static_cast<int64_t>(v[3]) * v[3] + static_cast<int64_t>(v[4]) * v[4] +
           static_cast<int64_t>(v[5]) * v[5];
}

// With bank and coords (batched path), the best track's parameters are fitted again from its
// hits instead of gathered from the three record arrays: one coordinate line per road instead
// of three scattered reads.
// With a scan job (job.data non-null), the grid's last block does that scan instead of roads:
// the kept list's per-block counts, in the same launch (it reads nothing the roads write).
__global__ __launch_bounds__(256) void k_best_finalize(svt_roads roads, Sizes n_roads_s,
                                                       svt_fitrec rec, Sizes n_combos_s,
                                                       svt_best best, int64_t cut, uint64_t *err,
                                                       int32_t skip_if_error,
                                                       const svt_fconst *bank,
                                                       const int16_t *coords, int32_t shift,
                                                       ScanJob job) {
    const int64_t road_blocks = job.data ? gridDim.x - 1 : gridDim.x;
    if (job.data && blockIdx.x == road_blocks) {
        __shared__ int64_t tmp[256 / kWaveSize + 1];
        if (skip_if_error && block_has_error(err)) {
            if (threadIdx.x == 0 && job.tot) *job.tot = -1;
            return;
        }
        const int64_t n = (load_size(job.n) + job.div - 1) / job.div;
        const int64_t carry = scan_column<256>(job.data, n, job.tot, tmp);
        if (threadIdx.x == 0 && job.cap >= 0 && carry > job.cap)
            report(err, SVT_ERRCLASS_CAPACITY, job.cap_index);
        return;
    }
    if (skip_if_error && has_error(err)) return;
    const int64_t n_roads = load_size(n_roads_s);
    const int64_t n_combos = load_size(n_combos_s);
    const int64_t stride = road_blocks * blockDim.x;
    for (int64_t r = gtid(); r < n_roads; r += stride) {
        uint64_t key = reinterpret_cast<uint64_t *>(best.chi2)[r];
        const int64_t cb = roads.combo_begin[r];
        const int64_t nc = roads.ncombo[r];
        if (key != UINT64_MAX && (key >> kKeyKBits) == kKeyChiMax && cb >= 0 &&
            nc <= (1 << kKeyKBits)) {
            // saturated key: exact scan of the road's records (chi2 >= 2^49 - 1 only)
            uint64_t bchi = UINT64_MAX;
            int64_t bk = 0;
            for (int64_t k = 0; k < nc && cb + k < n_combos; ++k) {
                int32_t vv[6];
                const int64_t c2 = rec.chi2 ? rec.chi2[cb + k]
                                            : refit_combo(bank, coords, shift, roads.nhits[r],
                                                          roads.hit_begin[r], roads.set[r],
                                                          static_cast<uint32_t>(k), vv, 6);
                if (c2 <= cut && c2 >= 0 && static_cast<uint64_t>(c2) < bchi) {
                    bchi = static_cast<uint64_t>(c2);
                    bk = k;
                }
            }
            if (bchi != UINT64_MAX) {
                const int64_t g = cb + bk;
                best.k[r] = static_cast<int32_t>(bk);
                best.chi2[r] = static_cast<int64_t>(bchi);
                if (rec.p0) {
                    best.p0[r] = rec.p0[g];
                    best.p1[r] = rec.p1[g];
                    best.p2[r] = rec.p2[g];
                } else {
                    int32_t vv[6];
                    refit_combo(bank, coords, shift, roads.nhits[r], roads.hit_begin[r],
                                roads.set[r], static_cast<uint32_t>(bk), vv, 3);
                    best.p0[r] = vv[0];
                    best.p1[r] = vv[1];
                    best.p2[r] = vv[2];
                }
                continue;
            }
            key = UINT64_MAX;
        }
        if (key == UINT64_MAX) {
            best.k[r] = -1;
            best.p0[r] = INT32_MIN;
            best.p1[r] = INT32_MIN;
            best.p2[r] = INT32_MIN;
            best.chi2[r] = INT64_MAX;
        } else {
            const int32_t k = static_cast<int32_t>(key & ((1u << kKeyKBits) - 1));
            const int64_t g = cb + k;
            best.k[r] = k;
            best.chi2[r] = static_cast<int64_t>(key >> kKeyKBits);
            const bool in = g >= 0 && g < n_combos && k < nc;
            if (bank && coords && in) {
                int32_t p[6];
                refit_combo(bank, coords, shift, roads.nhits[r], roads.hit_begin[r],
                            roads.set[r], static_cast<uint32_t>(k), p, 3);
                best.p0[r] = p[0];
                best.p1[r] = p[1];
                best.p2[r] = p[2];
            } else {
                best.p0[r] = in ? rec.p0[g] : INT32_MIN;
                best.p1[r] = in ? rec.p1[g] : INT32_MIN;
                best.p2[r] = in ? rec.p2[g] : INT32_MIN;
            }
        }
    }
}

// Accept flags of combinations base .. base + 15 as a bit mask (one 16-byte load when aligned).
__device__ inline uint32_t accept_bits16(const uint8_t *__restrict__ accept, int64_t base,
                                         int64_t n) {
    uint32_t bits = 0;
    if (base + 16 <= n && (reinterpret_cast<uintptr_t>(accept + base) & 15) == 0) {
        const uint4 v = *reinterpret_cast<const uint4 *>(accept + base);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                bits |= ((w[q] >> (8 * c)) & 0xFFu) ? (1u << (4 * q + c)) : 0u;
    } else {
        for (int e = 0; e < 16; ++e) {
            const int64_t i = base + e;
            if (i < n && accept[i]) bits |= 1u << e;
        }
    }
    return bits;
}

// ---- kept list: ascending indices of accepted combinations -------------------------------
__global__ __launch_bounds__(kSegThreads) void k_kept_write(const uint8_t *__restrict__ accept,
                                                            Sizes n_s,
                                                            const int64_t *__restrict__ kb_prefix,
                                                            int64_t *kept, int64_t kept_cap,
                                                            uint64_t *err) {
    __shared__ int64_t tmp[kSegThreads / kWaveSize + 1];
    const int64_t n = load_size(n_s);
    const int64_t nb = (n + kKeptBlock - 1) / kKeptBlock;
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t base = b * kKeptBlock + static_cast<int64_t>(threadIdx.x) * 16;
        uint32_t bits = accept_bits16(accept, base, n);
        int64_t tot;
        int64_t pos = block_excl_scan<int64_t, kSegThreads>(__popc(bits), tmp, tot) + kb_prefix[b];
        while (bits) {
            const int e = __ffs(bits) - 1;
            bits &= bits - 1;
            if (pos < kept_cap) kept[pos] = base + e;
            ++pos;
        }
    }
    (void)err;
}

// Kept-only mode: per block of kKeptBlock combinations, the accepted ones in ascending order.
// One wave per block (lane i reads the flags of combinations 64 i .. 64 i + 63 of the block), so
// that many blocks are in flight at once: the work per block is a short chain of dependent
// reads.  The block's accepted offsets are compacted in LDS and then spread evenly over the
// lanes.  The
// block's roads lie between the first road of its fit tile and the first road of the next tile;
// their combo_begin values are staged in the wave's LDS slice (up to kKeptRoads of them, else
// searched in place), each accepted combination finds its road by binary search and is fitted
// again from the grouped coordinates.
constexpr int kKeptRoads = 512;
__global__ __launch_bounds__(kSegThreads) void k_kept_refit(
    const uint8_t *__restrict__ accept, Sizes n_s, Sizes nr_s,
    const int64_t *__restrict__ kb_prefix, svt_roads roads,
    const int32_t *__restrict__ tile_first_road, int64_t tile_combos,
    const svt_fconst *__restrict__ bank, int32_t n_sets, const int16_t *__restrict__ coords,
    int32_t shift, int64_t *kept, svt_fitrec rec, int64_t kept_cap, uint64_t *err) {
    constexpr int kWaves = kSegThreads / kWaveSize;
    // After a data or capacity error the accept flags, the tile marks and the road table are
    // not (all) written: nothing here may be read.
    if (has_error(err)) return;
    __shared__ int64_t s_cb[kWaves][kKeptRoads];
    __shared__ uint16_t s_acc[kWaves][kKeptBlock];  // accepted offsets inside the block, in order
    const int wv = threadIdx.x / kWaveSize;
    const int lane = lane_id();
    const int64_t n = load_size(n_s);
    const int64_t n_roads = load_size(nr_s);
    const int64_t nb = (n + kKeptBlock - 1) / kKeptBlock;
    const int64_t n_tiles = (n + tile_combos - 1) / tile_combos;
    for (int64_t b = static_cast<int64_t>(blockIdx.x) * kWaves + wv; b < nb;
         b += static_cast<int64_t>(gridDim.x) * kWaves) {
        const int64_t base = b * kKeptBlock + static_cast<int64_t>(lane) * 64;
        uint64_t bits = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            bits |= static_cast<uint64_t>(accept_bits16(accept, base + 16 * q, n)) << (16 * q);
        const int cnt = __popcll(bits);
        const int incl = wave_incl_scan(cnt);
        const int tot = __shfl(incl, kWaveSize - 1);
        if (tot == 0) continue;  // uniform within the wave
        const int64_t pos0 = kb_prefix[b];
        uint16_t *acc_l = s_acc[wv];
        {
            int o = incl - cnt;
            uint64_t m = bits;
            while (m) {
                acc_l[o++] = static_cast<uint16_t>(lane * 64 + __builtin_ctzll(m));
                m &= m - 1;
            }
        }
        const int64_t t0 = (b * kKeptBlock) / tile_combos;
        const int64_t t1 = ((b + 1) * kKeptBlock - 1) / tile_combos + 1;
        const int64_t r_lo = tile_first_road[t0];
        const int64_t r_hi = t1 < n_tiles ? tile_first_road[t1] : n_roads - 1;
        if (r_lo < 0 || r_hi < r_lo || r_hi >= n_roads) {  // marks inconsistent with the roads
            if (lane == 0) report(err, SVT_ERRCLASS_INDEX, static_cast<uint64_t>(b * kKeptBlock));
            continue;
        }
        const int64_t nloc = r_hi - r_lo + 1;
        const bool staged = nloc <= kKeptRoads;
        int64_t *cb_l = s_cb[wv];
        if (staged)
            for (int64_t j = lane; j < nloc; j += kWaveSize) cb_l[j] = roads.combo_begin[r_lo + j];
        __builtin_amdgcn_wave_barrier();  // one wave: its LDS writes precede its reads
        // the block's accepted combinations, spread evenly over the lanes
        for (int j = lane; j < tot; j += kWaveSize) {
            const int64_t i = b * kKeptBlock + acc_l[j];
            const int64_t pos = pos0 + j;
            int64_t lo = 0, hi = nloc - 1;  // last road with combo_begin <= i
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                const int64_t cb = staged ? cb_l[mid] : roads.combo_begin[r_lo + mid];
                if (cb <= i) lo = mid; else hi = mid - 1;
            }
            const int64_t r = r_lo + lo;
            const int64_t k = i - (staged ? cb_l[lo] : roads.combo_begin[r]);
            const int32_t set = roads.set[r];
            if (k < 0 || k >= roads.ncombo[r] || set < 0 || set >= n_sets) {
                report(err, SVT_ERRCLASS_INDEX, static_cast<uint64_t>(i));
                continue;
            }
            if (pos < kept_cap) {
                int32_t v[6];
                const int64_t c2 = refit_combo(bank, coords, shift, roads.nhits[r],
                                               roads.hit_begin[r], set,
                                               static_cast<uint32_t>(k), v, 6);
                kept[pos] = i;
                if (rec.p0) rec.p0[pos] = v[0];
                if (rec.p1) rec.p1[pos] = v[1];
                if (rec.p2) rec.p2[pos] = v[2];
                if (rec.chi2) rec.chi2[pos] = c2;
                if (rec.c0) rec.c0[pos] = v[3];
                if (rec.c1) rec.c1[pos] = v[4];
                if (rec.c2) rec.c2[pos] = v[5];
            }
        }
        __builtin_amdgcn_wave_barrier();  // the slice is reused by the wave's next block
    }
}

// The header and the first n_roads per-road results of a batch, back to back in one buffer
// (layout in svt_gather_results).  When the buffer is host memory every store crosses the bus
// once; a closing system-scope fence in every thread that stored makes them visible to the
// host with the kernel's end (the grid is sized for the capacity, and the threads past the
// batch's roads store nothing and skip the costly fence).
__global__ void k_gather(svt_roads roads, svt_best best, int64_t road_cap, const int64_t *n_words,
                         const int64_t *n_roads, const int64_t *n_combos, const int64_t *n_kept,
                         const uint64_t *err, int64_t *out, int64_t out_roads) {
    const int64_t nr = *n_roads;
    if (gtid() == 0) {
        out[0] = *n_words;
        out[1] = nr;
        out[2] = *n_combos;
        out[3] = n_kept ? *n_kept : -1;
        out[4] = static_cast<int64_t>(*err);
        out[5] = out[6] = out[7] = 0;
    }
    if (nr >= 0 && nr <= out_roads && nr <= road_cap) {
        int64_t *chi2 = out + 8;
        int32_t *col = reinterpret_cast<int32_t *>(chi2 + nr);
        const int32_t *src[7] = {best.n_accept, best.k, best.p0, best.p1, best.p2, roads.event,
                                 roads.set};
        for (int64_t i = gtid(); i < nr; i += gstride()) {
            chi2[i] = best.chi2[i];
#pragma unroll
            for (int a = 0; a < 7; ++a) col[a * nr + i] = src[a][i];
        }
    }
    if (gtid() == 0 || gtid() < nr) __threadfence_system();
}

inline int64_t clamp_grid(int64_t blocks, int64_t maxb) {
    if (blocks < 1) return 1;
    return blocks < maxb ? blocks : maxb;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
hipError_t launch_scan(int64_t *data, Sizes n, int64_t div, int64_t *tot, int64_t cap,
                       uint32_t cap_index, uint64_t *err, bool skip_if_error, hipStream_t s) {
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, s, data, n, div, tot, cap, cap_index,
                       err, static_cast<int32_t>(skip_if_error));
    return hipGetLastError();
}

hipError_t launch_combo_count(const svt_roads &roads, Sizes n_roads, int64_t grid_blocks,
                              int64_t *rb_sums, uint64_t *err, hipStream_t s) {
    const int64_t g = grid_blocks < 1 ? 1 : grid_blocks;
    hipLaunchKernelGGL(k_combo_count, dim3(g), dim3(kRoadBlock), 0, s, roads, n_roads, rb_sums,
                       err);
    return hipGetLastError();
}

hipError_t launch_combo_begin(const svt_roads &roads, Sizes n_roads, int64_t grid_blocks,
                              const int64_t *rb_prefix, int32_t *combo_road, int64_t combo_cap,
                              uint64_t *err, hipStream_t s) {
    const int64_t g = grid_blocks < 1 ? 1 : grid_blocks;
    hipLaunchKernelGGL(k_combo_begin, dim3(g), dim3(kRoadBlock), 0, s, roads, n_roads, rb_prefix,
                       combo_road, combo_cap, err);
    return hipGetLastError();
}

hipError_t launch_materialize(const svt_roads &roads, int64_t n_roads, const int64_t *d_n_combos,
                              int64_t combo_cap, int32_t *combo_road, uint32_t *combo_hits,
                              uint64_t *err, hipStream_t s) {
    if (n_roads <= 0 || (!combo_road && !combo_hits)) return hipSuccess;
    if (combo_cap < 1) return hipSuccess;
    const int64_t tiles = (combo_cap - 1) / kListTile + 1;
    if (tiles <= kListGrid)
        hipLaunchKernelGGL(k_materialize<false>, dim3(static_cast<unsigned>(tiles)),
                           dim3(kListThreads), 0, s, roads, n_roads, d_n_combos, combo_cap,
                           combo_road, combo_hits, err);
    else
        hipLaunchKernelGGL(k_materialize<true>, dim3(kListGrid), dim3(kListThreads), 0, s, roads,
                           n_roads, d_n_combos, combo_cap, combo_road, combo_hits, err);
    return hipGetLastError();
}

hipError_t launch_fit_plain(const svt_fconst *bank, const svt_config &cfg,
                            const svt_roads &roads, int64_t n_roads, const int16_t *hit_coord,
                            int64_t n_hits, const int32_t *combo_road,
                            const uint32_t *combo_hits, int64_t n_combos, const svt_fitrec &out,
                            uint64_t *err, int num_cus, hipStream_t s) {
    if (n_combos <= 0) return hipSuccess;
    // 45 KB of LDS: three workgroups a compute unit
    const int64_t g = clamp_grid((n_combos + kFitTile - 1) / kFitTile, 3 * num_cus);
    hipLaunchKernelGGL(k_fit_plain, dim3(g), dim3(kFitThreads), 0, s, bank, cfg, roads, n_roads,
                       hit_coord, n_hits, combo_road, combo_hits, n_combos, out, err);
    return hipGetLastError();
}

hipError_t launch_select(const svt_config &cfg, const svt_roads &roads, int64_t n_roads,
                         const int32_t *combo_road, const svt_fitrec &rec, int64_t n_combos,
                         uint8_t *accept, const svt_best &best, int64_t *kb_counts,
                         uint64_t *err, hipStream_t s) {
    if (n_roads > 0) {
        const int64_t g = clamp_grid((n_roads + 255) / 256, 1 << 16);
        hipLaunchKernelGGL(k_best_init, dim3(g), dim3(256), 0, s, best, n_roads);
    }
    if (n_combos > 0) {
        const int64_t g = clamp_grid((n_combos + kKeptBlock - 1) / kKeptBlock, 1 << 16);
        hipLaunchKernelGGL(k_select_mark, dim3(g), dim3(kSegThreads), 0, s, cfg, roads, n_roads,
                           combo_road, rec.chi2, n_combos, accept, best, kb_counts, err);
    }
    if (n_roads > 0)
        return launch_best_finalize(roads, Sizes{n_roads, nullptr, n_roads}, rec,
                                    Sizes{n_combos, nullptr, n_combos}, best, cfg.chi2_cut, err,
                                    false, nullptr, nullptr, 0, ScanJob{}, s);
    return hipGetLastError();
}

hipError_t launch_best_finalize(const svt_roads &roads, Sizes n_roads, const svt_fitrec &rec,
                                Sizes n_combos, const svt_best &best, int64_t cut,
                                uint64_t *err, bool skip_if_error, const svt_fconst *bank,
                                const int16_t *coords, int32_t shift, const ScanJob &job,
                                hipStream_t s) {
    const int64_t g = clamp_grid((n_roads.cap + 255) / 256, 1 << 14) + (job.data ? 1 : 0);
    hipLaunchKernelGGL(k_best_finalize, dim3(g), dim3(256), 0, s, roads, n_roads, rec, n_combos,
                       best, cut, err, static_cast<int32_t>(skip_if_error), bank, coords, shift,
                       job);
    return hipGetLastError();
}

hipError_t launch_kept_write(const uint8_t *accept, Sizes n_combos, int64_t grid_blocks,
                             const int64_t *kb_prefix, int64_t *kept, int64_t kept_cap,
                             uint64_t *err, hipStream_t s) {
    const int64_t g = clamp_grid(grid_blocks, 1 << 16);
    hipLaunchKernelGGL(k_kept_write, dim3(g), dim3(kSegThreads), 0, s, accept, n_combos,
                       kb_prefix, kept, kept_cap, err);
    return hipGetLastError();
}

hipError_t launch_gather(const svt_roads &roads, const svt_best &best, int64_t road_cap,
                         const int64_t *d_n_words, const int64_t *d_n_roads,
                         const int64_t *d_n_combos, const int64_t *d_n_kept,
                         const uint64_t *d_err, void *out, int64_t out_roads, hipStream_t s) {
    const int64_t g = clamp_grid((out_roads + 255) / 256, 1024);
    hipLaunchKernelGGL(k_gather, dim3(g), dim3(256), 0, s, roads, best, road_cap, d_n_words,
                       d_n_roads, d_n_combos, d_n_kept, d_err, static_cast<int64_t *>(out),
                       out_roads);
    return hipGetLastError();
}

}  // namespace svt

namespace svt {
hipError_t launch_kept_refit(const uint8_t *accept, Sizes n_combos, Sizes n_roads,
                             int64_t grid_blocks, const int64_t *kb_prefix, const svt_roads &roads,
                             const int32_t *tile_first_road, int64_t tile_combos,
                             const svt_fconst *bank, int32_t n_sets, const int16_t *coords,
                             int32_t shift, int64_t *kept, const svt_fitrec &rec,
                             int64_t kept_cap, uint64_t *err, hipStream_t s) {
    // one wave per kept block, four per workgroup
    const int64_t g = clamp_grid((grid_blocks + 3) / 4, 1 << 16);
    hipLaunchKernelGGL(k_kept_refit, dim3(g), dim3(kSegThreads), 0, s, accept, n_combos, n_roads,
                       kb_prefix, roads, tile_first_road, tile_combos, bank, n_sets, coords,
                       shift, kept, rec, kept_cap, err);
    return hipGetLastError();
}
}  // namespace svt
