// The batched pass in two kernels over wave-sized units of hit words.
//
//   k_unit_count   reads every word once and counts, per unit of 256 words, the roads and events
//                  that start there and the combinations of those roads; the counts become
//                  running counts inside each of at most 512 ranges of units, and range totals.
//   k_unit_fit     one workgroup of 16 waves per compute unit; each scans the range totals, and
//                  then every wave takes units on its own and runs the loop nest of section II-A
//                  on them: unpack the words, write the road table, build the coordinate tables
//                  of the unit's roads, fit every combination, write the records, pick each
//                  road's best track.
//
// The end of the first kernel is the only point where waves wait for each other's counts, so no
// status words have to be cleared before a pass or polled in it, and the words, which are a
// twentieth of the records written, are read a second time instead of travelling to the second
// kernel as a road table and grouped coordinates.  Inside the fitting kernel nothing is shared
// between waves but the constant bank: a wave's chain of loads, LDS writes and scans overlaps
// the arithmetic and the stores of the 15 others.
//
// Measured on one GPU, us a pass: 3000 events of 64 roads 49 (four kernels before: a pre-pass with
// look-back, fits of flat tiles, best tracks, a reset: 75), 4000 events of 2048 roads 3940 (4510),
// 8192 uneven events with a kept list 237 (320), 100 events of 8 roads 17 back to back (23).
#include "svt_fit.h"
#include "svt_units.h"

namespace svt {
namespace {

constexpr int kThreads = kUnitWaves * kWaveSize;
constexpr int kEntries = kUnitSpan + 1;  // roads that start in a unit's span, and the end of the last

// ---- counting -----------------------------------------------------------------------------------
struct CArgs {
    const uint32_t *words;
    Sizes nw;
    int64_t *nw_copy;        // the word count for the later kernels (nw_copy[1] is the fit kernel's)
    uint32_t *ticket;        // units dealt out late, cleared here
    svt_config cfg;
    const svt_fconst *bank;  // nullable: unpack only
    UnitSet *sets;           // the packed bank
    UnitRec *rec;            // per unit
    RangeTot *tot;           // per range
    uint32_t *fine;          // per unit (fine_slices), of the first kPieces (nullable: not wanted)
    uint32_t *copy;          // words in device memory (nullable: they are there already)
    UnitKeep *keep;          // to start at no accepted combination (nullable: no kept list),
    unsigned long long *group;  // and the counts per kKeepGroup units
    int64_t n_group;
    SliceAcc *acc;           // to clear
    int64_t n_acc;
};

// Row j of a constant set in the fit's layout, for every set of the bank.
__device__ void pack_bank(const CArgs &a) {
    for (int s = threadIdx.x; s < a.cfg.n_sets; s += kThreads) {
        const svt_fconst &F = a.bank[s];
        int32_t f[30], q[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
#pragma unroll
            for (int l = 0; l < 5; ++l) f[5 * j + l] = F.f[j][l];
            q[j] = F.q[j];
        }
        UnitSet &o = a.sets[s];
#pragma unroll
        for (int j = 0; j < 6; ++j)
            o.row[j] = make_uint4(static_cast<uint32_t>(pack16(f[5 * j], f[5 * j + 1])),
                                  static_cast<uint32_t>(pack16(f[5 * j + 2], f[5 * j + 3])),
                                  static_cast<uint32_t>(pack16(f[5 * j + 4], 0)),
                                  static_cast<uint32_t>(q[j]));
        o.narrow = narrow_ok(f, q, a.cfg.shift) ? 1u : 0u;
    }
}

__device__ __forceinline__ uint64_t with_extra(uint32_t combos, uint32_t extra) {
    return combos | (static_cast<uint64_t>(extra) << kExtraShift);
}

// Bound by vector instructions, some 190 a unit, where there are many units (2.6e8 words: 0.42 ms,
// 2.4 TB/s; the pre-pass it replaces wrote 10 bytes a word more and took 1.55), by its latency where
// there are few (1.9e6 words: 7.7 us of which a launch that does nothing is half).  Two workgroups
// of 16 waves a compute unit: 64 registers a lane.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_unit_count(CArgs a) {
    __shared__ uint2 s_ent[kUnitWaves][kEntries + 1];
    __shared__ uint2 s_agg[2][kUnitWaves];
    __shared__ uint32_t s_err[3][kUnitWaves];
    const int wave = threadIdx.x / kWaveSize, lane = lane_id();
    const int64_t n = load_size(a.nw);
    const int64_t nu = (n + kUnitWords - 1) / kUnitWords;
    // with a bank, the last workgroup packs it and counts nothing
    const int ranges = static_cast<int>(gridDim.x) - (a.bank ? 1 : 0);
    if (a.keep)
        for (int64_t i = gtid(); i < a.n_group; i += gstride()) a.group[i * kKeepStride] = 0;
    for (int64_t i = gtid(); i < a.n_acc; i += gstride()) a.acc[i] = SliceAcc{0, 0, 0};
    if (static_cast<int>(blockIdx.x) == ranges) {
        if (threadIdx.x == 0) {
            *a.nw_copy = a.nw.dev ? *a.nw.dev : a.nw.host;
        }
        if (threadIdx.x < kDealers) a.ticket[threadIdx.x * kDealerStride] = 0;
        pack_bank(a);
        return;
    }
    const int64_t per = units_per_range(nu, ranges);
    const int64_t lo_u = per * blockIdx.x;
    const int64_t hi_u = lo_u + per < nu ? lo_u + per : nu;
    if (lo_u >= hi_u) {
        if (threadIdx.x == 0) a.tot[blockIdx.x] = RangeTot{0, 0, 0, ~0u, ~0u, ~0u, 0};
        return;
    }
    uint2 *S = s_ent[wave];
    const bool few = a.fine && nu < kPieces;
    uint32_t roads = 0, events = 0;  // of the range, before the units in hand
    uint64_t combos = 0;
    uint32_t fine_all = 0;
    uint32_t bad_word = ~0u, over_road = ~0u, set_road = ~0u;
    int buf = 0;
    for (int64_t u0 = lo_u; u0 < hi_u; u0 += kUnitWaves, buf ^= 1) {
        const int64_t u = u0 + wave;
        uint32_t agg = 0, cs = 0, my_over = ~0u, my_set = ~0u;
        if (u < hi_u) {
            const int64_t base = u * kUnitWords;
            const int nloc = static_cast<int>(n - base < kUnitSpan ? n - base : kUnitSpan);
            const UnitWords uw = load_unit(a.words, base, nloc);
            const int j0 = kUnitLane * lane;
            uint32_t top = 0;
#pragma unroll
            for (int e = 0; e < kUnitLane; ++e) top = w_layer(uw.w[e]) > top ? w_layer(uw.w[e]) : top;
            const bool bad = ballot(top >= static_cast<uint32_t>(SVT_N_LAYERS)) != 0;
            lds_order();
            UnitScan sc;
            if (nloc < kUnitSpan || bad)
                sc = enter_unit<true>(S, uw, nloc);
            else
                sc = enter_unit<false>(S, uw, nloc);
            const uint32_t nr = sc.roads;
            lds_order();
            if (a.copy) {
#pragma unroll
                for (int e = 0; e < kUnitLane; ++e)
                    if (j0 + e < kUnitWords && j0 + e < nloc) a.copy[base + j0 + e] = uw.w[e];
            }
            if (bad) {  // the first of the unit's own words with a bad layer
                uint32_t b = ~0u;
#pragma unroll
                for (int e = kUnitLane - 1; e >= 0; --e)
                    if (j0 + e < kUnitWords && j0 + e < nloc &&
                        w_layer(uw.w[e]) >= static_cast<uint32_t>(SVT_N_LAYERS))
                        b = static_cast<uint32_t>(base - lo_u * kUnitWords) + j0 + e;
                b = wave_min(b);
                bad_word = b < bad_word ? b : bad_word;
            }
            if (a.cfg.n_sets < 256) {
                uint32_t b = ~0u;
#pragma unroll
                for (int e = kUnitLane - 1; e >= 0; --e)
                    if (sc.road[e] < nr && j0 + e < nloc &&
                        w_rtag(uw.w[e]) >= static_cast<uint32_t>(a.cfg.n_sets))
                        b = sc.road[e];
                my_set = wave_min(b);
            }
            uint32_t csum = 0, ne = 0, y0 = uw.before;
            for (uint32_t r0 = 0; r0 < nr; r0 += kWaveSize) {
                const uint32_t rl = r0 + lane;
                const uint64_t mine = lanes_below(nr - r0 < kWaveSize ? nr - r0 : kWaveSize);
                bool over = false;
                uint32_t c = 0;
                uint2 e0 = make_uint2(0, 0);
                if (rl < nr) {
                    e0 = S[rl];
                    const uint32_t nh = road_hits(e0, S[rl + 1], a.cfg.max_hits, over);
                    c = over ? 0 : road_combos(nh);
                }
                ne += __popcll(ballot(starts_event(e0.y, y0)) & mine);
                y0 = lane_value(e0.y, 63);
                csum += c;
                const uint64_t m = ballot(over);
                if (m && my_over == ~0u) my_over = r0 + __builtin_ctzll(m);
            }
            cs = lane_value(scan64(csum), 63);
            agg = nr | (ne << 16);
        }
        if (lane == 0) s_agg[buf][wave] = make_uint2(agg, cs);
        __syncthreads();  // (the other buffer takes the next round's counts)
        // this wave's running counts: the waves before it, from 16 lanes (at most 16 * 256 roads
        // or events: 16 bits each)
        uint2 v = make_uint2(0, 0);
        if (lane < kUnitWaves) v = s_agg[buf][lane];
        const uint32_t past = v.y > 0 ? v.y - 1 : 0, more = past >> kSliceBits[2];
        const uint32_t sre = scan16(v.x), scn = scan16(v.y), sme = scan16(more);
        const uint32_t ex = lane_value(sre - v.x, wave), ex_c = lane_value(scn - v.y, wave),
                       ex_m = lane_value(sme - more, wave);
        if (few) {  // (these are the range's only units; for all batches it costs 2 us of 94)
            const uint32_t fine = (past >> kSliceBits[0]) | ((past >> kSliceBits[1]) << kFineBits);
            const uint32_t sf = scan16(fine), ex_f = lane_value(sf - fine, wave);
            if (u < hi_u && lane == 0) a.fine[u] = ex_f;
            fine_all = lane_value(sf, kUnitWaves - 1);
        }
        const uint32_t ex_r = ex & 0xFFFFu, ex_e = ex >> 16;
        if (u < hi_u) {
            if (lane == 0) {
                a.rec[u] = UnitRec{roads + ex_r, events + ex_e, combos + with_extra(ex_c, ex_m)};
                if (a.keep) a.keep[u].count = 0;
            }
            if (my_over != ~0u && over_road == ~0u) over_road = roads + ex_r + my_over;
            if (my_set != ~0u && set_road == ~0u) set_road = roads + ex_r + my_set;
        }
        const uint32_t all = lane_value(sre, kUnitWaves - 1);
        roads += all & 0xFFFFu;
        events += all >> 16;
        combos += with_extra(lane_value(scn, kUnitWaves - 1), lane_value(sme, kUnitWaves - 1));
    }
    if (lane == 0) {
        s_err[0][wave] = bad_word;
        s_err[1][wave] = over_road;
        s_err[2][wave] = set_road;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kUnitWaves; ++w) {
            bad_word = s_err[0][w] < bad_word ? s_err[0][w] : bad_word;
            over_road = s_err[1][w] < over_road ? s_err[1][w] : over_road;
            set_road = s_err[2][w] < set_road ? s_err[2][w] : set_road;
        }
        a.tot[blockIdx.x] =
            RangeTot{roads, events, combos, bad_word, over_road, set_road, fine_all};
    }
}

// ---- fitting ------------------------------------------------------------------------------------
struct UArgs {
    const uint32_t *words;   // in device memory
    int64_t *d_nw;           // the word count (nw_copy); d_nw[1]: for k_unit_keep (KArgs)
    int64_t word_cap;
    uint32_t *ticket;
    int32_t ranges;          // ranges the counting kernel dealt units to
    svt_config cfg;
    const UnitSet *sets;
    const UnitRec *rec;
    const RangeTot *tot;
    const uint32_t *fine;
    svt_roads roads;
    int64_t road_cap;
    svt_fitrec out;
    uint8_t *accept;
    svt_best best;
    int64_t combo_cap;
    int64_t *d_n_roads;
    int64_t *d_n_combos;
    uint64_t *err;
    UnitKeep *keep;          // nullable: no kept list
    unsigned long long *group;
    uint32_t *slots;         // slot_bytes per unit
    uint32_t slot_bytes;
    SliceAcc *acc;
};

// Slices of the given length before a unit, from the start of its range.
__device__ __forceinline__ uint32_t slices_before(const UnitRec *rec, const uint32_t *fine, int64_t u,
                                                  int step) {
    return step == 2 ? static_cast<uint32_t>(read_rec(rec, u).combos >> kExtraShift)
                     : fine_slices(in_memory(fine)[u], step);
}

constexpr int kTabCap = 768;   // coordinate-pair table entries of the roads fitted together
constexpr int kTabPad = 8;     // a dummy slot reads up to 7 entries before or after its table

// Per road with combinations, while its tables are in LDS (two 16-byte reads per lane):
//   a: division magic of n4 | 4 * n4 << 24; of n2 * n3 | n2 * n3 << 24; first combination, end (from
//      GB, the unit's first combination rounded down to a whole group)
//   b: its first group less its first item; hits per layer | road << 24; table of the (h0, h1)
//      pairs | of the (h2, h3) pairs << 16; table of layer 4 | constant set << 16 (tables in bytes)
struct RoadRow {
    uint4 a, b;
};

struct alignas(16) WaveLds {
    union {
        uint2 ent[kEntries];
        int32_t xt[kTabPad + kTabCap + kTabPad];
    };
    union {
        struct {
            uint32_t chi[4 * kWaveSize];
            uint32_t mark[kWaveSize];  // window item -> a road starts there (zero between uses)
        };
        uint32_t place[SVT_N_LAYERS * kUnitFitRoads];  // layer, road: where its words' coordinates go
    };
    RoadRow road[kUnitFitRoads];
    unsigned long long key[kUnitFitRoads];
    uint32_t nacc[kUnitFitRoads];
};

constexpr uint64_t kComboMask = (1ull << kExtraShift) - 1;
struct RangeBase {
    uint64_t roads;
    uint64_t combos;
    uint32_t events;
    uint32_t extra;   // slices past their unit's first, before the range
};
// Running counts at the start of every range, as each workgroup works them out for itself.
struct RangeLds {
    RangeBase base[kMaxRanges];
    uint64_t roads[kUnitWaves], combos[kUnitWaves], err[kUnitWaves], fine[kUnitWaves];
    uint32_t events[kUnitWaves], extra[kUnitWaves];
};
struct BatchTotals {
    int64_t n_roads, n_combos;
    uint64_t err;    // the first error found in the words, or a capacity that is too small
    uint32_t extra, events;
    int step;        // the slices' length: kSliceBits[step]
};

struct ULds {
    // The kernel's arguments, for what a unit uses once: held in scalar registers they would all
    // be live through the fit, which spills them and then vector registers too.
    UArgs args;
    UnitSet bank[256];
    RangeLds range;
    WaveLds w[kUnitWaves];
    uint32_t magic[72];
    uint32_t next;
};
static_assert(sizeof(ULds) <= 160 * 1024, "LDS of a compute unit");

// A lane fits groups of 2^kGroupBits consecutive combinations: 4 with records, whose int32 arrays
// take them as 16 bytes each; 8 without, which halves the windows and what each spends on finding
// the lanes' roads and first combinations (2000 events of 2048 roads: 955 us a pass with 4, 905
// with 8).
template <int REC>
constexpr int kGroupBits = REC == kRecNone ? 3 : 2;

// The rows of G consecutive combinations from their coordinate pairs.  J0..5: rows computed
// (the kept-only mode needs the chi-square rows only).
template <int MODE, int J0, int G>
struct FitGroup {
    int32_t v[6][G];
    uint64_t chi2[G];  // MODE == kFitNarrow: below 2^32
};

// One row of four combinations: (seed + three dot products) >> shift.  Written out because the
// compiler picks the accumulate-in-place form of the dot product, which copies the seed into
// every accumulator first (18 of about 130 instructions), and in this order because a dot
// product's result may be read by another kind of instruction only after three others.
__device__ __forceinline__ void row4(uint32_t f01, uint32_t f23, uint32_t f4, uint32_t seed,
                                     const int32_t *x01, const int32_t *x23, const int32_t *x4,
                                     int32_t shift, int32_t *v) {
    asm("v_dot2_i32_i16 %0, %4, %8, %7\n\t"
        "v_dot2_i32_i16 %1, %4, %9, %7\n\t"
        "v_dot2_i32_i16 %2, %4, %10, %7\n\t"
        "v_dot2_i32_i16 %3, %4, %11, %7\n\t"
        "v_dot2_i32_i16 %0, %5, %12, %0\n\t"
        "v_dot2_i32_i16 %1, %5, %13, %1\n\t"
        "v_dot2_i32_i16 %2, %5, %14, %2\n\t"
        "v_dot2_i32_i16 %3, %5, %15, %3\n\t"
        "v_dot2_i32_i16 %0, %6, %16, %0\n\t"
        "v_dot2_i32_i16 %1, %6, %17, %1\n\t"
        "v_dot2_i32_i16 %2, %6, %18, %2\n\t"
        "v_dot2_i32_i16 %3, %6, %19, %3\n\t"
        "v_ashrrev_i32 %0, %20, %0\n\t"
        "v_ashrrev_i32 %1, %20, %1\n\t"
        "v_ashrrev_i32 %2, %20, %2\n\t"
        "v_ashrrev_i32 %3, %20, %3"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
        : "v"(f01), "v"(f23), "v"(f4), "v"(seed), "v"(x01[0]), "v"(x01[1]), "v"(x01[2]),
          "v"(x01[3]), "v"(x23[0]), "v"(x23[1]), "v"(x23[2]), "v"(x23[3]), "v"(x4[0]), "v"(x4[1]),
          "v"(x4[2]), "v"(x4[3]), "v"(shift));
}

template <int MODE, int J0, int G>
__device__ __forceinline__ void fit_rows(const UnitSet &c, const int32_t *x01, const int32_t *x23,
                                         const int32_t *x4, int32_t shift, uint32_t qlmask,
                                         FitGroup<MODE, J0, G> &f) {
#pragma unroll
    for (int j = J0; j < 6; ++j) {
        const uint4 r = c.row[j];
        const uint32_t seed = MODE == kFitNarrow ? r.w : r.w & qlmask;
#pragma unroll
        for (int h = 0; h < G; h += 4)
            row4(r.x, r.y, r.z, seed, x01 + h, x23 + h, x4 + h, shift, f.v[j] + h);
        if (MODE != kFitNarrow) {
            const int32_t qh = static_cast<int32_t>(r.w) >> shift;
#pragma unroll
            for (int e = 0; e < G; ++e) f.v[j][e] += qh;
        }
    }
#pragma unroll
    for (int e = 0; e < G; ++e) {
        if (MODE == kFitNarrow)
            f.chi2[e] = static_cast<uint32_t>(
                mad_i24(f.v[5][e], f.v[5][e],
                        mad_i24(f.v[3][e], f.v[3][e], mad_i24(f.v[4][e], f.v[4][e], 0))));
        else
            f.chi2[e] = static_cast<uint64_t>(static_cast<int64_t>(f.v[3][e]) * f.v[3][e] +
                                              static_cast<int64_t>(f.v[4][e]) * f.v[4][e] +
                                              static_cast<int64_t>(f.v[5][e]) * f.v[5][e]);
    }
}

// One combination of a road from its tables, with 64-bit chi-square.
__device__ __forceinline__ Fit fit_one(const RoadRow &r, const UnitSet &c, const int32_t *xt,
                                       uint32_t k, int32_t shift, uint32_t qlmask) {
    const uint32_t n4 = r.a.x >> 26, n23 = r.a.y >> 24;
    const uint32_t q4 = div_small(k, r.a.x), h4 = k - q4 * n4;
    const uint32_t i01 = div_small(q4, r.a.y), i23 = q4 - i01 * n23;
    const int32_t x01 = *at_byte(xt + i01, r.b.z & 0xFFFFu), x23 = *at_byte(xt + i23, r.b.z >> 16),
                  x4 = *at_byte(xt + h4, r.b.w & 0xFFFFu);
    Fit f;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const uint4 w = c.row[j];
        int32_t acc = dot2(static_cast<int32_t>(w.x), x01, static_cast<int32_t>(w.w & qlmask));
        acc = dot2(static_cast<int32_t>(w.y), x23, acc);
        acc = dot2(static_cast<int32_t>(w.z), x4, acc);
        f.v[j] = (acc >> shift) + (static_cast<int32_t>(w.w) >> shift);
    }
    f.chi2 = static_cast<int64_t>(f.v[3]) * f.v[3] + static_cast<int64_t>(f.v[4]) * f.v[4] +
             static_cast<int64_t>(f.v[5]) * f.v[5];
    return f;
}

// Fit the combinations of roads c0 .. c1 - 1 of the unit, whose tables are in LDS, in windows of
// up to 64 items, from item from_item to before n_items.  An item is the part of a group of G
// consecutive combinations that lies in one road: item j of a road covers its group j, so a lane
// finds its road among the window's few by comparing with their first items, and fits with one
// road's constants.  A group cut by a road boundary is two or more neighbouring items; the lane of its
// first one collects the others' slots from the lanes after it, so that every group of the
// window is written by one lane with the same store instructions as its neighbours.
template <int MODE, int REC>
__device__ __forceinline__ void fit_windows(const UArgs &a, const ULds &L, WaveLds &W, int c0,
                                            int c1, uint32_t first_item, uint32_t from_item,
                                            uint32_t n_items, int64_t GB, int32_t shift,
                                            uint32_t qlmask, InMemory<uint32_t> *keep_at,
                                            uint32_t &kept) {
    constexpr int J0 = REC == kRecNone ? 3 : 0;
    // Windows end where a 128-byte line of the int32 record arrays does (8 groups): a line
    // written in two parts reaches memory in parts.  On 4000 events of 2048 roads windows that
    // end anywhere took 5.09 ms, at 8 groups 4.05 ms, at 32 (a line of accept bytes too) 4.34 ms.
    // Without records the lanes left idle weigh more (at 1, 2 and 4 groups of 8: 902, 908, 911 us).
    constexpr int G = 1 << kGroupBits<REC>;
    constexpr uint32_t kWhole = (1u << G) - 1u;
    constexpr int kLineGroups = REC == kRecNone ? 1 : 8;
    const int lane = lane_id();
    const uint32_t xt_at = lds_address(W.xt + kTabPad);
    const uint32_t cut32 = a.cfg.chi2_cut < 0xFFFFFFFFll ? static_cast<uint32_t>(a.cfg.chi2_cut)
                                                         : 0xFFFFFFFFu;
    const int32_t g_abs = static_cast<int32_t>(GB >> kGroupBits<REC>) & (kLineGroups - 1);
    int rcur = c0 - 1 + static_cast<int>(__popcll(
                            ballot(lane >= c0 && lane < c1 && first_item <= from_item)));
    for (uint32_t i0 = from_item; i0 < n_items;) {
        int nit = n_items - i0 < kWaveSize ? static_cast<int>(n_items - i0) : kWaveSize;
        const uint32_t i = i0 + lane;
        // the lane's road: the roads that start at or before its item, marked in LDS
        if (lane > rcur && lane < c1 && first_item - i0 < kWaveSize) W.mark[first_item - i0] = 1;
        lds_order();
        const uint32_t mk = W.mark[lane];
        const uint64_t starts = ballot(mk != 0);
        if (mk) W.mark[lane] = 0;
        const int ri = rcur + bits_below(starts) + static_cast<int>(mk);
        const uint4 ma = W.road[ri].a, mb = W.road[ri].b;
        const int32_t rb = static_cast<int32_t>(ma.z), end = static_cast<int32_t>(ma.w);
        const int32_t g = static_cast<int32_t>(i + mb.x);
        if (i0 + nit < n_items) {
            // end the window where a line of the record arrays ends, and at a whole group
            const int32_t gl = static_cast<int32_t>(lane_value(g, nit - 1)) + g_abs;
            const int32_t stop = (gl & ~(kLineGroups - 1)) - g_abs;
            nit = __popcll(ballot(g < stop) & (~0ull >> (kWaveSize - nit)));
        }
        const uint64_t active_m = ~0ull >> (kWaveSize - nit);  // (nit > 0)
        const bool active = __builtin_amdgcn_inverse_ballot_w64(active_m);
        const int32_t rel = G * g;
        const int32_t k0 = active ? rel - rb : 0, kc = k0 < 0 ? 0 : k0;
        uint32_t slots;  // the group's combinations that are the road's
        {
            const int32_t lo = kc - k0, hi = end - rel < G ? end - rel : G;
            slots = bit_field(active ? hi - lo : 0, lo);
        }
        // ---- the combinations' table entries, stepped with carries (a slot outside the road
        // reads a neighbouring entry and is not written)
        int32_t x01[G], x23[G], x4[G];
        {
            const uint32_t n4b = ma.x >> 24, n23 = ma.y >> 24;
            const uint32_t s4 = xt_at + (mb.w & 0xFFFFu), s23 = xt_at + (mb.z >> 16);
            const uint32_t q4 = div_small(static_cast<uint32_t>(kc), ma.x);
            const uint32_t i01 = div_small(q4, ma.y), i23 = q4 - mul_u24(i01, n23);
            uint32_t a4 = s4 + 4 * static_cast<uint32_t>(k0) - mul_u24(q4, n4b);  // < s4 before the road
            uint32_t a23 = s23 + 4 * i23, a01 = xt_at + (mb.z & 0xFFFFu) + 4 * i01;
            const uint32_t e4 = s4 + n4b, e23 = s23 + 4 * n23;
#pragma unroll
            for (int e = 0; e < G; ++e) {
                x01[e] = lds_read(a01);
                x23[e] = lds_read(a23);
                x4[e] = lds_read(a4);
                if (e < G - 1) {
                    a4 += 4;
                    const bool c4 = a4 == e4;
                    a4 = c4 ? s4 : a4;
                    a23 = c4 ? a23 + 4 : a23;
                    const bool c23 = a23 == e23;
                    a23 = c23 ? s23 : a23;
                    a01 = c23 ? a01 + 4 : a01;
                }
            }
        }
        FitGroup<MODE, J0, G> f;
        fit_rows<MODE, J0, G>(L.bank[mb.w >> 16], x01, x23, x4, shift, qlmask, f);
        uint32_t acc = 0;
        bool near = true;
        if (MODE == kFitNarrow) {
            uint32_t least = ~0u;
#pragma unroll
            for (int e = 0; e < G; ++e) {
                const uint32_t c = static_cast<uint32_t>(f.chi2[e]);
                least = c < least ? c : least;
            }
            near = ballot(least <= cut32) != 0 && a.cfg.chi2_cut >= 0;
        }
        if (near) {  // a chi-square of the window may pass
#pragma unroll
            for (int e = 0; e < G; ++e) {
                const bool ok = MODE == kFitNarrow
                                    ? static_cast<uint32_t>(f.chi2[e]) <= cut32
                                    : static_cast<int64_t>(f.chi2[e]) <= a.cfg.chi2_cut;
                acc |= ok ? 1u << e : 0u;
            }
            acc &= slots;
            const uint32_t cnt = static_cast<uint32_t>(__popc(acc));
            uint32_t pos = 0;
            if (REC == kRecNone || a.keep) {
                // in the order of the combinations: the lanes' items are, and their slots
                const uint64_t some = ballot(acc != 0);
                if (ballot(cnt > 1) == 0) {
                    pos = kept + bits_below(some);
                    kept += __popcll(some);
                } else {
                    const uint32_t upto = scan64(cnt);
                    pos = kept + upto - cnt;
                    kept += lane_value(upto, 63);
                }
            }
            if (acc) atomicAdd(&W.nacc[ri], cnt);
            // (slot by slot: taking a lane's accepted ones in a loop, each picked out of the registers,
            // costs as much with 4 and twice as much with 8)
#pragma unroll
            for (int e = 0; e < G; ++e)
                if ((acc >> e) & 1u) {
                    atomicMin(&W.key[ri],
                              static_cast<unsigned long long>(best_key(
                                  static_cast<int64_t>(f.chi2[e]), static_cast<uint32_t>(k0 + e))));
                    if ((REC == kRecNone || a.keep) && keep_at) {
                        const uint32_t c = static_cast<uint32_t>(rel + e);
                        if (REC == kRecNone) {
                            if (pos < a.slot_bytes / 16)
                                reinterpret_cast<InMemory<U32x4> *>(keep_at)[pos] =
                                    U32x4{c | (mb.w >> 16 << 24), static_cast<uint32_t>(x01[e]),
                                          static_cast<uint32_t>(x23[e]), static_cast<uint32_t>(x4[e])};
                        } else if (pos < a.slot_bytes / 4) {
                            keep_at[pos] = c;
                        }
                    }
                    ++pos;
                }
        }
        // ---- groups cut by a road boundary: the first item's lane takes the others' slots
        const uint32_t gp = dpp<kDppPrev>(static_cast<uint32_t>(g), ~0u);
        const uint64_t cont_m = ballot(static_cast<uint32_t>(g) == gp) & active_m & ~1ull;
        const bool cont = __builtin_amdgcn_inverse_ballot_w64(cont_m);
        for (uint64_t m = cont_m; m; m &= m >> 1) {
            // (a lane whose source is switched off keeps its value, so the lanes that give a
            // slot stay on with those that take it; what the givers are left with is not read)
            const uint32_t take = dpp<kDppNext>(cont ? slots | (acc << 8) : 0u);
            const uint32_t on = (take & ~slots) | (cont ? slots : 0u);
#pragma unroll
            for (int e = 0; e < G; ++e)
                if ((on >> e) & 1u) {
#pragma unroll
                    for (int j = J0; j < (REC == kRecRows ? 6 : 3); ++j)
                        f.v[j][e] = static_cast<int32_t>(
                            dpp<kDppNext>(static_cast<uint32_t>(f.v[j][e]),
                                          static_cast<uint32_t>(f.v[j][e])));
                    if (REC != kRecNone) {
                        const uint32_t l = static_cast<uint32_t>(f.chi2[e]);
                        uint32_t h = static_cast<uint32_t>(f.chi2[e] >> 32);
                        if (MODE != kFitNarrow) h = dpp<kDppNext>(h, h);
                        f.chi2[e] = (static_cast<uint64_t>(h) << 32) | dpp<kDppNext>(l, l);
                    }
                }
            slots |= take & 0xFFu;
            acc |= take >> 8;
        }
        // ---- records
        const bool head = __builtin_amdgcn_inverse_ballot_w64(active_m & ~cont_m);
        const uint32_t at = static_cast<uint32_t>(rel);  // from GB
        int32_t *p0 = a.out.p0 + GB, *p1 = a.out.p1 + GB, *p2 = a.out.p2 + GB;
        int64_t *pc = a.out.chi2 + GB;
        uint8_t *pa = a.accept + GB;
        if (head && slots == kWhole) {
            const uint32_t o1 = offset_of(at), o4 = offset_of(4 * at);
            if (REC != kRecNone) {
                store_nt(at_byte(p0, o4), f.v[0]);
                store_nt(at_byte(p1, o4), f.v[1]);
                store_nt(at_byte(p2, o4), f.v[2]);
                if (MODE != kFitNarrow) {
                    store_nt(pc + at, static_cast<int64_t>(f.chi2[0]),
                             static_cast<int64_t>(f.chi2[1]));
                    store_nt(pc + at + 2, static_cast<int64_t>(f.chi2[2]),
                             static_cast<int64_t>(f.chi2[3]));
                }
            }
            if (REC == kRecRows) {
                if (a.out.c0) store_nt(at_byte(a.out.c0 + GB, o4), f.v[3]);
                if (a.out.c1) store_nt(at_byte(a.out.c1 + GB, o4), f.v[4]);
                if (a.out.c2) store_nt(at_byte(a.out.c2 + GB, o4), f.v[5]);
            }
            constexpr uint32_t spread = 0x204081u, ones = 0x01010101u;  // a bit to a byte
            if (G == 4)
                *reinterpret_cast<uint32_t *>(at_byte(pa, o1)) = mul_u24(acc, spread) & ones;
            else
                *reinterpret_cast<U32Pair *>(at_byte(pa, o1)) =
                    U32Pair{mul_u24(acc & 0xFu, spread) & ones, mul_u24(acc >> 4, spread) & ones};
        } else if (head) {  // a group shared with the unit before or after this one
#pragma unroll
            for (int e = 0; e < G; ++e)
                if ((slots >> e) & 1u) {
                    if (REC != kRecNone) {
                        p0[at + e] = f.v[0][e];
                        p1[at + e] = f.v[1][e];
                        p2[at + e] = f.v[2][e];
                        if (MODE != kFitNarrow) pc[at + e] = static_cast<int64_t>(f.chi2[e]);
                    }
                    if (REC == kRecRows) {
                        if (a.out.c0) a.out.c0[GB + at + e] = f.v[3][e];
                        if (a.out.c1) a.out.c1[GB + at + e] = f.v[4][e];
                        if (a.out.c2) a.out.c2[GB + at + e] = f.v[5][e];
                    }
                    pa[at + e] = (acc >> e) & 1u;
                }
        }
        if (REC != kRecNone && MODE == kFitNarrow) {
            // A lane's four chi-squares are 32 bytes: stored from where they are, the wave's two
            // store instructions would each write every other 16 bytes of the lines they touch.
            // Through LDS each instruction writes whole lines.
            const int32_t g0 = static_cast<int32_t>(lane_value(g, 0));
            if (head)
                *reinterpret_cast<uint4 *>(W.chi + 4 * (g - g0)) =
                    make_uint4(static_cast<uint32_t>(f.chi2[0]), static_cast<uint32_t>(f.chi2[1]),
                               static_cast<uint32_t>(f.chi2[2]), static_cast<uint32_t>(f.chi2[3]));
            const int32_t first = rb > rel ? rb : rel, past = end < rel + 4 ? end : rel + 4;
            const int32_t w0 = static_cast<int32_t>(lane_value(first, 0)) - 4 * g0,
                          w1 = static_cast<int32_t>(lane_value(past, nit - 1)) - 4 * g0;
            lds_order();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int32_t t = 2 * lane + 2 * kWaveSize * h;
                const uint2 c = *reinterpret_cast<const uint2 *>(W.chi + t);
                int64_t *q = pc + 4 * g0;
                if (t >= w0 && t + 2 <= w1)
                    store_nt(at_byte(q, offset_of(8 * static_cast<uint32_t>(t))),
                             static_cast<int64_t>(c.x), static_cast<int64_t>(c.y));
                else if (t + 1 >= w0 && t < w1) {
                    if (t >= w0) q[t] = c.x;
                    if (t + 1 < w1) q[t + 1] = c.y;
                }
            }
            lds_order();
        }
        rcur = static_cast<int>(lane_value(static_cast<uint32_t>(ri), nit - 1));
        i0 += nit;
    }
}

// One unit, or with SLICED (a batch that has units cut into slices) one slice of a unit: its roads
// with combinations from the c0-th on, as many as the tables have room for.  Returns the first one
// left over, for a further call, or 0.
template <int REC, bool SLICED>
__device__ __forceinline__ int run_unit(const UArgs &hot, const ULds &L, WaveLds &W, int64_t u,
                                        uint32_t slice, int step, int c0, uint32_t &kept,
                                        int64_t n, int64_t per) {
    const int lane = lane_id();
    const int32_t shift = hot.cfg.shift;
    const uint32_t qlmask = (1u << shift) - 1u;
    const int64_t base = u * kUnitWords;
    const int nloc = static_cast<int>(n - base < kUnitSpan ? n - base : kUnitSpan);
    const UnitWords uw = load_unit(hot.words, base, nloc);
    const UnitRec rec = read_rec(L.args.rec, u);
    const RangeBase rbase = L.range.base[static_cast<uint32_t>(u) / static_cast<uint32_t>(per)];
    const bool table = c0 == 0 && (!SLICED || slice == 0);  // the unit's road table is to be written
    const int64_t R0 = static_cast<int64_t>(uni(rec.roads) + uni(rbase.roads));
    const int64_t CB0 = static_cast<int64_t>(uni(rec.combos) & kComboMask) +
                        static_cast<int64_t>(uni(rbase.combos));
    constexpr int kBits = kGroupBits<REC>;
    const int64_t GB = CB0 & ~((1ll << kBits) - 1);
    const uint32_t o = static_cast<uint32_t>(CB0 - GB);

    // ---- roads: entries, hits per layer, combinations, road table -------------------------------
    UnitScan sc;
    if (nloc < kUnitSpan)
        sc = enter_unit<true>(W.ent, uw, nloc);
    else
        sc = enter_unit<false>(W.ent, uw, nloc);
    const uint32_t nr = sc.roads;
    if (nr == 0) return 0;
    lds_order();
    uint32_t c_run = 0, ev_run = rec.events + rbase.events - 1, y0 = uw.before;
    int nf = 0;
    for (uint32_t r0 = 0; r0 < nr; r0 += kWaveSize) {
        const uint32_t rl = r0 + lane;
        const uint64_t mine_m = lanes_below(nr - r0 < kWaveSize ? nr - r0 : kWaveSize);
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(mine_m);
        uint32_t nh = 0, c = 0;
        uint2 e0 = make_uint2(0, 0);
        if (mine) {
            e0 = W.ent[rl];
            bool over;
            nh = road_hits(e0, W.ent[rl + 1], hot.cfg.max_hits, over);
            c = over ? 0 : road_combos(nh);
        }
        const uint32_t pos = entry_pos(e0), tag = (e0.y >> 16) & 0xFFu;
        const uint32_t cs = scan64(c);
        const uint32_t cb = c_run + cs - c;
        c_run += lane_value(cs, 63);
        const uint64_t em = ballot(starts_event(e0.y, y0)) & mine_m, fm = ballot(c > 0);
        y0 = lane_value(e0.y, 63);
        const int fi = nf + bits_below(fm);
        nf += __popcll(fm);
        const uint32_t evn = ev_run + bits_below(em) +
                             (__builtin_amdgcn_inverse_ballot_w64(em) ? 1u : 0u);
        ev_run += __popcll(em);
        if (mine) {
            // (for its words: its index among the roads that may be fitted now, past 63 for none)
            W.ent[rl].y = c > 0 ? static_cast<uint32_t>(fi - c0) : ~0u;
            if (c > 0) W.road[fi].b = make_uint4(o + cb, nh | (rl << 24), tag, 0);
        }
        if (mine && table) {
            const UArgs &a = L.args;
            const int64_t r = R0 + rl;
            in_memory(a.roads.event)[r] = static_cast<int32_t>(evn);
            in_memory(a.roads.set)[r] = static_cast<int32_t>(tag);
            in_memory(a.roads.hit_begin)[r] = base + pos;
            in_memory(a.roads.nhits)[r] = nh;
            in_memory(a.roads.ncombo)[r] = static_cast<int32_t>(c);
            in_memory(a.roads.combo_begin)[r] = CB0 + cb;
            if (c == 0) {
                in_memory(a.best.n_accept)[r] = 0;
                in_memory(a.best.k)[r] = -1;
                in_memory(a.best.p0)[r] = INT32_MIN;
                in_memory(a.best.p1)[r] = INT32_MIN;
                in_memory(a.best.p2)[r] = INT32_MIN;
                in_memory(a.best.chi2)[r] = INT64_MAX;
            }
        }
    }
    if (nf == 0) return 0;
    if (lane == 0) W.ent[nr].y = ~0u;  // (the same for words of no road of the unit)
    lds_order();

    // ---- words: rank among the road's hits on the layer, and the road's index; all entries are read
    // before the first is used
    uint32_t rank[kUnitLane], road_of[kUnitLane];
    {
        uint2 ent[kUnitLane];
        uint32_t hits = sc.hits;
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) ent[e] = W.ent[sc.road[e] < nr ? sc.road[e] : nr];
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) {
            rank[e] = __builtin_amdgcn_ubfe(hits - ent[e].x, 6 * w_layer(uw.w[e]), 4);
            road_of[e] = ent[e].y;
            hits += sc.hit[e];
        }
        if (nloc < kUnitSpan)
#pragma unroll
            for (int e = 0; e < kUnitLane; ++e)
                if (kUnitLane * lane + e >= nloc) road_of[e] = ~0u;
    }
    // ---- one road with combinations per lane: roads c0 .. c1 - 1 are fitted now -----------------
    const bool road = lane < nf && lane >= c0;
    W.key[lane] = ~0ull;
    W.nacc[lane] = 0;
    const uint4 pre = road ? W.road[lane].b : make_uint4(0, 0, 0, 0);
    lds_order();
    const uint32_t nh = pre.y, n4 = nh_of(nh, 4), n01 = nh_of(nh, 0) * nh_of(nh, 1),
                   n23 = nh_of(nh, 2) * nh_of(nh, 3);
    const uint32_t ntab = n01 + n23 + n4, rb = pre.x, end = rb + n01 * n23 * n4;
    const uint32_t n_it = road ? ((end - 1) >> kBits) - (rb >> kBits) + 1 : 0;
    const uint32_t tend = scan64(ntab);
    const bool take = road && tend <= kTabCap;
    const int c1 = c0 + __popcll(ballot(take));
    const uint32_t it_end = scan64(take ? n_it : 0);
    const uint32_t item = it_end - n_it;
    uint32_t n_items = lane_value(it_end, 63), from_item = 0;
    const bool narrow = ballot(take && !L.bank[pre.z].narrow) == 0;
    // groups ga .. gb - 1 of the unit are this slice's (the last slice takes what is left over)
    const int bits = SLICED ? kSliceBits[0] + 2 * step : kSliceBits[2];
    const uint32_t slices = SLICED && c_run > 1u << bits ? ((c_run - 1) >> bits) + 1 : 1;
    const int group_bits = bits - kBits;
    const uint32_t ga = slice << group_bits,
                   gb = slice + 1 < slices ? ga + (1u << group_bits) : ~0u >> 1;
    if (SLICED && slices > 1) {
        // the items are in the order of their groups: count those before ga and before gb
        const uint32_t g = rb >> kBits;
        uint32_t before = ga > g ? ga - g : 0, upto = gb > g ? gb - g : 0;
        before = take ? (before < n_it ? before : n_it) : 0;
        upto = take ? (upto < n_it ? upto : n_it) : 0;
        from_item = lane_value(scan64(before), 63);
        n_items = lane_value(scan64(upto), 63);
        if (from_item == n_items && c1 < nf) return c1;
    }
    if (take) {
        RoadRow row;
        const uint32_t t = tend - ntab;
        const uint32_t p01 = 4 * t, p23 = p01 + 4 * n01, p4 = p23 + 4 * n23;
        row.a = make_uint4(L.magic[n4] | (n4 << 26), L.magic[n23] | (n23 << 24), rb, end);
        row.b = make_uint4((rb >> kBits) - item, nh, p01 | (p23 << 16), p4 | (pre.z << 16));
        W.road[lane] = row;
        // Where a word's coordinate goes, by layer: bytes from the tables' start (12 bits), and on per
        // rank (6 bits, from bit 12); bytes from one entry to the next (6 bits, from 18); entries.
        const uint32_t n0 = nh_of(nh, 0), n1 = nh_of(nh, 1), n2 = nh_of(nh, 2), n3 = nh_of(nh, 3);
        uint32_t *place = W.place + (lane - c0);
        place[0] = p01 | (n1 << 14) | (4u << 18) | (n1 << 24);
        place[kUnitFitRoads] = (p01 + 2) | (4u << 12) | (n1 << 20) | (n0 << 24);
        place[2 * kUnitFitRoads] = p23 | (n3 << 14) | (4u << 18) | (n3 << 24);
        place[3 * kUnitFitRoads] = (p23 + 2) | (4u << 12) | (n3 << 20) | (n2 << 24);
        place[4 * kUnitFitRoads] = p4 | (4u << 12) | (1u << 24);
    }
    lds_order();
    // Tables of coordinate pairs, (x0 | x1 << 16) at h0 * n1 + h1 and the same for layers 2 and 3,
    // and of layer 4: each word writes its half of the entries it belongs to, the lane's words
    // side by side.
    {
        char *xt = reinterpret_cast<char *>(W.xt + kTabPad);
        uint32_t cnt[kUnitLane], step[kUnitLane], at[kUnitLane], most = 0;
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e)
            at[e] = W.place[w_layer(uw.w[e]) * kUnitFitRoads + (road_of[e] & (kUnitFitRoads - 1))];
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) {
            const uint32_t pl = at[e];
            cnt[e] = road_of[e] < static_cast<uint32_t>(c1 - c0) ? pl >> 24 : 0u;
            step[e] = (pl >> 18) & 0x3Fu;
            at[e] = (pl & 0xFFFu) + mul_u24(rank[e], (pl >> 12) & 0x3Fu);
            most = cnt[e] > most ? cnt[e] : most;
        }
        for (uint32_t r = 0; ballot(r < most); ++r)
#pragma unroll
            for (int e = 0; e < kUnitLane; ++e) {
                if (r < cnt[e])
                    *reinterpret_cast<int16_t *>(xt + at[e]) = static_cast<int16_t>(w_coord(uw.w[e]));
                at[e] += step[e];
            }
    }
    lds_order();
    W.mark[lane] = 0;
    lds_order();
    InMemory<uint32_t> *keep_at = nullptr;
    if ((REC == kRecNone || hot.keep) && slices == 1)
        keep_at = in_memory(L.args.slots) + u * (hot.slot_bytes / 4);
    if (narrow)
        fit_windows<kFitNarrow, REC>(hot, L, W, c0, c1, item, from_item, n_items, GB, shift,
                                     qlmask, keep_at, kept);
    else
        fit_windows<kFitSplit, REC>(hot, L, W, c0, c1, item, from_item, n_items, GB, shift,
                                    qlmask, keep_at, kept);
    lds_order();

    // ---- best tracks ----------------------------------------------------------------------------
    if (lane >= c0 && lane < c1) {
        const RoadRow row = W.road[lane];
        unsigned long long key = W.key[lane];
        uint32_t nacc = W.nacc[lane];
        bool whole = true;
        if (SLICED && slices > 1) {
            // a road with groups in other slices too: every one of them adds what it found, and
            // the last to do so has the whole of it
            const uint32_t g_first = row.a.z >> kBits, g_last = (row.a.w - 1) >> kBits;
            const bool touched = g_last >= ga && g_first < gb;
            const bool cut = touched && (g_first < ga || g_last >= gb);
            whole = touched && !cut;
            if (cut) {
                const uint32_t s0 = g_first >> group_bits;
                uint32_t s1 = g_last >> group_bits;
                s1 = s1 < slices ? s1 : slices - 1;
                // the batch's number of the slice after the road's first one
                const uint32_t x = slices_before(L.args.rec, L.args.fine, u, step) +
                                   L.range.base[static_cast<uint32_t>(u) / static_cast<uint32_t>(per)]
                                       .extra + s0;
                // Everything here is an atomic at agent scope, so it is enough that the first two are
                // done before the third starts; a fence would also write back what the L2 holds of
                // the records (37 uneven events: 23.5 us with fences, 19.3 without; 1900 units cut in
                // two: 241 and 24).
                InMemory<SliceAcc> *acc = in_memory(L.args.acc) + x;
                __hip_atomic_fetch_max(&acc->key, ~key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(&acc->nacc, nacc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                whole = (__hip_atomic_fetch_add(&acc->arrived, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) & 0xFFu) == s1 - s0;
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (whole) {
                    key = ~__hip_atomic_load(&acc->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    nacc = __hip_atomic_load(&acc->nacc, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (whole) {
            const UArgs &a = L.args;
            const int64_t r = R0 + (row.b.y >> 24);
            const UnitSet &c = L.bank[row.b.w >> 16];
            const int32_t *xt = W.xt + kTabPad;
            int32_t k = -1, v0 = INT32_MIN, v1 = INT32_MIN, v2 = INT32_MIN;
            int64_t chi2 = INT64_MAX;
            if (key != ~0ull && (key >> kKeyKBits) == kKeyChiMax) {
                // saturated key (chi2 >= 2^49 - 1, extreme constants only): exact rescan
                for (uint32_t q = 0; q < row.a.w - row.a.z; ++q) {
                    const int64_t c2 = fit_one(row, c, xt, q, shift, qlmask).chi2;
                    if (c2 <= a.cfg.chi2_cut && c2 < chi2) {
                        chi2 = c2;
                        k = static_cast<int32_t>(q);
                    }
                }
            } else if (key != ~0ull) {
                k = static_cast<int32_t>(key & ((1u << kKeyKBits) - 1));
                chi2 = static_cast<int64_t>(key >> kKeyKBits);
            }
            if (k >= 0) {
                const Fit f = fit_one(row, c, xt, static_cast<uint32_t>(k), shift, qlmask);
                v0 = f.v[0];
                v1 = f.v[1];
                v2 = f.v[2];
            }
            in_memory(a.best.n_accept)[r] = static_cast<int32_t>(nacc);
            in_memory(a.best.k)[r] = k;
            in_memory(a.best.p0)[r] = v0;
            in_memory(a.best.p1)[r] = v1;
            in_memory(a.best.p2)[r] = v2;
            in_memory(a.best.chi2)[r] = chi2;
        }
    }
    lds_order();
    if (c1 < nf) return c1;
    if ((REC == kRecNone || hot.keep) && kept > 0 && lane == 0) {
        InMemory<UnitKeep> *k = in_memory(L.args.keep) + u;
        const uint32_t most = hot.slot_bytes / (REC == kRecNone ? 16 : 4);
        k->size = nr | (c_run << kKeepRoadBits) | (slices > 1 ? kKeepCut : 0u);
        k->combo = static_cast<uint64_t>(CB0);
        k->road = static_cast<uint32_t>(R0);
        if (slices > 1) {
            const uint32_t x =
                slices_before(L.args.rec, L.args.fine, u, step) +
                L.range.base[static_cast<uint32_t>(u) / static_cast<uint32_t>(per)].extra;
            k->acc = x;
            __hip_atomic_fetch_add(&k->count, kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (slice + 1 < slices)
                __hip_atomic_fetch_add(&in_memory(L.args.acc)[x + slice].arrived, kept << 8,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            k->count = kept | (kept > most ? kKeepSearch : 0u);
        }
        __hip_atomic_fetch_add(in_memory(L.args.group) + u / kKeepGroup * kKeepStride,
                               static_cast<unsigned long long>(kept), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    return 0;
}

// The unit and slice of the batch's extra slice number e (slices past their unit's first, counted
// in the units' order).  One wave; 64 units or ranges are compared at a time.
__device__ int64_t find_extra(const UArgs &a, const ULds &L, uint32_t e, int64_t nu, int64_t per,
                              int n_ranges, int step, uint32_t &slice) {
    const int lane = lane_id();
    int r = -1;  // last range whose extras start at or before e
    for (int r0 = 0; r0 < n_ranges; r0 += kWaveSize)
        r += __popcll(ballot(r0 + lane < n_ranges && L.range.base[r0 + lane].extra <= e));
    e -= uni(L.range.base[r].extra);
    const int64_t lo = r * per, hi = lo + per < nu ? lo + per : nu;
    int64_t u = lo - 1;  // last unit whose extras start at or before e
    uint32_t first = 0;
    for (int64_t u0 = lo; u0 < hi; u0 += kWaveSize) {
        uint32_t x = ~0u;
        if (u0 + lane < hi) x = slices_before(a.rec, a.fine, u0 + lane, step);
        const uint64_t m = ballot(x <= e);  // a prefix of the lanes
        if (m == 0) break;
        u += __popcll(m);
        first = lane_value(x, 63 - __builtin_clzll(m));
    }
    slice = e - first + 1;
    return u;
}

// The wave's units (unit_share).  The last eighth is divided among the dealers and goes by ticket to the
// waves that finish first (one counter for all of them would hand out a unit every 12 ns: 93 us for
// 7500 units, 51 with 32).  Slices past their unit's first come before everything else, dealt out to
// the workgroups in turn.
template <int REC, bool SLICED>
__device__ __forceinline__ void run_units(const UArgs &a, ULds &L, int64_t n, int64_t nu,
                                          int64_t per, int n_ranges, uint32_t extra, int step) {
    const int wave = threadIdx.x / kWaveSize, lane = lane_id();
    const UnitShare share = unit_share(nu, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
    const uint32_t my_extra =
        SLICED && extra > blockIdx.x ? (extra - blockIdx.x - 1) / gridDim.x + 1 : 0;
    bool late = false;
    int64_t u = 0, past = 0;
    while (true) {
        uint32_t slice = 0;
        if (u >= past) {
            uint32_t k = 0;
            if (!late) {
                if (lane == 0) k = atomicAdd(&L.next, 1u);
                k = uni(k);
                if (SLICED && k < my_extra) {
                    u = find_extra(a, L, blockIdx.x + k * gridDim.x, nu, per, n_ranges, step, slice);
                } else {
                    u = share.lo + (k - my_extra);
                    late = u >= share.hi;
                }
                past = u + 1;
            }
            if (late) {
                if (share.p_lo >= share.p_hi) break;
                if (lane == 0) k = atomicAdd(a.ticket + share.dealer * kDealerStride, 1u);
                u = share.p_lo + uni(k) * share.batch;
                past = u + share.batch < share.p_hi ? u + share.batch : share.p_hi;
                if (u >= share.p_hi) break;
            }
        }
        int c = 0;
        uint32_t kept = 0;
        do {
            c = run_unit<REC, SLICED>(a, L, L.w[wave], u, slice, step, c, kept, n, per);
        } while (c != 0);
        ++u;
    }
}

// Scan the totals of the ranges, whose totals t the first threads have loaded (`per` units each);
// all threads of the workgroup.
__device__ __forceinline__ BatchTotals scan_ranges(const RangeTot &t, int ranges, int64_t nu,
                                                   int64_t per,
                                                   int64_t nw, int64_t word_cap, int64_t road_cap,
                                                   int64_t combo_cap, int pieces, RangeLds &L) {
    const int tid = threadIdx.x, wave = tid / kWaveSize, lane = lane_id();
    const int waves = (ranges + kWaveSize - 1) / kWaveSize;  // that hold ranges, at most 8
    const uint64_t cc = t.combos & kComboMask;
    const uint32_t ee = static_cast<uint32_t>(t.combos >> kExtraShift);
    uint64_t fine_before = 0;  // slices of 512, and of 2048 in the upper half
    RangeBase b{};
    if (wave < waves) {
        const uint64_t ir = scan64(static_cast<uint64_t>(t.roads)), ic = scan64(cc);
        const uint32_t iv = scan64(t.events), ie = scan64(ee);
        b = RangeBase{ir - t.roads, ic - cc, iv - t.events, ie - ee};
        const uint64_t f = fine_slices(t.fine, 0) |
                           (static_cast<uint64_t>(fine_slices(t.fine, 1)) << 32);
        const uint64_t sf = scan64(f);
        fine_before = sf - f;
        if (lane == kWaveSize - 1) {
            L.fine[wave] = sf;
            L.roads[wave] = ir;
            L.combos[wave] = ic;
            L.events[wave] = iv;
            L.extra[wave] = ie;
        }
        // the first error, in the ranges' order; a road's index from the wave's first range
        uint64_t err = SVT_NO_ERROR;
        const bool bad = tid < ranges && (t.bad_word & t.over_road & t.set_road) != ~0u;
        if (ballot(bad)) {
            auto note = [&](uint64_t cls, uint32_t idx, uint64_t from) {
                const uint64_t v = (cls << 56) | (from + idx);
                if (bad && idx != ~0u && v < err) err = v;
            };
            note(SVT_ERRCLASS_LAYER, t.bad_word, static_cast<uint64_t>(tid * per) * kUnitWords);
            note(SVT_ERRCLASS_HITS, t.over_road, b.roads);
            note(SVT_ERRCLASS_SET, t.set_road, b.roads);
#pragma unroll
            for (int d = kWaveSize / 2; d > 0; d >>= 1) {
                const uint64_t ov = __shfl_xor(err, d, kWaveSize);
                err = ov < err ? ov : err;
            }
        }
        if (lane == 0) L.err[wave] = err;
    }
    __syncthreads();
    BatchTotals all{0, 0, SVT_NO_ERROR, 0, 0, 2};
    uint64_t first = SVT_NO_ERROR, fine_all = 0;
    for (int w = 0; w < waves; ++w) {
        uint64_t e = L.err[w];
        if (e != SVT_NO_ERROR && (e >> 56) != SVT_ERRCLASS_LAYER)
            e += static_cast<uint64_t>(all.n_roads);  // roads before the wave's ranges
        first = e < first ? e : first;
        if (w == wave) {
            b.roads += static_cast<uint64_t>(all.n_roads);
            b.combos += static_cast<uint64_t>(all.n_combos);
            b.events += all.events;
            b.extra += all.extra;
            fine_before += fine_all;
        }
        all.n_roads += static_cast<int64_t>(L.roads[w]);
        all.n_combos += static_cast<int64_t>(L.combos[w]);
        all.events += L.events[w];
        all.extra += L.extra[w];
        fine_all += L.fine[w];
    }
    if (nu < pieces) {  // the smallest slices that leave at most `pieces` (and so fit their accumulators)
        const uint32_t room = pieces - static_cast<uint32_t>(nu);
        const uint32_t e0 = static_cast<uint32_t>(fine_all), e1 = static_cast<uint32_t>(fine_all >> 32);
        if (e0 <= room) {
            all.step = 0;
            all.extra = e0;
            b.extra = static_cast<uint32_t>(fine_before);
        } else if (e1 <= room) {
            all.step = 1;
            all.extra = e1;
            b.extra = static_cast<uint32_t>(fine_before >> 32);
        }
    }
    if (tid < ranges) L.base[tid] = b;
    auto cap_err = [](uint64_t i) {
        return (static_cast<uint64_t>(SVT_ERRCLASS_CAPACITY) << 56) | i;
    };
    if (nw > word_cap) all.err = cap_err(3);
    if (all.n_combos > combo_cap) all.err = cap_err(1);
    if (all.n_roads > road_cap) all.err = cap_err(0);
    all.err = first < all.err ? first : all.err;
    __syncthreads();
    return all;
}

// What bounds it: with records the stores of large batches (2e9 combinations: 44.7 GB in 9.45 ms,
// 4.73 TB/s, where a copy of 4 GiB moves 4.78 and these stores alone 5.4), at 7500 units the
// issue of vector instructions, 2000 a unit of which 0.4 unpack, and the last units' run-out (43 us
// for 151 MB); without records the vector instructions (2e5 units: 4.15e8 wave instructions in 790
// us).  One workgroup of 16 waves a compute unit is what LDS holds: 7 KB a wave and 42 KB for all.
template <int REC>
__global__ __launch_bounds__(kThreads) void k_unit_fit(UArgs a) {
    __shared__ ULds L;
    const int tid = threadIdx.x;
    // everything from memory at once: nothing here waits for the word count
    RangeTot t{};
    if (tid < a.ranges) t = a.tot[tid];
    const int64_t nw = *a.d_nw;
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(a.sets);
        uint4 *dst = reinterpret_cast<uint4 *>(L.bank);
        const int n16 = a.cfg.n_sets * static_cast<int>(sizeof(UnitSet) / 16);
        for (int i = tid; i < n16; i += kThreads) dst[i] = src[i];
    }
    if (tid < 72) L.magic[tid] = magic_of(tid > 0 ? static_cast<uint32_t>(tid) : 1u);
    if (tid == 0) L.next = 0;
    {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(
            (const void *)__builtin_amdgcn_kernarg_segment_ptr());
        if (tid < static_cast<int>(sizeof(UArgs) / 4))
            reinterpret_cast<uint32_t *>(&L.args)[tid] = src[tid];
    }
    const int64_t n = nw < 0 ? 0 : nw > a.word_cap ? a.word_cap : nw;
    const int64_t nu = (n + kUnitWords - 1) / kUnitWords;
    const int64_t per = units_per_range(nu, a.ranges);
    const int n_ranges = a.ranges;
    const BatchTotals all =
        scan_ranges(t, a.ranges, nu, per, nw, a.word_cap, a.road_cap, a.combo_cap,
                    REC == kRecNone ? kPiecesKeptOnly : kPieces, L.range);
    if (blockIdx.x == 0 && tid == 0) {
        *a.err = all.err;
        a.d_nw[1] = all.err != SVT_NO_ERROR ? -1 : kSliceBits[0] + 2 * all.step;
        *a.d_n_roads = all.n_roads;
        *a.d_n_combos = all.n_combos;
    }
    if (all.err != SVT_NO_ERROR) return;

    const uint32_t extra = uni(all.extra);
    if (extra == 0)
        run_units<REC, false>(a, L, n, nu, per, n_ranges, extra, 0);
    else
        run_units<REC, true>(a, L, n, nu, per, n_ranges, extra, all.step);
}

// ---- the kept list ---------------------------------------------------------------------------------
// The accepted combinations in ascending order, and in kept-only mode (ONLY) their fit values.  A
// workgroup takes kKeepGroup units: the groups' counts before it give its place in the list, its
// units' counts theirs.  The accepted combinations of all its units are then spread over the
// threads, each fitting from the coordinates that the unit's wave left (neither the accept flags
// nor the road table is read: with those, scan and refit took 410 us behind the fits of 4e8
// combinations).
//
// Whether the fits ran is read from a word that only the fitting kernel writes: a list that is too
// short is reported in the error word by this kernel, while other workgroups start.  With records the
// list then holds its first kept_cap entries; in kept-only mode nothing is written to it.
struct KArgs {
    const int64_t *d_nw;   // word count; [1]: bits of the slices' length, -1 if the batch has an error
    int64_t word_cap;
    const UnitKeep *keep;
    const unsigned long long *group;
    const SliceAcc *acc;
    const uint32_t *slots;
    uint32_t slot_bytes;
    const UnitSet *sets;
    int32_t n_sets;
    const uint32_t *words;
    svt_roads roads;
    const uint8_t *accept;
    svt_fitrec rec;
    int32_t shift;
    int64_t *kept;      // nullable: the count alone
    int64_t kept_cap;
    int64_t *d_n_kept;
    uint64_t *err;
    int32_t parts;      // workgroups that share a group
};

__device__ __forceinline__ void keep_record(const KArgs &a, const UnitSet &c, int64_t pos,
                                            int32_t x01, int32_t x23, int32_t x4) {
    const uint32_t qlmask = (1u << a.shift) - 1u;
    int32_t v[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const uint4 w = c.row[j];
        int32_t acc = dot2(static_cast<int32_t>(w.x), x01, static_cast<int32_t>(w.w & qlmask));
        acc = dot2(static_cast<int32_t>(w.y), x23, acc);
        acc = dot2(static_cast<int32_t>(w.z), x4, acc);
        v[j] = (acc >> a.shift) + (static_cast<int32_t>(w.w) >> a.shift);
    }
    a.rec.p0[pos] = v[0];
    a.rec.p1[pos] = v[1];
    a.rec.p2[pos] = v[2];
    a.rec.chi2[pos] = static_cast<int64_t>(v[3]) * v[3] + static_cast<int64_t>(v[4]) * v[4] +
                      static_cast<int64_t>(v[5]) * v[5];
    if (a.rec.c0) a.rec.c0[pos] = v[3];
    if (a.rec.c1) a.rec.c1[pos] = v[4];
    if (a.rec.c2) a.rec.c2[pos] = v[5];
}

template <bool ONLY>
__global__ __launch_bounds__(kKeepGroup) void k_unit_keep(KArgs a) {
    __shared__ uint32_t s_pre[kKeepGroup];    // accepted before the unit, in the group
    __shared__ uint32_t s_quick[kKeepGroup];  // those of them that wait in slots
    __shared__ uint64_t s_first[kKeepGroup];  // the unit's first combination
    __shared__ int32_t s_cb[kKeepGroup];      // a searched unit's roads: first combination
    __shared__ uint16_t s_part[kKeepGroup];   // parts to be searched before the unit's
    __shared__ int32_t s_item[kKeepGroup];    // accepted combinations of one, in order
    __shared__ uint64_t s_tmp[kKeepGroup / kWaveSize + 1];
    __shared__ ulonglong2 s_sum[kKeepGroup / kWaveSize];
    __shared__ UnitSet s_bank[ONLY ? 256 : 1];
    const int tid = threadIdx.x;
    if (a.d_nw[1] < 0) {
        if (blockIdx.x == 0 && tid == 0) *a.d_n_kept = -1;
        return;
    }
    const int64_t nw = *a.d_nw;
    const int64_t n = nw < 0 ? 0 : nw > a.word_cap ? a.word_cap : nw;
    const int64_t nu = (n + kUnitWords - 1) / kUnitWords;
    const int64_t groups = (nu + kKeepGroup - 1) / kKeepGroup;
    const int64_t g = blockIdx.x / a.parts;
    const int part = static_cast<int>(blockIdx.x) % a.parts;
    // accepted in the groups before this one, and in all of them: one barrier for both, four counts
    // read at once
    const bool some = g < groups && a.kept && a.group[g * kKeepStride] != 0;
    if (blockIdx.x != 0 && !some) return;
    uint64_t before = 0, sum = 0;
    for (int64_t i0 = tid; i0 < groups; i0 += 4 * kKeepGroup) {
        uint64_t c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t i = i0 + e * kKeepGroup;
            c[e] = i < groups ? a.group[i * kKeepStride] : 0;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sum += c[e];
            before += i0 + e * kKeepGroup < g ? c[e] : 0;
        }
    }
    before = scan64(before);
    sum = scan64(sum);
    if (lane_id() == kWaveSize - 1) s_sum[tid / kWaveSize] = make_ulonglong2(before, sum);
    __syncthreads();
    before = sum = 0;
    for (int w = 0; w < kKeepGroup / kWaveSize; ++w) {
        before += s_sum[w].x;
        sum += s_sum[w].y;
    }
    const int64_t base = static_cast<int64_t>(before);
    const bool over = a.kept && static_cast<int64_t>(sum) > a.kept_cap;
    if (blockIdx.x == 0 && tid == 0) {
        *a.d_n_kept = static_cast<int64_t>(sum);
        if (over) report(a.err, SVT_ERRCLASS_CAPACITY, 2);
    }
    if (!some || (ONLY && over)) return;
    const int64_t u0 = g * kKeepGroup;
    UnitKeep mine{};
    if (u0 + tid < nu) mine = a.keep[u0 + tid];
    const uint32_t cnt = mine.count & ~kKeepSearch;
    const uint32_t quick = (mine.count & kKeepSearch) || (mine.size & kKeepCut) ? 0 : cnt;
    uint64_t tot;
    // (26 bits of accepted combinations, 17 of those in slots and 14 of parts are what 256 units can hold)
    const int slice_bits = static_cast<int>(a.d_nw[1]);
    const int part_bits = slice_bits > kKeepPartBits ? slice_bits : kKeepPartBits;
    auto parts_in = [&](uint32_t size) {
        return size & kKeepCut
                   ? static_cast<int>((((size & ~kKeepCut) >> kKeepRoadBits) - 1) >> part_bits) + 1
                   : 1;
    };
    const uint32_t parts_of = cnt > quick ? parts_in(mine.size) : 0;
    const uint64_t ex = block_excl_scan<uint64_t, kKeepGroup>(
        cnt | (static_cast<uint64_t>(quick) << 28) | (static_cast<uint64_t>(parts_of) << 48), s_tmp,
        tot);
    s_pre[tid] = static_cast<uint32_t>(ex & 0xFFFFFFFu);
    s_quick[tid] = static_cast<uint32_t>(ex >> 28) & 0xFFFFFu;
    s_first[tid] = mine.combo;
    s_part[tid] = static_cast<uint16_t>(ex >> 48);
    __syncthreads();
    const uint32_t n_quick = static_cast<uint32_t>(tot >> 28) & 0xFFFFFu;
    const int n_search = static_cast<int>(tot >> 48);
    // Every thread reads all six rows of a set, another one than its neighbours': from LDS where the
    // workgroup has enough to fit for the copy to pay (3.1e6 kept of 4e8 combinations: 101 us with
    // the rows from memory, 92 from LDS; at 84 thousand kept, three to a thread, 7.0 and 7.6).
    const uint32_t stride = a.parts * kKeepGroup;
    const bool staged = ONLY && n_quick > 4 * stride;
    if (staged) {
        const uint4 *src = reinterpret_cast<const uint4 *>(a.sets);
        uint4 *dst = reinterpret_cast<uint4 *>(s_bank);
        const int n16 = a.n_sets * static_cast<int>(sizeof(UnitSet) / 16);
        for (int i = tid; i < n16; i += kKeepGroup) dst[i] = src[i];
        __syncthreads();
    }
    auto find = [&](uint32_t i, int &unit) {  // where accepted combination i of the group waits
        int lo = 0, hi = kKeepGroup - 1;      // last unit that starts at or before it
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_quick[mid] <= i) lo = mid; else hi = mid - 1;
        }
        unit = lo;
        return a.slots + (u0 + lo) * (a.slot_bytes / 4) + (ONLY ? 4 : 1) * (i - s_quick[lo]);
    };
    auto read = [&](const uint32_t *slot) {
        return ONLY ? *reinterpret_cast<const uint4 *>(slot) : make_uint4(*slot, 0, 0, 0);
    };
    // Four at a time: a slot that is read behind stores waits until they are done, 5 us under load.
    constexpr int kAtOnce = 4;
    for (uint32_t i0 = part * kKeepGroup + tid; i0 < n_quick; i0 += kAtOnce * stride) {
        int unit[kAtOnce];
        uint4 v[kAtOnce];
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e) {
            const uint32_t i = i0 + e * stride;
            if (i < n_quick) v[e] = read(find(i, unit[e]));
        }
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e) {
            const uint32_t i = i0 + e * stride;
            if (i >= n_quick) break;
            const int64_t pos = base + s_pre[unit[e]] + (i - s_quick[unit[e]]);
            if (pos >= a.kept_cap) break;
            constexpr int bits = kGroupBits<ONLY ? kRecNone : kRecFit>;
            const int64_t GB = static_cast<int64_t>(s_first[unit[e]] & ~((uint64_t{1} << bits) - 1));
            if (ONLY) {
                a.kept[pos] = GB + (v[e].x & 0xFFFFFFu);
                const int32_t x01 = static_cast<int32_t>(v[e].y), x23 = static_cast<int32_t>(v[e].z),
                              x4 = static_cast<int32_t>(v[e].w);
                if (staged)
                    keep_record(a, s_bank[v[e].x >> 24], pos, x01, x23, x4);
                else
                    keep_record(a, a.sets[v[e].x >> 24], pos, x01, x23, x4);
            } else {
                a.kept[pos] = GB + v[e].x;
            }
        }
    }
    constexpr int kWalk = 8;  // words read at once: one by one, a road's take 20 us
    // ---- units whose accepted combinations are found again: their accept flags in order, each
    // one's road by its first combination and its hits by walking the road's words
    for (int sq = part; sq < n_search; sq += a.parts) {
        int q = 0;  // last unit whose parts start at or before this one: it has parts
        for (int hi = kKeepGroup - 1; q < hi;) {
            const int mid = (q + hi + 1) >> 1;
            if (s_part[mid] <= sq) q = mid; else hi = mid - 1;
        }
        const UnitKeep k = a.keep[u0 + q];
        const int nr = static_cast<int>(k.size & ((1u << kKeepRoadBits) - 1)),
                  len = static_cast<int>((k.size & ~kKeepCut) >> kKeepRoadBits);
        const int64_t CB0 = static_cast<int64_t>(k.combo), R0 = static_cast<int64_t>(k.road);
        // the part, and the accepted combinations in it and before it
        const int at_part = sq - s_part[q], parts = parts_in(k.size);
        const int to = part_bits - slice_bits, s0 = at_part << to, s1 = s0 + (1 << to);
        uint32_t skip = 0, here = 0;
        if (parts > 1) {
            for (int i = tid; i < s1; i += kKeepGroup) {  // (counts of the last slice are not kept)
                const uint32_t c = i < s0 || at_part + 1 < parts ? a.acc[k.acc + i].arrived >> 8 : 0;
                skip += i < s0 ? c : 0;
                here += i < s0 ? 0 : c;
            }
            const uint64_t sums = block_sum<uint64_t, kKeepGroup>(
                skip | (static_cast<uint64_t>(here) << 32), s_tmp);
            skip = static_cast<uint32_t>(sums);
            here = static_cast<uint32_t>(sums >> 32);
        }
        if (at_part + 1 == parts) here = (k.count & ~kKeepSearch) - skip;
        if (here == 0) continue;
        __syncthreads();
        if (tid < nr) s_cb[tid] = static_cast<int32_t>(a.roads.combo_begin[R0 + tid] - CB0);
        // its combinations, from the unit's first: i0 .. end - 1, in whole 4-byte words of flags where
        // those lie inside (parts are cut at whole groups, multiples of 4)
        constexpr int kGroup = 1 << kGroupBits<ONLY ? kRecNone : kRecFit>;
        const int in_group = static_cast<int>(CB0 & (kGroup - 1));
        const int i0 = at_part > 0 ? (at_part << part_bits) - in_group : -static_cast<int>(CB0 & 3);
        const int end = at_part + 1 < parts ? ((at_part + 1) << part_bits) - in_group : len;
        auto flags = [&](int i) {
            uint32_t w = 0;
            if (i >= 0 && i + 4 <= end) {
                w = *reinterpret_cast<const uint32_t *>(a.accept + CB0 + i);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e >= 0 && i + e < end)
                        w |= static_cast<uint32_t>(a.accept[CB0 + i + e]) << (8 * e);
            }
            return w;
        };
        const int64_t at = base + s_pre[q] + skip;
        const int per = ((end - i0 + kKeepGroup - 1) / kKeepGroup + 3) & ~3;  // at most 36
        const int mine0 = i0 + per * tid;
        uint64_t bits = 0;
        for (int v = 0; 4 * v < per; ++v)
            // flag bytes are 0 or 1: bits 0, 8, 16, 24 to 4 v .. 4 v + 3
            bits |= static_cast<uint64_t>(((flags(mine0 + 4 * v) * 0x10204080u) >> 28) & 0xFu)
                    << (4 * v);
        uint64_t all;
        const uint32_t rank = static_cast<uint32_t>(block_excl_scan<uint64_t, kKeepGroup>(
            static_cast<uint64_t>(__popcll(bits)), s_tmp, all));
        // dealt out again, one to a thread: accepted combinations come in runs (193 such units of
        // 2e5 cost 32 us as the last ones to finish, now 9)
        for (uint32_t first = 0; first < all; first += kKeepGroup) {
            uint32_t r2 = rank - first;
            for (uint64_t m = bits; m; m &= m - 1, ++r2)
                if (r2 < static_cast<uint32_t>(kKeepGroup)) s_item[r2] = mine0 + __builtin_ctzll(m);
            __syncthreads();
            const int i = s_item[tid];
            __syncthreads();
            const int64_t pos = at + first + tid;
            if (first + tid >= all || pos >= a.kept_cap) continue;
            a.kept[pos] = CB0 + i;
            if (!ONLY) continue;
            int lo = 0, hi = nr - 1;  // last road that starts at or before i
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_cb[mid] <= i) lo = mid; else hi = mid - 1;
            }
            const int64_t r = R0 + lo;
            const uint32_t nh = a.roads.nhits[r];
            uint32_t c = static_cast<uint32_t>(i - s_cb[lo]);
            uint32_t want = 0, words = 0;  // hit index per layer, 6 bits a layer
#pragma unroll
            for (int l = SVT_N_LAYERS - 1; l >= 0; --l) {  // layer 0 most significant
                const uint32_t nl = nh_of(nh, l);
                want |= (c % nl) << (6 * l);
                c /= nl;
                words += nl;
            }
            const uint32_t *w = a.words + a.roads.hit_begin[r];
            int32_t x[SVT_N_LAYERS] = {0, 0, 0, 0, 0};
            uint32_t seen = 0;
            for (uint32_t j0 = 0; j0 < words; j0 += kWalk) {
                uint32_t y[kWalk];
#pragma unroll
                for (int e = 0; e < kWalk; ++e) y[e] = w[j0 + e < words ? j0 + e : words - 1];
#pragma unroll
                for (int e = 0; e < kWalk; ++e) {
                    const uint32_t l = w_layer(y[e]);
                    const bool hit = j0 + e < words &&
                                     ((seen >> (6 * l)) & 63u) == ((want >> (6 * l)) & 63u);
                    seen += 1u << (6 * l);
#pragma unroll
                    for (int q2 = 0; q2 < SVT_N_LAYERS; ++q2)
                        if (hit && l == static_cast<uint32_t>(q2)) x[q2] = w_coord(y[e]);
                }
            }
            keep_record(a, a.sets[a.roads.set[r]], pos, pack16(x[0], x[1]), pack16(x[2], x[3]),
                        x[4]);
        }
    }
}

// ---- the unpack stage on its own ------------------------------------------------------------------
// The road table (event, set, hit_begin, nhits) and every word's coordinate at its place among its
// road's hits grouped by layer.  No bank and no tables: two workgroups of 16 waves fit a compute
// unit, and the waves take the units in turn.  With the counting kernel 24 us at 1.9e6 words, half of
// it the launches' own (33 before: flags, scan, lists and a kernel per road).
struct TArgs {
    const uint32_t *words;
    int64_t n;
    int32_t ranges;
    int32_t max_hits;
    const UnitRec *rec;
    const RangeTot *tot;
    svt_roads roads;
    int64_t road_cap;
    int16_t *hit_coord;
    int64_t *d_n_roads;
    uint64_t *err;
};
struct TWaveLds {
    uint2 ent[kEntries];
    uint32_t nh[kUnitWords];
    int16_t coord[kUnitSpan];
};

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_unit_table(TArgs a) {
    __shared__ RangeLds s_range;
    __shared__ TWaveLds s_wave[kUnitWaves];
    const int lane = lane_id(), wave = threadIdx.x / kWaveSize;
    TWaveLds &W = s_wave[wave];
    const int64_t nu = (a.n + kUnitWords - 1) / kUnitWords;
    const int64_t per = units_per_range(nu, a.ranges);
    RangeTot t{};
    if (static_cast<int>(threadIdx.x) < a.ranges) t = a.tot[threadIdx.x];
    const BatchTotals all =
        scan_ranges(t, a.ranges, nu, per, a.n, a.n, a.road_cap, INT64_MAX, 0, s_range);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *a.err = all.err;
        *a.d_n_roads = all.n_roads;
    }
    if (all.err != SVT_NO_ERROR) return;
    for (int64_t u = static_cast<int64_t>(blockIdx.x) * kUnitWaves + wave; u < nu;
         u += static_cast<int64_t>(gridDim.x) * kUnitWaves) {
        const int64_t base = u * kUnitWords;
        const int nloc = static_cast<int>(a.n - base < kUnitSpan ? a.n - base : kUnitSpan);
        const UnitWords uw = load_unit(a.words, base, nloc);
        const UnitRec rec = a.rec[u];
        const RangeBase rb = s_range.base[static_cast<uint32_t>(u) / static_cast<uint32_t>(per)];
        lds_order();
        UnitScan sc;
        if (nloc < kUnitSpan)
            sc = enter_unit<true>(W.ent, uw, nloc);
        else
            sc = enter_unit<false>(W.ent, uw, nloc);
        const uint32_t nr = sc.roads;
        if (nr == 0) continue;
        lds_order();
        uint32_t ev_run = rec.events + rb.events - 1, y0 = uw.before;
        for (uint32_t r0 = 0; r0 < nr; r0 += kWaveSize) {
            const uint32_t rl = r0 + lane;
            uint2 e0 = make_uint2(0, 0);
            if (rl < nr) e0 = W.ent[rl];
            const uint64_t em = ballot(starts_event(e0.y, y0)) &
                                lanes_below(nr - r0 < kWaveSize ? nr - r0 : kWaveSize);
            y0 = lane_value(e0.y, 63);
            const uint32_t evn = ev_run + bits_below(em) +
                                 (__builtin_amdgcn_inverse_ballot_w64(em) ? 1u : 0u);
            ev_run += __popcll(em);
            if (rl < nr) {
                bool over;
                const uint32_t nh = road_hits(e0, W.ent[rl + 1], a.max_hits, over);
                const int64_t r = static_cast<int64_t>(rec.roads + rb.roads) + rl;
                W.nh[rl] = nh;
                a.roads.event[r] = static_cast<int32_t>(evn);
                a.roads.set[r] = static_cast<int32_t>((e0.y >> 16) & 0xFFu);
                a.roads.hit_begin[r] = base + entry_pos(e0);
                a.roads.nhits[r] = nh;
            }
        }
        lds_order();
        uint32_t hits = sc.hits;
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) {
            const uint32_t rl = sc.road[e];
            if (rl < nr && kUnitLane * lane + e < nloc) {
                const uint2 ent = W.ent[rl];
                const uint32_t l = w_layer(uw.w[e]), nh = W.nh[rl];
                uint32_t p = entry_pos(ent) + (((hits - ent.x) >> (6 * l)) & 0x3Fu);
#pragma unroll
                for (int q = 0; q < SVT_N_LAYERS - 1; ++q)
                    p += static_cast<uint32_t>(q) < l ? nh_of(nh, q) : 0u;
                W.coord[p] = static_cast<int16_t>(w_coord(uw.w[e]));
            }
            hits += sc.hit[e];
        }
        lds_order();
        const int lo = static_cast<int>(entry_pos(W.ent[0])),
                  hi = static_cast<int>(entry_pos(W.ent[nr]));
        for (int j = lo + lane; j < hi; j += kWaveSize) a.hit_coord[base + j] = W.coord[j];
        lds_order();
    }
}

}  // namespace

int64_t unit_count(int64_t words) { return (words + kUnitWords - 1) / kUnitWords; }
int64_t unit_rec_bytes(int64_t words) {
    return static_cast<int64_t>(sizeof(UnitRec)) * unit_count(words);
}
// (and behind the ranges' totals the counts of fine slices per unit)
int64_t unit_range_bytes() {
    return static_cast<int64_t>(sizeof(RangeTot)) * kMaxRanges + 4ll * kPieces;
}
// Slices past their unit's first, and so accumulators: a batch's combinations over the largest slice, or
// where a smaller one is taken fewer than the pieces that it may leave (scan_ranges).
constexpr int64_t kUnitSlices = (7 * 32768) >> kSliceBits[0];  // of 7 roads of 8^5 in a unit
int64_t unit_slices(int64_t combos) {
    const int64_t small = combos >> kSliceBits[0];
    return (combos >> kSliceBits[2]) + (small < kPieces ? small : kPieces) + 1;
}
int64_t unit_acc_bytes(int64_t combos) {
    return static_cast<int64_t>(sizeof(SliceAcc)) * unit_slices(combos);
}
int64_t unit_keep_bytes(int64_t words) {
    return static_cast<int64_t>(sizeof(UnitKeep)) * unit_count(words);
}
int64_t unit_keep_group_bytes(int64_t words) {
    return 8 * kKeepStride * ((unit_count(words) + kKeepGroup - 1) / kKeepGroup);
}
int64_t unit_slot_bytes(int64_t words, bool less) {
    return (less ? kKeepSlotsLess : kKeepSlots) * unit_count(words);
}
int64_t unit_ticket_bytes() { return 4ll * kDealers * kDealerStride; }
int64_t unit_bank_bytes() { return static_cast<int64_t>(sizeof(UnitSet)) * 256; }

// Ranges the units of a capacity are counted in: one workgroup each.
static int unit_ranges(int64_t words) {
    const int64_t r = (unit_count(words > 0 ? words : 1) + kUnitWaves - 1) / kUnitWaves;
    return static_cast<int>(r < kMaxRanges ? r : kMaxRanges);
}

hipError_t launch_unpack(const uint32_t *words, int64_t n_words, const svt_config &cfg,
                         const svt_roads &roads, int64_t road_cap, int16_t *hit_coord,
                         int64_t *d_n_roads, uint64_t *err, void *rec, void *tot, int num_cus,
                         hipStream_t s) {
    const int ranges = unit_ranges(n_words);
    CArgs c{};
    c.words = words;
    c.nw = Sizes{n_words, nullptr, n_words};
    c.cfg = cfg;
    c.rec = static_cast<UnitRec *>(rec);
    c.tot = static_cast<RangeTot *>(tot);
    hipLaunchKernelGGL(k_unit_count, dim3(ranges), dim3(kThreads), 0, s, c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    TArgs t{words, n_words, ranges, cfg.max_hits, c.rec, c.tot, roads, road_cap, hit_coord,
            d_n_roads, err};
    const int64_t groups = (unit_count(n_words > 0 ? n_words : 1) + kUnitWaves - 1) / kUnitWaves;
    const int grid = static_cast<int>(groups < 2 * num_cus ? groups : 2 * num_cus);
    hipLaunchKernelGGL(k_unit_table, dim3(grid), dim3(kThreads), 0, s, t);
    return hipGetLastError();
}

// Workgroups of k_unit_keep that share a group of units, of n groups.
static int64_t keep_parts(int64_t n) {
    const int64_t most = 2048 / n, few = 1024 / n < 128 ? 1024 / n : 128;
    const int64_t parts = few > 32 ? few : 32;
    return most < 1 ? 1 : parts < most ? parts : most;
}

hipError_t launch_units(const UnitsLaunch &p, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    const int64_t units = unit_count(p.word_cap > 0 ? p.word_cap : 1);
    const int ranges = unit_ranges(p.word_cap);
    CArgs c{};
    c.words = p.words;
    c.nw = Sizes{0, p.d_n_words, p.word_cap};
    c.nw_copy = p.nw_copy;
    c.ticket = p.ticket;
    c.cfg = p.cfg;
    c.bank = p.bank;
    c.sets = static_cast<UnitSet *>(p.sets);
    c.rec = static_cast<UnitRec *>(p.rec);
    c.tot = static_cast<RangeTot *>(p.tot);
    c.fine = reinterpret_cast<uint32_t *>(c.tot + kMaxRanges);
    c.copy = p.copy;
    c.keep = p.d_n_kept ? static_cast<UnitKeep *>(p.keep) : nullptr;
    c.group = reinterpret_cast<unsigned long long *>(p.keep_groups);
    c.n_group = (units + kKeepGroup - 1) / kKeepGroup;
    c.acc = static_cast<SliceAcc *>(p.acc);
    // (cleared by as many workgroups as the words need: not for more slices than those can have, 448 a
    // unit of 7 roads of 8^5 combinations.  3000 words under a capacity of 8e8 combinations: 24.4 us a
    // pass with room for all of those cleared, 16.3 now)
    const int64_t slices = unit_slices(p.combo_cap), most = kUnitSlices * units;
    c.n_acc = slices < most ? slices : most;
    hipLaunchKernelGGL(k_unit_count, dim3(ranges + 1), dim3(kThreads), 0, s,
                       c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    UArgs a{};
    a.words = p.copy ? p.copy : p.words;
    a.d_nw = p.nw_copy;
    a.word_cap = p.word_cap;
    a.ticket = p.ticket;
    a.ranges = ranges;
    a.cfg = p.cfg;
    a.sets = c.sets;
    a.rec = c.rec;
    a.tot = c.tot;
    a.fine = c.fine;
    a.roads = p.roads;
    a.road_cap = p.road_cap;
    a.out = p.out;
    a.accept = p.accept;
    a.best = p.best;
    a.combo_cap = p.combo_cap;
    a.d_n_roads = p.d_n_roads;
    a.d_n_combos = p.d_n_combos;
    a.err = p.err;
    a.keep = c.keep;
    a.group = c.group;
    a.slots = static_cast<uint32_t *>(p.slots);
    a.slot_bytes = p.less_slots ? kKeepSlotsLess : kKeepSlots;
    a.acc = c.acc;
    const int grid = static_cast<int>(units < p.num_cus ? units : p.num_cus);
    if (start && (e = hipEventRecord(start, s)) != hipSuccess) return e;
    if (p.kept_only)
        hipLaunchKernelGGL((k_unit_fit<kRecNone>), dim3(grid), dim3(kThreads), 0, s, a);
    else if (p.out.c0 || p.out.c1 || p.out.c2)
        hipLaunchKernelGGL((k_unit_fit<kRecRows>), dim3(grid), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((k_unit_fit<kRecFit>), dim3(grid), dim3(kThreads), 0, s, a);
    e = hipGetLastError();
    if (e == hipSuccess && stop) e = hipEventRecord(stop, s);
    if (e != hipSuccess || !p.d_n_kept) return e;
    KArgs k{};
    k.d_nw = p.nw_copy;
    k.word_cap = p.word_cap;
    k.keep = c.keep;
    k.group = c.group;
    k.acc = c.acc;
    k.slots = a.slots;
    k.slot_bytes = a.slot_bytes;
    k.sets = c.sets;
    k.n_sets = p.cfg.n_sets;
    k.words = a.words;
    k.roads = p.roads;
    k.accept = p.accept;
    k.rec = p.out;
    k.shift = p.cfg.shift;
    k.kept = p.kept;
    k.kept_cap = p.kept_cap;
    k.d_n_kept = p.d_n_kept;
    k.err = p.err;
    // Few groups are shared by several workgroups each: by 32 where that fills the chip (30 groups of
    // units, 84 thousand kept: 6.8 us, with 68 9.5), by up to 128 where there are fewer still (a pass
    // over 1000 uneven events, 7 groups, every combination accepted, its flags searched in parts of 4096:
    // 270 us with 32, 167 with 128; the list of 37 such events at the usual cut 11.4 and 7.9).
    k.parts = static_cast<int32_t>(keep_parts(c.n_group));
    const int kgrid = p.kept ? static_cast<int>(c.n_group) * k.parts : 1;
    if (p.kept_only)
        hipLaunchKernelGGL(k_unit_keep<true>, dim3(kgrid), dim3(kKeepGroup), 0, s, k);
    else
        hipLaunchKernelGGL(k_unit_keep<false>, dim3(kgrid), dim3(kKeepGroup), 0, s, k);
    return hipGetLastError();
}

}  // namespace svt
