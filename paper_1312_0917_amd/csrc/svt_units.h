// Wave-sized units of the batched pass: what the counting kernel and the fitting kernel share.
//
// A unit is 256 consecutive hit words and belongs to one wave.  The wave stages 64 words more:
// a road that starts among the unit's words may run past them, and a road with combinations has
// at most 5 * 8 = 40 words.  A lane holds five consecutive words of the 320, so one wave-wide
// scan of packed counts gives every word its road, its event and its rank among its road's hits
// on its layer; nothing is walked word by word.
#pragma once

#include "svt_common.h"

namespace svt {

constexpr int kUnitWords = 256;                      // words a unit owns
constexpr int kUnitSpan = 320;                       // words staged
constexpr int kUnitLane = kUnitSpan / kWaveSize;     // 5 consecutive words per lane
constexpr int kUnitFitRoads = 64;  // roads with combinations that start in a unit: each has at
                                   // least 5 words, so at most (256 + 35) / 5 = 58
constexpr int kUnitWaves = 16;     // waves of a workgroup of either kernel
constexpr int kDealers = 32;       // counters that deal out the last units,
constexpr int kDealerStride = 32;  // a 128-byte line apart
constexpr int kMaxRanges = 512;    // contiguous ranges of units whose totals are scanned together

// A unit with many combinations is cut into slices, so that no wave works long after the others have
// finished (a unit of the largest roads holds 2e5 combinations, a usual one 800 to 3000).  The counting
// kernel counts the slices past each unit's first for three lengths, and the fitting kernel takes the
// smallest of 512, 2048 and 8192 combinations that leaves at most kPieces units and slices together, half
// of the chip's 4096 waves: a slice unpacks its unit again, so slices pay while waves would be idle.  Us
// a pass with records, 8192 for all / by this rule / with all 4096 waves: 65 units of uneven roads 51 / 23
// / 23, 512 of them 55 / 33 / 31, 1024 57 / 58 / 42, but 1024 units of 800 combinations 24 / 24 / 26.  (Going
// by the number of units alone, 94 units of roads of 8^5 were cut into 38 thousand slices: 375, now 150.)
// In kept-only mode a unit's fits take half the time, and what a cut unit accepted is found again from
// its flags, 6 us for the list kernel: with 256 and 512 pieces 128 units of 800 combinations take 24 and 29.
constexpr int kSliceBits[3] = {9, 11, 13};
constexpr int kPieces = 2048, kPiecesKeptOnly = 256;
static_assert(kPiecesKeptOnly <= kPieces, "the slices' accumulators are sized for kPieces (unit_slices)");
// Counts before a unit, from the start of its range.
struct alignas(16) UnitRec {
    uint32_t roads, events;
    uint64_t combos;     // 40 bits; above them the slices of 8192 past each unit's first
};
constexpr int kExtraShift = 40;
// The slices of 512 and 2048 beside them, where there are fewer units than pieces: a range then has 16
// units, with at most 104 roads of 40 words, so 13 bits of the one and 11 of the other.
constexpr int kFineBits = 13;
__host__ __device__ inline uint32_t fine_slices(uint32_t x, int step) {
    return step == 1 ? x >> kFineBits : x & ((1u << kFineBits) - 1);
}
// What the slices of a unit find out together about a road cut by a slice's end, at the first such
// end, and the slice that ends there about itself: zero to start with.
struct alignas(16) SliceAcc {
    unsigned long long key;  // complement of the smallest key
    uint32_t nacc;
    uint32_t arrived;        // slices that have added theirs | the slice's accepted combinations << 8
};
// What a unit's wave leaves for the kept list: the number of its accepted combinations, and where
// its roads and combinations are.  The accepted combinations themselves wait in the unit's slots,
// as indices (4 bytes) or with their coordinates (16).  A unit that accepts more than it has slots,
// or is cut into slices (kKeepCut), is searched: they are found again from the accept flags, in parts
// of a slice or 2^kKeepPartBits combinations, each by a workgroup that has the counts of the slices
// before it from their accumulators.
// (With one workgroup for a whole unit a pass over 1000 uneven events, every combination accepted,
// took 562 us, 1050 kept-only: 233 and 407 now; scan, compaction and refit of the flat list 406 and 570.)
// With 1024 bytes of slots that is one unit in 1000 of 2048-road events and one in 200 of the
// uneven ones (512 bytes, where the workspace has no more: 4 and 9 in 100).
struct UnitKeep {
    uint32_t count;   // | kKeepSearch
    uint32_t size;    // roads (at most 256) | combinations (at most 2.4e5) << kKeepRoadBits | kKeepCut
    uint64_t combo;   // the unit's first
    uint32_t road;    // the same of the roads
    uint32_t acc;     // accumulator of the end of the unit's first slice
};
constexpr uint32_t kKeepSearch = 1u << 31;
constexpr uint32_t kKeepCut = 1u << 31;
constexpr int kKeepRoadBits = 9;
constexpr int kKeepPartBits = 12;
constexpr int kKeepSlots = 1024, kKeepSlotsLess = 512;  // bytes per unit
constexpr int kKeepGroup = 256;   // units a workgroup of k_unit_keep takes, with a common count,
constexpr int kKeepStride = 16;   // a 128-byte line apart: every unit adds to one (side by side
                                  // they held up the fits of 7500 units for 26 us)
// Totals of a range of units, and the first errors in it (all ones: none).
struct alignas(16) RangeTot {
    uint32_t roads, events;
    uint64_t combos;     // as in UnitRec
    uint32_t bad_word;   // word with a layer field out of range (index in the range)
    uint32_t over_road;  // road with too many hits on a layer (index in the range)
    uint32_t set_road;   // road whose tag has no constant set (index in the range)
    uint32_t fine;       // slices of 512 and 2048 (fine_slices)
};

// A constant set as the fit reads it: row j is f0|f1, f2|f3, f4|0 (int16 pairs) and the offset.
// 112 bytes: with a stride of 28 dwords the 16-byte reads of the sets one wave works on start in
// different LDS banks.
struct alignas(16) UnitSet {
    uint4 row[6];
    uint32_t narrow;  // the set's bounds allow 32-bit sums (narrow_ok)
    uint32_t pad[3];
};
static_assert(sizeof(UnitSet) == 112, "LDS bank spread of the staged constant sets");

// ---- cross-lane helpers ------------------------------------------------------------------------
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t x, uint32_t old = 0) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        static_cast<int>(old), static_cast<int>(x), CTRL, ROWS, 0xF, false));
}
constexpr int kDppNext = 0x130;  // lane i reads lane i + 1 (lane 63: the given default)
constexpr int kDppPrev = 0x138;  // lane i reads lane i - 1 (lane 0: the given default)

// Inclusive scan over the wave's 64 lanes, all of them active.
__device__ __forceinline__ uint32_t scan64(uint32_t x) {
    x += dpp<0x111>(x);
    x += dpp<0x112>(x);
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    x += dpp<0x142, 0xA>(x);
    x += dpp<0x143, 0xC>(x);
    return x;
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
    return dpp<CTRL, ROWS>(static_cast<uint32_t>(x)) |
           (static_cast<uint64_t>(dpp<CTRL, ROWS>(static_cast<uint32_t>(x >> 32))) << 32);
}
__device__ __forceinline__ uint64_t scan64(uint64_t x) {
    x += dpp64<0x111>(x);
    x += dpp64<0x112>(x);
    x += dpp64<0x114>(x);
    x += dpp64<0x118>(x);
    x += dpp64<0x142, 0xA>(x);
    x += dpp64<0x143, 0xC>(x);
    return x;
}
// The same over the first 16 lanes (each row of 16 on its own).
__device__ __forceinline__ uint32_t scan16(uint32_t x) {
    x += dpp<0x111>(x);
    x += dpp<0x112>(x);
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    return x;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), lane));
}
__device__ __forceinline__ uint32_t uni(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
}
__device__ __forceinline__ uint64_t uni(uint64_t x) {
    return static_cast<uint64_t>(uni(static_cast<uint32_t>(x))) |
           (static_cast<uint64_t>(uni(static_cast<uint32_t>(x >> 32))) << 32);
}
// __ballot takes an int: its argument goes through a register and is compared once more
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// A 32-bit offset in bytes from a pointer that is the same in all lanes.  offset_of keeps the
// compiler from widening it where it is computed: widened next to the access, it needs no 64-bit
// address.
__device__ __forceinline__ uint32_t offset_of(uint32_t o) {
    asm("" : "+v"(o));
    return o;
}
template <typename T>
__device__ __forceinline__ T *at_byte(T *p, uint32_t o) {
    return reinterpret_cast<T *>(reinterpret_cast<char *>(p) + o);
}
__device__ __forceinline__ const int32_t *at_byte(const int32_t *p, uint32_t o) {
    return reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(p) + o);
}
// 8 bytes at an address that is a multiple of 4
typedef uint32_t U32Pair __attribute__((ext_vector_type(2), aligned(4)));
// A pointer that was itself read from LDS points to memory, which the compiler cannot know: it would
// use flat accesses, and a flat store holds up every later wait for LDS until memory has taken it.
template <typename T>
using InMemory = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ InMemory<T> *in_memory(T *p) {
    return (InMemory<T> *)p;
}
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
// LDS by 32-bit address
typedef __attribute__((address_space(3))) const int32_t LdsInt;
__device__ __forceinline__ uint32_t lds_address(const int32_t *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((LdsInt *)p));
}
__device__ __forceinline__ int32_t lds_read(uint32_t at) { return *(LdsInt *)static_cast<uintptr_t>(at); }
// bits off .. off + width - 1, both below 32
__device__ __forceinline__ uint32_t bit_field(int32_t width, int32_t off) {
    uint32_t r;
    asm("v_bfm_b32 %0, %1, %2" : "=v"(r) : "v"(width), "v"(off));
    return r;
}
// number of set bits of m below the calling lane
__device__ __forceinline__ int bits_below(uint64_t m) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(
        static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0)));
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int d = kWaveSize / 2; d > 0; d >>= 1) {
        const uint32_t o = __shfl_xor(v, d, kWaveSize);
        v = o < v ? o : v;
    }
    return v;
}
// One wave's LDS writes before its own later LDS reads (the hardware keeps a wave's LDS accesses in
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ UnitRec read_rec(const UnitRec *rec, int64_t u) {
    const U32x4 v = *(in_memory(reinterpret_cast<const U32x4 *>(rec)) + u);
    return UnitRec{v.x, v.y, v.z | (static_cast<uint64_t>(v.w) << 32)};
}

// ---- a unit's words ---------------------------------------------------------------------------
struct UnitWords {
    uint32_t w[kUnitLane];  // words 5 * lane + e of the span (0 past the input)
    uint32_t before;        // the word before the unit; for the first unit one that differs from
                            // its first word in both tags
};

// nloc: words of the batch from the unit's first on, at most kUnitSpan
__device__ __forceinline__ UnitWords load_unit(const uint32_t *__restrict__ words, int64_t base,
                                               int nloc) {
    UnitWords u;
    const uint32_t *p = words + base;
    const int j0 = kUnitLane * lane_id();
    if (nloc == kUnitSpan) {
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) u.w[e] = p[j0 + e];
    } else {
#pragma unroll
        for (int e = 0; e < kUnitLane; ++e) u.w[e] = j0 + e < nloc ? p[j0 + e] : 0u;
    }
    u.before = base > 0 ? p[-1] : ~p[0];
    return u;
}

// Hits are counted per layer in one 32-bit word, 6 bits a layer.  Running counts over a unit
// overflow their fields, but the difference of two of them is the sum of 2^(6 l) over the hits in
// between all the same, and its fields are the hits per layer wherever none reaches 64 (a road
// longer than 5 * 8 words is illegal whatever they hold).
__device__ __forceinline__ uint32_t layer_unit(uint32_t w) { return 1u << (6 * w_layer(w)); }

// What a lane knows of its words.
struct UnitScan {
    uint32_t hit[kUnitLane];   // what word e adds to the hit counts
    uint32_t hits;             // hit counts before the lane's first word
    uint32_t road[kUnitLane];  // word e's road, among those that start in the span (all ones: one that
                               // starts before it)
    uint32_t roads;            // roads that start among the unit's own words (uniform)
};

// A road's entry: x = hit counts before its first word; y = that word's index in the unit (9
// bits), bits 16..31: its tags.  The road ends where the next entry starts; entry [roads owned] is
// the end of the last one: the first road start past the unit, or the end of the staged words.
__device__ __forceinline__ uint32_t entry_pos(uint2 e) { return e.y & 0x1FFu; }

__device__ __forceinline__ uint64_t lanes_below(int k) { return k > 0 ? ~0ull >> (kWaveSize - k) : 0; }

// Scan the words and write an entry for every road that starts in the span.  Road starts are kept as
// one mask of lanes per word, in scalar registers: counting them there and with mbcnt took 35 fewer
// vector instructions, of 250 in the counting kernel, than flags in a register and a scan.
// CHECK: the span may hold words past the input or layer fields out of range, which count nothing.
template <bool CHECK>
__device__ __forceinline__ UnitScan enter_unit(uint2 *S, const UnitWords &u, int nloc) {
    UnitScan s;
    const uint32_t j0 = kUnitLane * lane_id();
    uint64_t starts[kUnitLane];
    uint32_t prev = dpp<kDppPrev>(u.w[kUnitLane - 1], u.before), hits = 0, before = 0;
    uint32_t all = 0;
    s.roads = 0;
#pragma unroll
    for (int e = 0; e < kUnitLane; ++e) {
        const uint32_t x = u.w[e];
        starts[e] = ballot((x ^ prev) > 0xFFFFu);
        if (CHECK) starts[e] &= lanes_below((nloc - e + kUnitLane - 1) / kUnitLane);
        const uint64_t own = starts[e] & lanes_below((kUnitWords - e + kUnitLane - 1) / kUnitLane);
        all += __popcll(starts[e]);
        s.roads += __popcll(own);
        before = __builtin_amdgcn_mbcnt_hi(
            static_cast<uint32_t>(starts[e] >> 32),
            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(starts[e]), before));
        s.hit[e] = layer_unit(x);
        if (CHECK && (static_cast<int>(j0) + e >= nloc || w_layer(x) >= SVT_N_LAYERS)) s.hit[e] = 0;
        hits += s.hit[e];
        prev = x;
    }
    const uint32_t ih = scan64(hits);
    s.hits = ih - hits;
    uint32_t h = s.hits, rd = before - 1u;
#pragma unroll
    for (int e = 0; e < kUnitLane; ++e) {
        const bool start = __builtin_amdgcn_inverse_ballot_w64(starts[e]);
        rd += start ? 1u : 0u;
        s.road[e] = rd;
        if (start) S[rd] = make_uint2(h, (u.w[e] & 0xFFFF0000u) | (j0 + e));
        h += s.hit[e];
    }
    if (all == s.roads && lane_id() == 0)
        S[all] = make_uint2(lane_value(ih, 63), static_cast<uint32_t>(nloc));
    return s;
}

// Whether a road starts an event: its own entry against the road's before it, in the lane below (y0:
// what lane 0 compares with, the word before the unit or the last entry of the 64 before).
__device__ __forceinline__ bool starts_event(uint32_t y, uint32_t y0) {
    return (y ^ dpp<kDppPrev>(y, y0)) > 0xFFFFFFu;
}

// Hits of the road between two entries: 4 bits per layer, and whether it is illegal (too many
// words, or hits on a layer; such a road has no combinations).
__device__ __forceinline__ uint32_t road_hits(uint2 e0, uint2 e1, int max_hits, bool &over) {
    const uint32_t d = e1.x - e0.x;
    const uint32_t c0 = d & 63u, c1 = (d >> 6) & 63u, c2 = (d >> 12) & 63u, c3 = (d >> 18) & 63u,
                   c4 = (d >> 24) & 63u;
    // A count above max_hits shows in bit 5 of its field, as it is (32..40, in a road of at most 40
    // words) or with 31 - max_hits added; up to the lowest such field no addition carries.
    constexpr uint32_t ones = 0x01041041u;
    const uint32_t k = static_cast<uint32_t>(31 - max_hits) * ones;
    over = static_cast<int>(entry_pos(e1) - entry_pos(e0)) > SVT_N_LAYERS * max_hits ||
           ((d | (d + k)) & (ones << 5)) != 0;
    return (c0 & 0xFu) | ((c1 & 0xFu) << 4) | ((c2 & 0xFu) << 8) | ((c3 & 0xFu) << 12) |
           ((c4 & 0xFu) << 16);
}
__device__ __forceinline__ uint32_t road_combos(uint32_t nh) {
    return nh_of(nh, 0) * nh_of(nh, 1) * nh_of(nh, 2) * nh_of(nh, 3) * nh_of(nh, 4);
}

// Who fits which of nu units: workgroup `block` of `grid` takes units lo .. hi - 1 first; then, with the
// workgroups of the same dealer, what is left of p_lo .. p_hi - 1, `batch` units at a time.  Seven
// eighths of the units are dealt out beforehand, in contiguous ranges, so that the record lines two
// neighbouring units share are written from one compute unit; all of them where a wave has no second
// one to take, or where the workgroups are too few to serve every dealer.
struct UnitShare {
    int64_t lo, hi, p_lo, p_hi, batch;
    int dealer;
};
__host__ __device__ inline UnitShare unit_share(int64_t nu, int block, int grid) {
    const int64_t fixed =
        nu <= static_cast<int64_t>(grid) * kUnitWaves || grid < kDealers ? nu : nu - nu / 8;
    const int64_t pool = nu - fixed;
    UnitShare s;
    s.lo = fixed * block / grid;
    s.hi = fixed * (block + 1) / grid;
    s.dealer = block % kDealers;
    s.p_lo = fixed + pool * s.dealer / kDealers;
    s.p_hi = fixed + pool * (s.dealer + 1) / kDealers;
    s.batch = 1 + pool / (kDealers * 512);
    return s;
}

// Units of a range when nu units are dealt to at most `ranges` of them: a multiple of the waves
// of a workgroup.
__host__ __device__ inline int64_t units_per_range(int64_t nu, int64_t ranges) {
    const int64_t per = (nu + ranges - 1) / ranges;
    return (per + kUnitWaves - 1) / kUnitWaves * kUnitWaves;
}

}  // namespace svt
