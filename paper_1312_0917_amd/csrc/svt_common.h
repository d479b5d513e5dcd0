// Internal helpers shared by the HIP kernels of libsvt (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "svt.h"

namespace svt {

constexpr int kWaveSize = 64;
constexpr int kSegThreads = 256;          // threads of the selection kernels
constexpr int kPrepassBlockWords = 2048;  // words per block of the batched single-pass pre-pass
constexpr int kLookGroup = 64;            // pre-pass blocks per group of its two-level look-back
// look-back status words of the pre-pass: two per block, then two per group of kLookGroup blocks
inline int64_t prepass_status_words(int64_t nb_cap) {
    return 2 * nb_cap + 2 * ((nb_cap + kLookGroup - 1) / kLookGroup);
}
constexpr int kRoadBlock = 256;           // roads per block in road-table kernels
constexpr int kKeptBlock = 4096;          // combinations per block of the kept-list compaction
constexpr int kScanThreads = 1024;        // single-workgroup scan
constexpr int kKeyKBits = 15;             // best-track key: chi2 << 15 | k  (k < 8^5 = 2^15)
constexpr uint64_t kKeyChiMax = (1ull << 49) - 1;  // chi2 part of a key saturates here

// Order-preserving key of an accepted combination for one 64-bit atomicMin: exact whenever
// the smallest chi2 of the road is below kKeyChiMax; a saturated minimum means "rescan".
__device__ inline uint64_t best_key(int64_t chi2, uint32_t k) {
    uint64_t c = static_cast<uint64_t>(chi2);
    if (c > kKeyChiMax) c = kKeyChiMax;
    return (c << kKeyKBits) | k;
}
constexpr int kMaxTile = 8192;  // largest svt_tune.tile_combos
constexpr int64_t kMaxBatchWords = (1ll << 31) - 1;  // batched path: road and event counts fit 31 bits

// ---- error word: (class << 56) | index, smallest wins, all ones = none ------------------
__device__ inline void report(uint64_t *err, uint32_t cls, uint64_t index) {
    uint64_t v = (static_cast<uint64_t>(cls) << 56) | (index & ((1ull << 56) - 1));
    atomicMin(reinterpret_cast<unsigned long long *>(err), static_cast<unsigned long long>(v));
}

__device__ inline bool has_error(const uint64_t *err) {
    return *reinterpret_cast<const volatile uint64_t *>(err) != SVT_NO_ERROR;
}

// The same for a whole workgroup, read once: a kernel that reports errors itself changes the word
// while its workgroups start, and of one workgroup's waves some could leave and the others go on
// without them.  Contains a barrier.
__device__ inline bool block_has_error(const uint64_t *err) {
    __shared__ bool found;
    if (threadIdx.x == 0) found = has_error(err);
    __syncthreads();
    return found;
}

// ---- hit word fields (coord int13 | layer 3 | road tag 8 | event tag 8) -------------------
__device__ inline int32_t w_coord(uint32_t w) {
    return static_cast<int32_t>(w << 19) >> 19;  // sign-extend the low 13 bits
}
__device__ inline uint32_t w_layer(uint32_t w) { return (w >> 13) & 7u; }
__device__ inline uint32_t w_rtag(uint32_t w) { return (w >> 16) & 0xFFu; }
__device__ inline uint32_t w_etag(uint32_t w) { return w >> 24; }
__device__ inline uint32_t w_tags(uint32_t w) { return w >> 16; }  // road and event tag together

__device__ inline uint32_t nh_of(uint32_t packed, int l) { return (packed >> (4 * l)) & 0xFu; }

// ---- wave64 / block scans -----------------------------------------------------------------
__device__ inline int lane_id() { return __lane_id(); }

template <typename T>
__device__ inline T wave_incl_scan(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) {
        T t = __shfl_up(v, d, kWaveSize);
        if (lane >= d) v += t;
    }
    return v;
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
    for (int d = kWaveSize / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWaveSize);
    return v;
}

// Exclusive block scan for blockDim.x = NT threads; returns the exclusive prefix and the
// block total.  `tmp` must hold NT/64 + 1 elements of T in LDS.  Contains barriers.
template <typename T, int NT>
__device__ inline T block_excl_scan(T v, T *tmp, T &total) {
    constexpr int NW = NT / kWaveSize;
    const int lane = lane_id();
    const int wave = threadIdx.x / kWaveSize;
    T incl = wave_incl_scan(v);
    if (lane == kWaveSize - 1) tmp[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int w = 0; w < NW; ++w) {
            T t = tmp[w];
            tmp[w] = run;
            run += t;
        }
        tmp[NW] = run;
    }
    __syncthreads();
    T res = incl - v + tmp[wave];
    total = tmp[NW];
    __syncthreads();
    return res;
}

template <typename T, int NT>
__device__ inline T block_sum(T v, T *tmp) {
    constexpr int NW = NT / kWaveSize;
    T s = wave_sum(v);
    const int wave = threadIdx.x / kWaveSize;
    if (lane_id() == 0) tmp[wave] = s;
    __syncthreads();
    T tot = 0;
    for (int w = 0; w < NW; ++w) tot += tmp[w];
    __syncthreads();
    return tot;
}

// Grid-stride helpers
__device__ inline int64_t gtid() {
    return static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
}
__device__ inline int64_t gstride() { return static_cast<int64_t>(gridDim.x) * blockDim.x; }

}  // namespace svt

// ---- host-side launchers (defined in the .hip files) --------------------------------------
namespace svt {

struct Sizes {  // counts that can live on the host (plain path) or on the device (batch path)
    int64_t host;            // used when dev == nullptr
    const int64_t *dev;      // device scalar
    int64_t cap;             // kernels never use more than this many items
};

__device__ inline int64_t load_size(const Sizes &s) {
    int64_t v = s.dev ? *s.dev : s.host;
    if (v > s.cap) v = s.cap;
    return v < 0 ? 0 : v;
}

// In-place exclusive scan of ceil(n / div) int64 entries by one workgroup; the total goes to *tot (may
// be null).  When it exceeds cap (>= 0), a capacity error with index cap_index is reported.  With
// skip_if_error, an error already in *err makes it write a total of -1 and do nothing else.
hipError_t launch_scan(int64_t *data, Sizes n, int64_t div, int64_t *tot, int64_t cap,
                       uint32_t cap_index, uint64_t *err, bool skip_if_error, hipStream_t s);
hipError_t launch_combo_count(const svt_roads &roads, Sizes n_roads, int64_t grid_blocks,
                              int64_t *rb_sums, uint64_t *err, hipStream_t s);
// combo_road (nullable): receives the road of every listing tile's first combination, which
// launch_materialize starts from
hipError_t launch_combo_begin(const svt_roads &roads, Sizes n_roads, int64_t grid_blocks,
                              const int64_t *rb_prefix, int32_t *combo_road, int64_t combo_cap,
                              uint64_t *err, hipStream_t s);
hipError_t launch_materialize(const svt_roads &roads, int64_t n_roads, const int64_t *d_n_combos,
                              int64_t combo_cap, int32_t *combo_road, uint32_t *combo_hits,
                              uint64_t *err, hipStream_t s);
hipError_t launch_fit_plain(const svt_fconst *bank, const svt_config &cfg,
                            const svt_roads &roads, int64_t n_roads, const int16_t *hit_coord,
                            int64_t n_hits, const int32_t *combo_road,
                            const uint32_t *combo_hits, int64_t n_combos, const svt_fitrec &out,
                            uint64_t *err, int num_cus, hipStream_t s);
hipError_t launch_select(const svt_config &cfg, const svt_roads &roads, int64_t n_roads,
                         const int32_t *combo_road, const svt_fitrec &rec, int64_t n_combos,
                         uint8_t *accept, const svt_best &best, int64_t *kb_counts,
                         uint64_t *err, hipStream_t s);
hipError_t launch_kept_write(const uint8_t *accept, Sizes n_combos, int64_t grid_blocks,
                             const int64_t *kb_prefix, int64_t *kept, int64_t kept_cap,
                             uint64_t *err, hipStream_t s);
// Kept-only mode: the ascending indices of accepted combinations into kept[] and their fit
// values, compacted, into rec (entry i for combination kept[i]), fitted again from the grouped
// coordinates and the constant bank.  tile_first_road / tile_combos locate each block's roads.
// Does nothing when *err already holds an error (the inputs it reads are then incomplete).
hipError_t launch_kept_refit(const uint8_t *accept, Sizes n_combos, Sizes n_roads,
                             int64_t grid_blocks, const int64_t *kb_prefix, const svt_roads &roads,
                             const int32_t *tile_first_road, int64_t tile_combos,
                             const svt_fconst *bank, int32_t n_sets, const int16_t *coords,
                             int32_t shift, int64_t *kept, const svt_fitrec &rec,
                             int64_t kept_cap, uint64_t *err, hipStream_t s);

// One event per workgroup at a time (schedule 1 of svt_tune), after the pre-pass: the ablation of
// how the work is split.
struct EventsLaunch {
    const svt_fconst *bank;
    svt_config cfg;
    int wgs_per_cu;
    const int16_t *coords;     // workspace: coordinates grouped by layer inside each road
    svt_roads roads;
    const int64_t *d_n_roads;
    const int64_t *d_n_combos;
    const int64_t *d_n_events;
    const int32_t *event_first_road;
    svt_fitrec rec;
    uint8_t *accept;
    svt_best best;
    int64_t *kb_counts;        // per kKeptBlock combinations (null: kept list not wanted)
    uint32_t *ticket;
    uint64_t *err;
    int64_t road_cap;
    int64_t combo_cap;
    int64_t event_cap;
    int num_cus;
    bool kept_only;            // no per-combination records (accept flags still written)
};
hipError_t launch_fit_events(const EventsLaunch &f, hipStream_t s);
// Per road: turn the best-track key left in best.chi2 into (k, chi2, p0..p2), reading the
// parameters from the records, or fitting them again from the grouped coordinates when bank
// and coords are given (exact rescan of the records for a road whose key saturated).
// An in-place exclusive scan of ceil(n / div) counts with its total written to *tot and checked
// against cap (class CAPACITY, index cap_index) when cap >= 0; data == nullptr: no job.
struct ScanJob {
    int64_t *data = nullptr;
    Sizes n{};
    int64_t div = 1;
    int64_t *tot = nullptr;
    int64_t cap = -1;
    uint32_t cap_index = 0;
};
// Best track per road from the keys; with a scan job, one extra workgroup does that scan.
hipError_t launch_best_finalize(const svt_roads &roads, Sizes n_roads, const svt_fitrec &rec,
                                Sizes n_combos, const svt_best &best, int64_t cut,
                                uint64_t *err, bool skip_if_error, const svt_fconst *bank,
                                const int16_t *coords, int32_t shift, const ScanJob &job,
                                hipStream_t s);

// Single-pass unpack + combine of the batched path (decoupled look-back over word blocks).
struct PrepassLaunch {
    const uint32_t *words;
    Sizes nw;                  // device word count, capacity word_cap
    svt_config cfg;
    svt_roads roads;
    int64_t road_cap;
    int16_t *coords;           // grouped coordinates, word_cap entries
    svt_best best;             // best keys and n_accept are initialised here
    int64_t tile_combos;
    int32_t *tile_first_road;
    int64_t tiles_cap;
    int64_t combo_cap;
    int64_t *d_n_roads;
    int64_t *d_n_combos;
    int64_t *status;           // look-back status words (prepass_status_words(nb_cap))
    int64_t nb_cap;            // ceil(word_cap / kPrepassBlockWords)
    int64_t status_words;      // status words the reset clears
    uint32_t *ticket;          // of the event kernel, cleared by the reset
    uint64_t *err;
    int32_t *event_first_road; // first road of every event (event_cap entries)
    int64_t event_cap;
    int64_t *d_n_events;
};
// Clears the error word, the ticket, *d_n_kept (nullable), status[0 .. status_words) and
// zero[0 .. n_zero) (the kept-list block counts; nullable).
hipError_t launch_batch_reset(const PrepassLaunch &p, int64_t *nw_copy, int64_t *d_n_kept,
                              int64_t *zero, int64_t n_zero, hipStream_t s);
hipError_t launch_prepass(const PrepassLaunch &p, hipStream_t s);

// The batched pass over wave-sized units of words: a counting kernel and a fitting kernel
// (svt_units.hip), with `start` / `stop` (nullable) recorded around the second.
struct UnitsLaunch {
    const svt_fconst *bank;
    svt_config cfg;
    const uint32_t *words;
    const int64_t *d_n_words;
    int64_t word_cap;
    svt_roads roads;
    int64_t road_cap;
    svt_fitrec out;
    uint8_t *accept;
    svt_best best;
    int64_t combo_cap;
    int64_t *d_n_roads;
    int64_t *d_n_combos;
    uint64_t *err;
    int64_t *d_n_kept;         // null: no count and no kept list
    int64_t *kept;             // null: the count alone
    int64_t kept_cap;
    bool kept_only;            // no records but those of the kept list
    int64_t *nw_copy;          // workspace: the word count in device memory, and a word beside it,
    uint32_t *ticket;          // counters (unit_ticket_bytes),
    void *sets;                // the packed bank (unit_bank_bytes),
    void *rec;                 // running counts per unit (unit_rec_bytes),
    void *tot;                 // totals per range of units (unit_range_bytes),
    void *acc;                 // what slices of units share (unit_acc_bytes),
    void *keep;                // accepted combinations per unit (unit_keep_bytes),
    int64_t *keep_groups;      // and per group of units (unit_keep_group_bytes),
    void *slots;               // accepted combinations (unit_slot_bytes, 16-byte aligned;
    bool less_slots;           // the smaller number of them),
    uint32_t *copy;            // and the words, when the caller's are in host memory (else null)
    int num_cus;
};
// The unpack stage: the same counting kernel, and one that writes the road table (event, set,
// hit_begin, nhits) and the grouped coordinates.  rec and tot as in UnitsLaunch.
hipError_t launch_unpack(const uint32_t *words, int64_t n_words, const svt_config &cfg,
                         const svt_roads &roads, int64_t road_cap, int16_t *hit_coord,
                         int64_t *d_n_roads, uint64_t *err, void *rec, void *tot, int num_cus,
                         hipStream_t s);
int64_t unit_rec_bytes(int64_t words);
int64_t unit_range_bytes();
int64_t unit_acc_bytes(int64_t combos);
int64_t unit_keep_bytes(int64_t words);
int64_t unit_keep_group_bytes(int64_t words);
int64_t unit_slot_bytes(int64_t words, bool less);
int64_t unit_ticket_bytes();
int64_t unit_bank_bytes();
hipError_t launch_units(const UnitsLaunch &p, hipStream_t s, hipEvent_t start, hipEvent_t stop);

}  // namespace svt
