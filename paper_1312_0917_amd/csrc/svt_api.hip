// Host side of the libsvt C ABI: argument checks, workspace layout and launch sequences.  Every
// function only enqueues on the given stream.
#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <mutex>

#include "svt_common.h"

namespace svt {
// launcher of k_gather (svt_stages.hip), used by svt_gather_results only
hipError_t launch_gather(const svt_roads &roads, const svt_best &best, int64_t road_cap,
                         const int64_t *d_n_words, const int64_t *d_n_roads,
                         const int64_t *d_n_combos, const int64_t *d_n_kept,
                         const uint64_t *d_err, void *out, int64_t out_roads, hipStream_t s);
}  // namespace svt

using namespace svt;

namespace {

constexpr int64_t kAlign = 256;
inline int64_t align_up(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

bool config_ok(const svt_config *c) {
    return c && c->n_layers == SVT_N_LAYERS && c->shift >= 1 && c->shift <= 30 &&
           c->max_hits >= 1 && c->max_hits <= SVT_MAX_HITS && c->n_sets >= 1 && c->n_sets <= 256;
}

bool aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Workspace carving: a bump allocator over the caller's buffer.
struct Carver {
    char *base;
    int64_t used = 0;
    template <typename T>
    T *take(int64_t count) {
        T *p = base ? reinterpret_cast<T *>(base + used) : nullptr;
        used += align_up(static_cast<int64_t>(sizeof(T)) * (count > 0 ? count : 1));
        return p;
    }
};

struct UnpackWs {
    void *rec;  // running counts per unit
    void *tot;  // totals per range of units
};
UnpackWs carve_unpack(Carver &c, int64_t n_words) {
    UnpackWs w;
    w.rec = c.take<char>(unit_rec_bytes(n_words > 0 ? n_words : 1));
    w.tot = c.take<char>(unit_range_bytes());
    return w;
}

struct BatchWs {
    uint32_t *ticket;   // event schedule: events handed out,
    int64_t *n_events;  // events of the batch,
    int32_t *efr;       // first road of every event,
    int64_t events_cap;
    int64_t *status;    // look-back status words of the pre-pass,
    int64_t status_words;
    int64_t nb;         // its blocks,
    int32_t *tfr;       // first road of every tile,
    int64_t tiles_cap;
    int64_t *kb;        // accepted combinations per kKeptBlock
    int64_t kbn;
    int16_t *coords;    // and grouped coordinates
    int64_t *nw_copy;   // the batch's word count, copied to device memory by the first kernel; in
                        // the unit kernels [1] tells the last one whether the fits ran
    void *sets;         // unit kernels: the packed bank,
    void *tot;          // totals per range of units,
    uint32_t *dealers;  // counters of the units dealt out late,
    void *rec;          // running counts per unit,
    void *acc;          // what the slices of a large unit share,
    void *keep;         // accepted combinations per unit
    int64_t *keep_groups;  // and per group of units,
    // 4 bytes a word that a workspace may do without: a copy of the words when the caller's are in
    // host memory, else more room for accepted combinations
    uint32_t *copy;
    bool host_words;
};
// What the unit kernels need besides, in bytes.
int64_t unit_bytes(int64_t word_cap, int64_t combo_cap) {
    return align_up(unit_bank_bytes()) + align_up(unit_range_bytes()) +
           align_up(unit_ticket_bytes()) + align_up(unit_acc_bytes(combo_cap)) +
           align_up(unit_rec_bytes(word_cap > 0 ? word_cap : 1)) +
           align_up(unit_keep_bytes(word_cap > 0 ? word_cap : 1)) +
           align_up(unit_keep_group_bytes(word_cap > 0 ? word_cap : 1)) +
           2 * kAlign;  // (slots for the last unit, a whole one, in the coordinates' place)
}
// `copy`: with those 4 bytes a word
BatchWs carve_batch(Carver &c, int64_t word_cap, int64_t road_cap, int64_t combo_cap,
                    bool copy) {
    BatchWs w;
    w.ticket = c.take<uint32_t>(4);
    w.n_events = c.take<int64_t>(2);
    w.events_cap = road_cap > 0 ? road_cap : 1;  // every event holds at least one road
    w.efr = c.take<int32_t>(w.events_cap);
    w.nb = ceil_div(word_cap > 0 ? word_cap : 1, kPrepassBlockWords);
    w.status_words = prepass_status_words(w.nb);
    // (the space taken is what it was when a schedule with blocks of 1024 words used it, and the
    // tiles' for 4096 combinations each: the static workspace then holds what it held)
    const int64_t pairs = 2 * ceil_div(word_cap > 0 ? word_cap : 1, 1024);
    w.status = c.take<int64_t>(w.status_words > pairs ? w.status_words : pairs);
    w.tiles_cap = ceil_div(combo_cap > 0 ? combo_cap : 1, kKeptBlock) + 1;
    w.tfr = c.take<int32_t>(w.tiles_cap);
    w.kbn = ceil_div(combo_cap > 0 ? combo_cap : 1, kKeptBlock);
    w.kb = c.take<int64_t>(w.kbn);
    // grouped coordinates, with slack for 16-byte reads of the last span; the unit kernels keep
    // their accepted combinations there when they have no better place
    const int64_t slots = unit_slot_bytes(word_cap > 0 ? word_cap : 1, true) / 2;
    w.coords = c.take<int16_t>(word_cap + 16 > slots ? word_cap + 16 : slots);
    w.nw_copy = c.take<int64_t>(2);
    w.sets = c.take<char>(unit_bank_bytes());
    w.tot = c.take<char>(unit_range_bytes());
    w.dealers = c.take<uint32_t>(unit_ticket_bytes() / 4);
    w.rec = c.take<char>(unit_rec_bytes(word_cap > 0 ? word_cap : 1));
    w.acc = c.take<char>(unit_acc_bytes(combo_cap));
    w.keep = c.take<char>(unit_keep_bytes(word_cap > 0 ? word_cap : 1));
    w.keep_groups = c.take<int64_t>(unit_keep_group_bytes(word_cap > 0 ? word_cap : 1) / 8);
    w.copy = copy ? c.take<uint32_t>(unit_slot_bytes(word_cap > 0 ? word_cap : 1, false) / 4)
                  : nullptr;
    return w;
}
int64_t batch_bytes(int64_t word_cap, int64_t road_cap, int64_t combo_cap, bool copy) {
    Carver c{nullptr};
    carve_batch(c, word_cap, road_cap, combo_cap, copy);
    return c.used;
}

// Schedules TILES and ONEPASS run the same unit kernels (svt_units.hip); of the two, a zero
// schedule resolves to ONEPASS up to this many words (capacity), as it did when they differed.
constexpr int64_t kOnepassDefaultWords = 1 << 19;

bool tune_supported(const svt_tune &t) {
    const bool wg_ok = t.wg_size == 256 || t.wg_size == 512;
    const bool ch_ok = t.chunk_roads == 16 || t.chunk_roads == 32 || t.chunk_roads == 64;
    const bool tile_ok = t.tile_combos >= kKeptBlock && t.tile_combos <= kMaxTile &&
                         t.tile_combos % kKeptBlock == 0;
    const int occ_max = (t.schedule == SVT_SCHEDULE_ONEPASS || t.schedule == 0) ? 3 : 8;
    const bool occ_ok = t.wgs_per_cu >= 1 && t.wgs_per_cu <= occ_max;
    const bool sched_ok = t.schedule == 0 || t.schedule == SVT_SCHEDULE_TILES ||
                          t.schedule == SVT_SCHEDULE_EVENTS || t.schedule == SVT_SCHEDULE_ONEPASS;
    return wg_ok && ch_ok && tile_ok && occ_ok && sched_ok;
}

// Launch parameters for `t` (zero fields take the defaults).  A zero schedule stays zero when
// no capacity is given (word_cap < 0), and is chosen from the capacity otherwise.
svt_tune resolve_tune(const svt_tune *t, int64_t word_cap = -1) {
    svt_tune r{4096, 64, 256, 3, 0};
    if (t) {
        if (t->tile_combos) r.tile_combos = t->tile_combos;
        if (t->chunk_roads) r.chunk_roads = t->chunk_roads;
        if (t->wg_size) r.wg_size = t->wg_size;
        if (t->wgs_per_cu) r.wgs_per_cu = t->wgs_per_cu;
        if (t->schedule) r.schedule = t->schedule;
    }
    if (r.schedule == 0 && word_cap >= 0)
        r.schedule = word_cap <= kOnepassDefaultWords ? SVT_SCHEDULE_ONEPASS : SVT_SCHEDULE_TILES;
    return r;
}

// A tune is valid when its fields are, before the capacity picks a zero schedule (which must
// then suit both schedules), and after.
bool tune_ok(const svt_tune *t, int64_t word_cap) {
    return tune_supported(resolve_tune(t)) &&
           tune_supported(resolve_tune(t, word_cap));
}

int num_cus() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    static std::mutex mu;
    static std::map<int, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n = 0;
    cache[dev] = n;
    return n;
}

#define SVT_TRY(x)                                  \
    do {                                            \
        if ((x) != hipSuccess) return SVT_ERR_HIP;  \
    } while (0)

hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;
}  // namespace

extern "C" {

int32_t svt_abi_version(void) { return SVT_ABI_VERSION; }

svt_status svt_copy_async(void *dst, const void *src, int64_t bytes, int32_t kind,
                          hipStream_t stream) {
    if (bytes < 0 || (bytes > 0 && (!dst || !src))) return SVT_ERR_ARG;
    if (kind != SVT_COPY_H2D && kind != SVT_COPY_D2H) return SVT_ERR_ARG;
    if (bytes == 0) return SVT_OK;
    const hipMemcpyKind k = kind == SVT_COPY_H2D ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost;
    return hipMemcpyAsync(dst, src, static_cast<size_t>(bytes), k, stream) == hipSuccess
               ? SVT_OK
               : SVT_ERR_HIP;
}

svt_status svt_event_record(hipEvent_t event, hipStream_t stream) {
    if (!event) return SVT_ERR_ARG;
    return hipEventRecord(event, stream) == hipSuccess ? SVT_OK : SVT_ERR_HIP;
}

int32_t svt_event_done(hipEvent_t event) {
    if (!event) return SVT_ERR_ARG;
    const hipError_t e = hipEventQuery(event);
    if (e == hipSuccess) return 1;
    if (e == hipErrorNotReady) return 0;
    return SVT_ERR_HIP;
}

svt_status svt_mapped_pointer(void *host, void **dev) {
    if (!host || !dev) return SVT_ERR_ARG;
    *dev = nullptr;
    return hipHostGetDevicePointer(dev, host, 0) == hipSuccess && *dev ? SVT_OK : SVT_ERR_HIP;
}

svt_status svt_gather_results(const svt_roads *roads, const svt_best *best, int64_t road_cap,
                              const int64_t *d_n_words, const int64_t *d_n_roads,
                              const int64_t *d_n_combos, const int64_t *d_n_kept,
                              const uint64_t *d_err, void *out, int64_t out_roads,
                              hipStream_t stream) {
    if (!roads || !best || !d_n_words || !d_n_roads || !d_n_combos || !d_err || !out)
        return SVT_ERR_ARG;
    if (!roads->event || !roads->set || !best->n_accept || !best->k || !best->p0 || !best->p1 ||
        !best->p2 || !best->chi2)
        return SVT_ERR_ARG;
    if (road_cap < 0 || out_roads < 0 || out_roads > (INT64_MAX - 64) / 36) return SVT_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(out) % 8 != 0) return SVT_ERR_ARG;
    return launch_gather(*roads, *best, road_cap, d_n_words, d_n_roads, d_n_combos, d_n_kept, d_err,
                         out, out_roads, stream) == hipSuccess
               ? SVT_OK
               : SVT_ERR_HIP;
}

svt_status svt_tune_resolve(const svt_tune *tune, svt_tune *out) {
    if (!out) return SVT_ERR_ARG;
    *out = resolve_tune(tune);
    return tune_supported(*out) ? SVT_OK : SVT_ERR_ARG;
}

svt_status svt_tune_for_batch(const svt_tune *tune, int64_t word_cap, svt_tune *out) {
    if (!out || word_cap < 0) return SVT_ERR_ARG;
    *out = resolve_tune(tune, word_cap);
    return tune_ok(tune, word_cap) ? SVT_OK : SVT_ERR_ARG;
}

const char *svt_status_name(svt_status s) {
    switch (s) {
        case SVT_OK: return "SVT_OK";
        case SVT_ERR_ARG: return "SVT_ERR_ARG";
        case SVT_ERR_LAYER: return "SVT_ERR_LAYER";
        case SVT_ERR_HITS: return "SVT_ERR_HITS";
        case SVT_ERR_CAPACITY: return "SVT_ERR_CAPACITY";
        case SVT_ERR_HIP: return "SVT_ERR_HIP";
        case SVT_ERR_SET: return "SVT_ERR_SET";
        default: return "SVT_ERR_UNKNOWN";
    }
}

svt_status svt_error_decode(uint64_t err, int64_t *index) {
    if (err == SVT_NO_ERROR) {
        if (index) *index = -1;
        return SVT_OK;
    }
    const uint32_t cls = static_cast<uint32_t>(err >> 56);
    if (index) *index = static_cast<int64_t>(err & ((1ull << 56) - 1));
    switch (cls) {
        case SVT_ERRCLASS_LAYER: return SVT_ERR_LAYER;
        case SVT_ERRCLASS_HITS: return SVT_ERR_HITS;
        case SVT_ERRCLASS_SET: return SVT_ERR_SET;
        case SVT_ERRCLASS_CAPACITY: return SVT_ERR_CAPACITY;
        default: return SVT_ERR_ARG;
    }
}

int64_t svt_unpack_workspace(int64_t n_words) {
    if (n_words < 0) return -1;
    Carver c{nullptr};
    carve_unpack(c, n_words);
    return c.used;
}

int64_t svt_combine_workspace(int64_t n_roads) {
    if (n_roads < 0) return -1;
    return align_up(8 * ceil_div(n_roads > 0 ? n_roads : 1, kRoadBlock));
}

int64_t svt_select_workspace(int64_t n_combos) {
    if (n_combos < 0) return -1;
    return align_up(8 * ceil_div(n_combos > 0 ? n_combos : 1, kKeptBlock));
}

int64_t svt_batch_workspace(int64_t word_cap, int64_t road_cap, int64_t combo_cap,
                            const svt_tune *tune) {
    if (word_cap < 0 || word_cap > kMaxBatchWords || road_cap < 0 || combo_cap < 0) return -1;
    if (!tune_ok(tune, word_cap)) return -1;
    return batch_bytes(word_cap, road_cap, combo_cap, true);
}

svt_status svt_unpack(const uint32_t *words, int64_t n_words, const svt_config *cfg,
                      const svt_roads *roads, int64_t road_cap, int16_t *hit_coord,
                      int64_t *d_n_roads, uint64_t *d_err, void *d_work, int64_t work_bytes,
                      hipStream_t stream) {
    if (!config_ok(cfg) || !roads || n_words < 0 || road_cap < 0 || !d_n_roads || !d_err)
        return SVT_ERR_ARG;
    if (n_words > 0 && (!words || !hit_coord)) return SVT_ERR_ARG;
    if (road_cap > 0 && (!roads->event || !roads->set || !roads->hit_begin || !roads->nhits))
        return SVT_ERR_ARG;
    if (!d_work || work_bytes < svt_unpack_workspace(n_words) || !aligned(d_work, kAlign))
        return SVT_ERR_ARG;
    Carver c{static_cast<char *>(d_work)};
    UnpackWs w = carve_unpack(c, n_words);
    const int cus = num_cus();
    if (cus <= 0) return SVT_ERR_HIP;
    SVT_TRY(launch_unpack(words, n_words, *cfg, *roads, road_cap, hit_coord, d_n_roads, d_err,
                          w.rec, w.tot, cus, stream));
    return SVT_OK;
}

svt_status svt_combine(const svt_roads *roads, int64_t n_roads, const svt_config *cfg,
                       int32_t *combo_road, uint32_t *combo_hits, int64_t combo_cap,
                       int64_t *d_n_combos, uint64_t *d_err, void *d_work, int64_t work_bytes,
                       hipStream_t stream) {
    if (!config_ok(cfg) || !roads || n_roads < 0 || combo_cap < 0 || !d_n_combos || !d_err)
        return SVT_ERR_ARG;
    if (n_roads > 0 && (!roads->nhits || !roads->ncombo || !roads->combo_begin))
        return SVT_ERR_ARG;
    if (!d_work || work_bytes < svt_combine_workspace(n_roads) || !aligned(d_work, kAlign))
        return SVT_ERR_ARG;
    int64_t *rb = static_cast<int64_t *>(d_work);
    const int64_t rbn = ceil_div(n_roads > 0 ? n_roads : 1, kRoadBlock);
    const Sizes nr{n_roads, nullptr, n_roads};
    const bool listing = combo_road || combo_hits;
    SVT_TRY(launch_combo_count(*roads, nr, rbn, rb, d_err, stream));
    SVT_TRY(launch_scan(rb, nr, kRoadBlock, d_n_combos, listing ? combo_cap : -1, 1, d_err, true,
                        stream));
    SVT_TRY(launch_combo_begin(*roads, nr, rbn, rb, listing ? combo_road : nullptr, combo_cap,
                               d_err, stream));
    if (listing)
        SVT_TRY(launch_materialize(*roads, n_roads, d_n_combos, combo_cap, combo_road, combo_hits,
                                   d_err, stream));
    return SVT_OK;
}

svt_status svt_fit(const svt_fconst *bank, const svt_config *cfg, const svt_roads *roads,
                   int64_t n_roads, const int16_t *hit_coord, int64_t n_hits,
                   const int32_t *combo_road, const uint32_t *combo_hits, int64_t n_combos,
                   const svt_fitrec *out, uint64_t *d_err, hipStream_t stream) {
    if (!config_ok(cfg) || !roads || !out || !d_err || n_roads < 0 || n_hits < 0 || n_combos < 0)
        return SVT_ERR_ARG;
    if (n_combos > 0 && (!bank || !hit_coord || !combo_road || !combo_hits || !out->p0 ||
                         !out->p1 || !out->p2 || !out->chi2 || !roads->nhits ||
                         !roads->hit_begin || !roads->set))
        return SVT_ERR_ARG;
    const int cus = num_cus();
    if (cus <= 0) return SVT_ERR_HIP;
    SVT_TRY(launch_fit_plain(bank, *cfg, *roads, n_roads, hit_coord, n_hits, combo_road,
                             combo_hits, n_combos, *out, d_err, cus, stream));
    return SVT_OK;
}

svt_status svt_select(const svt_config *cfg, const svt_roads *roads, int64_t n_roads,
                      const int32_t *combo_road, const svt_fitrec *rec, int64_t n_combos,
                      uint8_t *accept, const svt_best *best, int64_t *kept, int64_t kept_cap,
                      int64_t *d_n_kept, uint64_t *d_err, void *d_work, int64_t work_bytes,
                      hipStream_t stream) {
    if (!config_ok(cfg) || !roads || !rec || !best || !d_err || n_roads < 0 || n_combos < 0 ||
        kept_cap < 0)
        return SVT_ERR_ARG;
    if (n_combos > 0 && (!combo_road || !rec->chi2 || !rec->p0 || !rec->p1 || !rec->p2 ||
                         !accept || !roads->combo_begin))
        return SVT_ERR_ARG;
    if (n_roads > 0 && (!best->n_accept || !best->k || !best->p0 || !best->p1 || !best->p2 ||
                        !best->chi2 || !roads->combo_begin || !roads->ncombo))
        return SVT_ERR_ARG;
    if (kept && !d_n_kept) return SVT_ERR_ARG;
    if (!d_work || work_bytes < svt_select_workspace(n_combos) || !aligned(d_work, kAlign))
        return SVT_ERR_ARG;
    int64_t *kb = static_cast<int64_t *>(d_work);
    const int64_t kbn = ceil_div(n_combos > 0 ? n_combos : 1, kKeptBlock);
    SVT_TRY(launch_select(*cfg, *roads, n_roads, combo_road, *rec, n_combos, accept, *best, kb,
                          d_err, stream));
    if (d_n_kept) {
        const Sizes nc{n_combos, nullptr, n_combos};
        SVT_TRY(launch_scan(kb, nc, kKeptBlock, d_n_kept, kept ? kept_cap : -1, 2, d_err, true,
                            stream));
        if (kept && n_combos > 0)
            SVT_TRY(launch_kept_write(accept, nc, kbn, kb, kept, kept_cap, d_err, stream));
    }
    return SVT_OK;
}

void svt_set_fused_timing_events(hipEvent_t start, hipEvent_t stop) {
    g_ev_start = start;
    g_ev_stop = stop;
}

static svt_status batch_sequence(const UnitsLaunch &o, const svt_tune &t, const BatchWs &w,
                                 bool timing, hipStream_t stream) {
    if (t.schedule != SVT_SCHEDULE_EVENTS) {  // two kernels, and with a kept list a third
        SVT_TRY(launch_units(o, stream, timing ? g_ev_start : nullptr,
                             timing ? g_ev_stop : nullptr));
        return SVT_OK;
    }
    uint64_t *err = o.err;
    PrepassLaunch p{};
    p.words = o.words;
    p.nw = Sizes{0, o.d_n_words, o.word_cap};
    p.cfg = o.cfg;
    p.roads = o.roads;
    p.road_cap = o.road_cap;
    p.coords = w.coords;
    p.best = o.best;
    p.tile_combos = t.tile_combos;
    p.tile_first_road = w.tfr;
    p.tiles_cap = w.tiles_cap;
    p.combo_cap = o.combo_cap;
    p.d_n_roads = o.d_n_roads;
    p.d_n_combos = o.d_n_combos;
    p.status = w.status;
    p.nb_cap = w.nb;
    p.status_words = w.status_words;
    p.ticket = w.ticket;
    p.err = err;
    p.event_first_road = w.efr;
    p.event_cap = w.events_cap;
    p.d_n_events = w.n_events;
    // (the kept-list block counts are cleared with the rest: the event kernel adds to them)
    SVT_TRY(launch_batch_reset(p, w.nw_copy, o.d_n_kept, o.d_n_kept ? w.kb : nullptr,
                               o.d_n_kept ? w.kbn : 0, stream));
    // after the reset the kernels read the word count from its copy in device memory
    p.nw = Sizes{0, w.nw_copy, o.word_cap};
    SVT_TRY(launch_prepass(p, stream));
    EventsLaunch f{};
    f.bank = o.bank;
    f.cfg = o.cfg;
    f.wgs_per_cu = t.wgs_per_cu;
    f.coords = w.coords;
    f.roads = o.roads;
    f.d_n_roads = o.d_n_roads;
    f.d_n_combos = o.d_n_combos;
    f.d_n_events = w.n_events;
    f.event_first_road = w.efr;
    f.rec = o.out;
    f.accept = o.accept;
    f.best = o.best;
    f.kb_counts = o.d_n_kept ? w.kb : nullptr;
    f.ticket = w.ticket;
    f.err = err;
    f.road_cap = o.road_cap;
    f.combo_cap = o.combo_cap;
    f.event_cap = w.events_cap;
    f.num_cus = o.num_cus;
    f.kept_only = o.kept_only;
    if (timing) SVT_TRY(hipEventRecord(g_ev_start, stream));
    SVT_TRY(launch_fit_events(f, stream));
    if (timing) SVT_TRY(hipEventRecord(g_ev_stop, stream));
    const Sizes nr{0, o.d_n_roads, o.road_cap};
    const Sizes nc{0, o.d_n_combos, o.combo_cap};
    // the kept list's block counts are scanned by one extra workgroup of the finalize launch
    ScanJob job;
    if (o.d_n_kept) {
        job.data = w.kb;
        job.n = nc;
        job.div = kKeptBlock;
        job.tot = o.d_n_kept;
        job.cap = o.kept ? o.kept_cap : -1;
        job.cap_index = 2;
    }
    SVT_TRY(launch_best_finalize(o.roads, nr, o.kept_only ? svt_fitrec{} : o.out, nc, o.best,
                                 o.cfg.chi2_cut, err, true, o.bank, w.coords, o.cfg.shift, job,
                                 stream));
    if (o.kept && o.kept_only)
        SVT_TRY(launch_kept_refit(o.accept, nc, nr, w.kbn, w.kb, o.roads, w.tfr, t.tile_combos,
                                  o.bank, o.cfg.n_sets, w.coords, o.cfg.shift, o.kept, o.out,
                                  o.kept_cap, err, stream));
    else if (o.kept)
        SVT_TRY(launch_kept_write(o.accept, nc, w.kbn, w.kb, o.kept, o.kept_cap, err, stream));
    return SVT_OK;
}

}  // extern "C"

namespace {

// ---- the workspace of svt_process_batch_static ----------------------------------------------
// One array per GPU in this library's code object, held until the process ends.  In host code
// its name is only the runtime's handle for it: the device address is taken once per device
// with hipGetSymbolAddress and used everywhere instead.
// (The unit kernels' part comes on top of SVT_STATIC_WORK_BYTES.  A batch that the rest admits has
// fewer than 2^24 words and 12e9 combinations, for they take 2 bytes a word and 12 bytes per 4096
// combinations there: 3 MiB for the units, 24 MB for the slices.)
constexpr int64_t kStaticUnitBytes = 30ll << 20;
static __device__ __align__(256) char scratch[SVT_STATIC_WORK_BYTES + kStaticUnitBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

svt_status static_workspace(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SVT_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SVT_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SVT_OK;
}

bool in_host_memory(const void *p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();  // not an address the runtime knows: take it as the caller's word
        return false;
    }
    return at.type == hipMemoryTypeHost;
}

// work_bytes value that selects the static workspace (d_work is then ignored)
constexpr int64_t kStaticWork = -2;

// svt_process_batch on the caller's workspace, or on the static one (work_bytes == kStaticWork).
svt_status process_batch(const svt_fconst *bank, const svt_config *cfg, const svt_tune *tune,
                         const uint32_t *words, const int64_t *d_n_words, int64_t word_cap,
                         const svt_roads *roads, int64_t road_cap, const svt_fitrec *rec,
                         uint8_t *accept, int64_t combo_cap, const svt_best *best, int64_t *kept,
                         int64_t kept_cap, int64_t *d_n_roads, int64_t *d_n_combos,
                         int64_t *d_n_kept, uint64_t *d_err, void *d_work, int64_t work_bytes,
                         int32_t flags, hipStream_t stream) {
    if (!config_ok(cfg) || !bank || !words || !d_n_words || !roads || !rec || !best ||
        !d_n_roads || !d_n_combos || !d_err || word_cap < 0 || word_cap > kMaxBatchWords ||
        road_cap < 0 || combo_cap < 0 ||
        kept_cap < 0)
        return SVT_ERR_ARG;
    if (kept && !d_n_kept) return SVT_ERR_ARG;
    const bool kept_only = (flags & SVT_BATCH_KEPT_ONLY) != 0;
    if (kept_only && (!kept || !d_n_kept)) return SVT_ERR_ARG;
    if (!roads->event || !roads->set || !roads->hit_begin || !roads->nhits ||
        !roads->combo_begin || !roads->ncombo)
        return SVT_ERR_ARG;
    if (!best->n_accept || !best->k || !best->p0 || !best->p1 || !best->p2 || !best->chi2)
        return SVT_ERR_ARG;
    if (!rec->p0 || !rec->p1 || !rec->p2 || !rec->chi2 || !accept) return SVT_ERR_ARG;
    const void *a16[] = {rec->p0, rec->p1, rec->p2, rec->chi2, rec->c0, rec->c1, rec->c2};
    for (const void *p : a16)
        if (p && !aligned(p, 16)) return SVT_ERR_ARG;
    if (!aligned(accept, 4)) return SVT_ERR_ARG;
    const svt_tune t = resolve_tune(tune, word_cap);
    if (!tune_ok(tune, word_cap)) return SVT_ERR_ARG;
    if (work_bytes == kStaticWork) {  // svt_process_batch_static
        if (flags & SVT_BATCH_GRAPH) return SVT_ERR_ARG;
        const int64_t limit = SVT_STATIC_WORK_BYTES + unit_bytes(word_cap, combo_cap);
        if (batch_bytes(word_cap, road_cap, combo_cap, false) > limit)
            return SVT_ERR_CAPACITY;
        const svt_status st = static_workspace(&d_work);
        if (st != SVT_OK) return st;
        work_bytes = limit;
    } else if (!d_work || work_bytes < svt_batch_workspace(word_cap, road_cap, combo_cap, &t) ||
               !aligned(d_work, kAlign)) {
        return SVT_ERR_ARG;
    }
    // words in host memory are read once over the bus: the counting kernel leaves a copy, where the
    // static workspace has room for one too (else both kernels read them in place)
    const bool copy = work_bytes >= batch_bytes(word_cap, road_cap, combo_cap, true);
    const int cus = num_cus();
    if (cus <= 0) return SVT_ERR_HIP;

    Carver c{static_cast<char *>(d_work)};
    BatchWs w = carve_batch(c, word_cap, road_cap, combo_cap, copy);
    w.host_words = copy && in_host_memory(words);
    UnitsLaunch o{};
    o.bank = bank;
    o.cfg = *cfg;
    o.words = words;
    o.d_n_words = d_n_words;
    o.word_cap = word_cap;
    o.roads = *roads;
    o.road_cap = road_cap;
    o.out = *rec;
    o.accept = accept;
    o.best = *best;
    o.combo_cap = combo_cap;
    o.d_n_roads = d_n_roads;
    o.d_n_combos = d_n_combos;
    o.err = d_err;
    o.d_n_kept = d_n_kept;
    o.kept = kept;
    o.kept_cap = kept_cap;
    o.kept_only = kept_only;
    o.nw_copy = w.nw_copy;
    o.ticket = w.dealers;
    o.sets = w.sets;
    o.rec = w.rec;
    o.tot = w.tot;
    o.acc = w.acc;
    o.keep = w.keep;
    o.keep_groups = w.keep_groups;
    o.less_slots = !w.copy || w.host_words;
    o.slots = o.less_slots ? static_cast<void *>(w.coords) : w.copy;
    o.copy = w.host_words ? w.copy : nullptr;
    o.num_cus = cus;

    // SVT_BATCH_GRAPH once replayed a captured graph of the launches.  A pass is two or three of
    // them now, and launching them takes the host 10 us where a replay takes 18 and holds the GPU
    // up a few more (750 events of 64 roads: 50 us a pass with a graph, 43 without), so they are
    // launched either way.  What a capture could not do is refused as before.
    if (flags & SVT_BATCH_GRAPH) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (!stream || hipStreamIsCapturing(stream, &st) != hipSuccess ||
            st != hipStreamCaptureStatusNone)
            return SVT_ERR_HIP;
    }
    const bool timing = !(flags & SVT_BATCH_GRAPH) && g_ev_start && g_ev_stop;
    return batch_sequence(o, t, w, timing, stream);
}

}  // namespace

extern "C" {

svt_status svt_process_batch(const svt_fconst *bank, const svt_config *cfg, const svt_tune *tune,
                             const uint32_t *words, const int64_t *d_n_words, int64_t word_cap,
                             const svt_roads *roads, int64_t road_cap, const svt_fitrec *rec,
                             uint8_t *accept, int64_t combo_cap, const svt_best *best,
                             int64_t *kept, int64_t kept_cap, int64_t *d_n_roads,
                             int64_t *d_n_combos, int64_t *d_n_kept, uint64_t *d_err,
                             void *d_work, int64_t work_bytes, int32_t flags,
                             hipStream_t stream) {
    if (work_bytes < 0) return SVT_ERR_ARG;
    return process_batch(bank, cfg, tune, words, d_n_words, word_cap, roads, road_cap, rec, accept,
                         combo_cap, best, kept, kept_cap, d_n_roads, d_n_combos, d_n_kept, d_err,
                         d_work, work_bytes, flags, stream);
}

svt_status svt_process_batch_static(const svt_fconst *bank, const svt_config *cfg,
                                    const svt_tune *tune, const uint32_t *words,
                                    const int64_t *d_n_words, int64_t word_cap,
                                    const svt_roads *roads, int64_t road_cap,
                                    const svt_fitrec *rec, uint8_t *accept, int64_t combo_cap,
                                    const svt_best *best, int64_t *kept, int64_t kept_cap,
                                    int64_t *d_n_roads, int64_t *d_n_combos, int64_t *d_n_kept,
                                    uint64_t *d_err, int32_t flags, hipStream_t stream) {
    return process_batch(bank, cfg, tune, words, d_n_words, word_cap, roads, road_cap, rec, accept,
                         combo_cap, best, kept, kept_cap, d_n_roads, d_n_combos, d_n_kept, d_err,
                         nullptr, kStaticWork, flags, stream);
}

svt_status svt_static_workspace_need(int64_t word_cap, int64_t road_cap, int64_t combo_cap,
                                     const svt_tune *tune, int64_t *need, int64_t *limit) {
    if (!need || !limit) return SVT_ERR_ARG;
    *limit = SVT_STATIC_WORK_BYTES;
    *need = svt_batch_workspace(word_cap, road_cap, combo_cap, tune);
    if (*need < 0) return SVT_ERR_ARG;
    *limit += unit_bytes(word_cap, combo_cap);
    if (*need > *limit)  // without room for a copy of the words
        *need = batch_bytes(word_cap, road_cap, combo_cap, false);
    return *need > *limit ? SVT_ERR_CAPACITY : SVT_OK;
}

void svt_release_graphs(void) {}  // (no graph is kept)

}  // extern "C"
