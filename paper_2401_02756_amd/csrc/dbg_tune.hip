// Autotuner: times complete builds of a calibration input under candidate
// configurations and keeps the fastest.  The search is coordinate-wise:
// binned mode over load factors, then over its partition's scatter shapes (and,
// with set shapes, their launch: dbg_tune.h); then
// (unless binned mode is already far ahead) the direct build over launch
// shapes, wavefront merging and load factors.  Choices are cached in the
// process and in a cache file keyed by device model.
#include "dbg_runtime.h"
#include "dbg_tune.h"

#include <sys/stat.h>

#include <cerrno>
#include <chrono>
#include <cstdio>
#include <string>

using namespace dbgrt;

namespace {

struct Workload {
    int device;
    uint32_t m;
    const uint64_t *read_begin;
    const uint32_t *ks;
    const uint64_t *expected;
    const uint8_t *d_reads;
    uint64_t reads_len;
    const uint64_t *d_offsets;
    uint32_t keep_flags;
    uint32_t repeats;
};

struct Outcome {
    int rc = DBG_OK;
    double ms = 0;
    uint64_t vertices = 0, inserts = 0;
};

uint32_t cand_flags(const Cand &c, uint32_t keep) {
    return (keep & (DBG_F_GRAPH | DBG_F_ENTRY32 | DBG_F_TIMING)) | (c.binned ? DBG_F_BINNED : 0u) |
           (c.merge ? DBG_F_MERGE : 0u);
}

// Build the workload repeats + 1 times under `c`; the median host time of
// the timed builds (tables reset between them), and the graph totals.
Outcome time_candidate(const Workload &w, const Cand &c) {
    Outcome o;
    std::vector<dbg_graph *> gs(w.m, nullptr);
    for (uint32_t i = 0; i < w.m && o.rc == DBG_OK; ++i) {
        dbg_config cfg;
        dbg_config_init(&cfg);
        cfg.expected_vertices = w.expected ? w.expected[i] : 0;
        cfg.load_factor = c.lf;
        cfg.device = w.device;
        cfg.flags = cand_flags(c, w.keep_flags);
        cfg.block_size = c.block;
        cfg.windows_per_thread = c.wpt;
        cfg.bin_chunks = c.bin_chunks;
        cfg.bin_scatter_div = c.bin_div;
        cfg.bin_shape1 = c.bin_shape1;
        cfg.bin_shape2 = c.bin_shape2;
        o.rc = dbg_create(&cfg, &gs[i]);
    }
    std::vector<int32_t> st(w.m, DBG_OK);
    std::vector<double> t;
    for (uint32_t r = 0; r <= w.repeats && o.rc == DBG_OK; ++r) {
        // a build starts from an empty table: the reset (lazy for binned
        // tables, a zero fill for direct ones) is part of its cost
        const auto t0 = std::chrono::steady_clock::now();
        for (dbg_graph *g : gs) dbg_reset(g);
        if (w.m == 1) {
            const uint64_t *off = w.d_offsets;
            o.rc = dbg_build_device(gs[0], w.d_reads, w.reads_len, off, w.read_begin[1], w.ks[0], nullptr);
            if (o.rc == DBG_OK) o.rc = dbg_sync(gs[0]);
        } else {
            o.rc = dbg_build_batch_device(gs.data(), w.m, w.read_begin, w.ks, w.d_reads, w.reads_len, w.d_offsets,
                                          st.data(), nullptr);
        }
        const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        if (r) t.push_back(ms);
    }
    if (o.rc == DBG_OK) {
        std::sort(t.begin(), t.end());
        o.ms = t[t.size() / 2];
        for (dbg_graph *g : gs) {
            dbg_stats s;
            dbg_get_stats(g, &s);
            o.vertices += s.vertices;
            o.inserts += s.inserts;
        }
    }
    for (dbg_graph *g : gs) dbg_destroy(g);
    return o;
}

std::mutex g_tune_mu;
std::map<std::string, dbg_tuning> g_tune_cache;  // key -> tuning; from_cache says where it came from
bool g_file_loaded = false;

// The cache file's path ("" when there is none).
std::string cache_path() {
    if (const char *p = std::getenv("DBG_TUNE_CACHE")) return p;
    if (const char *x = std::getenv("XDG_CACHE_HOME"); x && *x) return std::string(x) + "/libdbg/autotune.tsv";
    if (const char *h = std::getenv("HOME"); h && *h) return std::string(h) + "/.cache/libdbg/autotune.tsv";
    return "";
}

// Read the cache file into the process cache (under g_tune_mu).  Lines are
// "key<TAB>lf flags block wpt bin_chunks bin_div shape1 shape2 best_ms default_ms"; later
// lines of a key override earlier ones; malformed lines are skipped.
void load_cache_file() {
    g_file_loaded = true;
    const std::string path = cache_path();
    if (path.empty()) return;
    FILE *f = std::fopen(path.c_str(), "r");
    if (!f) return;
    char line[512];
    while (std::fgets(line, sizeof line, f)) {
        char *tab = std::strchr(line, '\t');
        if (!tab) continue;
        *tab = 0;
        dbg_tuning t{};
        unsigned flags = 0, block = 0, wpt = 0, chunks = 0, div = 0, sh1 = 0, sh2 = 0;
        if (std::sscanf(tab + 1, "%lf %u %u %u %u %u %u %u %lf %lf", &t.load_factor, &flags, &block, &wpt, &chunks,
                        &div, &sh1, &sh2, &t.best_ms, &t.default_ms) != 10 ||
            sh1 > 4 || sh2 > 4)
            continue;
        if (!(t.load_factor > 0 && t.load_factor < 1) || (flags & ~(uint32_t)(DBG_F_BINNED | DBG_F_MERGE)))
            continue;
        t.flags = flags;
        t.block_size = block;
        t.windows_per_thread = wpt;
        t.bin_chunks = chunks;
        t.bin_scatter_div = div;
        t.bin_shape1 = sh1;
        t.bin_shape2 = sh2;
        t.from_cache = 2;
        g_tune_cache[line] = t;
    }
    std::fclose(f);
}

// Append a tuning to the cache file, creating its directory (best effort:
// a cache that cannot be written only costs a later process the search).
void save_cache_line(const std::string &key, const dbg_tuning &t) {
    const std::string path = cache_path();
    if (path.empty()) return;
    for (size_t i = 1; i < path.size(); ++i)
        if (path[i] == '/') {
            const std::string dir = path.substr(0, i);
            if (mkdir(dir.c_str(), 0755) != 0 && errno != EEXIST) return;
        }
    FILE *f = std::fopen(path.c_str(), "a");
    if (!f) return;
    std::fprintf(f, "%s\t%.6g %u %u %u %u %u %u %u %.6f %.6f\n", key.c_str(), t.load_factor, t.flags, t.block_size,
                 t.windows_per_thread, t.bin_chunks, t.bin_scatter_div, t.bin_shape1, t.bin_shape2, t.best_ms,
                 t.default_ms);
    std::fclose(f);
}

// The device model: what a tuning depends on besides the workload.
std::string device_model(int device) {
    hipDeviceProp_t p{};
    if (hipGetDeviceProperties(&p, device) != hipSuccess) return "unknown";
    char buf[160];
    std::snprintf(buf, sizeof buf, "%s:%dcu:%zumb", p.gcnArchName, p.multiProcessorCount,
                  (size_t)(p.totalGlobalMem >> 20));
    for (char *c = buf; *c; ++c)
        if (*c == '\t' || *c == ' ' || *c == '\n') *c = '_';
    return buf;
}

int size_bucket(uint64_t x) {  // half-octaves
    if (!x) return -1;
    return (int)std::floor(2.0 * std::log2((double)x));
}

std::string cache_key(const Workload &w) {
    uint64_t kmask = 0;  // bit k - 1 for each k in 2 .. 64
    uint64_t ev = 0;
    for (uint32_t i = 0; i < w.m; ++i) {
        kmask |= 1ull << (w.ks[i] - 1);
        ev += w.expected ? w.expected[i] : 0;
    }
    char buf[160];
    // the version: of what was timed.  v4: automatic shapes sort tiles
    std::snprintf(buf, sizeof buf, "v4/%u/%llx/%d/%d/%d/%x", w.m, (unsigned long long)kmask,
                  size_bucket(w.reads_len), size_bucket(w.read_begin[w.m]), size_bucket(ev), w.keep_flags);
    return device_model(w.device) + "/" + buf;
}

}  // namespace

extern "C" {

void dbg_config_apply_tuning(dbg_config *cfg, const dbg_tuning *t) {
    if (!cfg || !t) return;
    cfg->load_factor = t->load_factor;
    cfg->block_size = t->block_size;
    cfg->windows_per_thread = t->windows_per_thread;
    cfg->bin_chunks = t->bin_chunks;
    cfg->bin_scatter_div = t->bin_scatter_div;
    cfg->bin_shape1 = t->bin_shape1;
    cfg->bin_shape2 = t->bin_shape2;
    cfg->flags = (cfg->flags & ~(uint32_t)(DBG_F_BINNED | DBG_F_MERGE)) | (t->flags & (DBG_F_BINNED | DBG_F_MERGE));
}

int dbg_autotune(int32_t device, uint32_t m, const uint64_t *read_begin, const uint32_t *ks,
                 const uint64_t *expected_vertices, const uint8_t *d_reads, uint64_t reads_len,
                 const uint64_t *d_offsets, uint32_t keep_flags, uint32_t repeats, uint32_t tune_flags,
                 dbg_tuning *out) {
    if (!out || m == 0 || !read_begin || !ks || !d_offsets || (!d_reads && reads_len) || read_begin[0] != 0)
        return DBG_E_INVAL;
    bool all_binnable = true, wide = false;
    for (uint32_t i = 0; i < m; ++i) {
        // k > 32 only for a single graph (batched builds take k <= 32)
        if (ks[i] < 2 || ks[i] > (m == 1 ? 64u : 32u) || read_begin[i + 1] < read_begin[i]) return DBG_E_INVAL;
        // binned passes take k <= 31, and 33 <= k <= 63 for a single graph
        if (!(ks[i] <= 31 || (m == 1 && binnable_k(ks[i])))) all_binnable = false;
        if (ks[i] > 32) wide = true;
    }
    if (device < 0 && hipGetDevice(&device) != hipSuccess) return DBG_E_DEVICE;
    DeviceGuard guard(device);
    if (!guard.ok) return DBG_E_DEVICE;
    Workload w{device, m, read_begin, ks, expected_vertices, d_reads, reads_len, d_offsets, keep_flags,
               repeats ? repeats : 3u};
    const std::string key = cache_key(w);
    if (!(tune_flags & DBG_TUNE_FORCE)) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        if (!g_file_loaded) load_cache_file();
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end()) {
            *out = it->second;
            out->candidates = 0;
            it->second.from_cache = 1;  // served from this process from now on
            return DBG_OK;
        }
    }

    dbg_tuning best{};
    best.best_ms = 1e300;
    uint32_t n = 0;
    bool have_ref = false;
    uint64_t ref_v = 0, ref_i = 0;
    int first_rc = DBG_OK;
    auto consider = [&](const Cand &c) -> double {
        const Outcome o = time_candidate(w, c);
        ++n;
        if (!have_ref && o.rc != DBG_OK && first_rc == DBG_OK) first_rc = o.rc;
        if (o.rc != DBG_OK) return 1e300;
        if (!have_ref) {
            have_ref = true;
            ref_v = o.vertices;
            ref_i = o.inserts;
        } else if (o.vertices != ref_v || o.inserts != ref_i) {
            return 1e300;  // never chosen: its graph differs from the reference candidate's
        }
        if (o.ms < best.best_ms) {
            best.best_ms = o.ms;
            best.load_factor = c.lf;
            best.flags = (c.binned ? DBG_F_BINNED : 0u) | (c.merge ? DBG_F_MERGE : 0u);
            best.block_size = c.binned ? 0 : c.block;
            best.windows_per_thread = c.binned ? 0 : c.wpt;
            best.bin_chunks = c.binned ? c.bin_chunks : 0;
            best.bin_scatter_div = c.binned ? c.bin_div : 0;
            best.bin_shape1 = c.binned ? c.bin_shape1 : 0;
            best.bin_shape2 = c.binned ? c.bin_shape2 : 0;
        }
        return o.ms;
    };

    double binned_best = 1e300;
    if (all_binnable) (void)search_binned(consider, &binned_best, &best.default_ms);
    // direct build: launch shape, then merging, then load factor
    Cand dc{false, 0.5, 256, 4, false};
    double dbest = consider(dc);
    if (!all_binnable) best.default_ms = dbest;
    if (dbest < 1.5 * binned_best) {
        for (uint32_t block : kBlocks)
            for (uint32_t wpt : kWpts) {
                if (block == 256 && wpt == 4) continue;
                const Cand c{false, 0.5, block, wpt, false};
                const double ms = consider(c);
                if (ms < dbest) dbest = ms, dc = c;
            }
        if (!wide) {  // the long-k build does not merge
            Cand mc = dc;
            mc.merge = true;
            const double mms = consider(mc);
            if (mms < dbest) dbest = mms, dc = mc;
        }
        for (double lf : kLoadFactors) {
            if (lf == 0.5) continue;
            Cand c = dc;
            c.lf = lf;
            const double ms = consider(c);
            if (ms < dbest) dbest = ms, dc = c;
        }
    }
    if (best.best_ms >= 1e300) return first_rc != DBG_OK ? first_rc : DBG_E_DEVICE;
    if (best.default_ms >= 1e300) best.default_ms = 0;
    best.candidates = n;
    best.from_cache = 0;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        if (!g_file_loaded) load_cache_file();
        g_tune_cache[key] = best;
        g_tune_cache[key].from_cache = 1;
        save_cache_line(key, best);
    }
    *out = best;
    return DBG_OK;
}

int dbg_autotune_space(uint32_t binned, dbg_tuning *out, uint32_t cap, uint32_t *n) {
    if (!n || (cap && !out)) return DBG_E_INVAL;
    uint32_t k = 0;
    auto put = [&](double lf, uint32_t flags, uint32_t block, uint32_t wpt, uint32_t ch, uint32_t dv, uint32_t s1,
                   uint32_t s2) {
        if (k < cap) {
            dbg_tuning t{};
            t.load_factor = lf;
            t.flags = flags;
            t.block_size = block;
            t.windows_per_thread = wpt;
            t.bin_chunks = ch;
            t.bin_scatter_div = dv;
            t.bin_shape1 = s1;
            t.bin_shape2 = s2;
            out[k] = t;
        }
        ++k;
    };
    for (double lf : kLoadFactors) {
        if (binned) {
            for (uint32_t ch : kBinChunks)
                for (const auto &sh : kBinShapes)
                    for (uint32_t dv : kBinDivs) put(lf, DBG_F_BINNED, 0, 0, ch, dv, sh[0], sh[1]);
        } else {
            for (uint32_t block : kBlocks)
                for (uint32_t wpt : kWpts)
                    for (uint32_t merge : {0u, (uint32_t)DBG_F_MERGE}) put(lf, merge, block, wpt, 0, 0, 0, 0);
        }
    }
    *n = k;
    return DBG_OK;
}

}  // extern "C"
