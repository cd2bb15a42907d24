// Host-side logic of the runtime, checked on the CPU (no device call is
// made): the binned table geometry, the size classes that key captured
// passes, and the host count of windows and k-mers that dbg_build uses to
// validate and size its input.  Prints one line per failure and "ok" at the
// end; the exit status is the number of failures (capped at 100).
#include "dbg_runtime.h"
#include "dbg_tune.h"

#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

static int failures = 0;
#define CHECK(cond, ...)                          \
    do {                                          \
        if (!(cond)) {                            \
            if (failures < 20) {                  \
                std::printf("FAIL %s: ", #cond);  \
                std::printf(__VA_ARGS__);         \
                std::printf("\n");                \
            }                                     \
            ++failures;                           \
        }                                         \
    } while (0)

static void check_geometry(uint64_t cap) {
    uint32_t d1 = 0, fan = 0;
    uint64_t parts = 0;
    const uint64_t want = std::max<uint64_t>(1, (cap + dbgk::kSegSlots - 1) / dbgk::kSegSlots);
    const bool ok = dbgrt::binned_geometry(cap, &d1, &fan, &parts);
    const bool fits = want <= (uint64_t)dbgk::kMaxD1 * dbgk::kMaxFan;
    if (!ok) {
        // refused only when no split into at most kMaxD1 x kMaxFan exists
        CHECK(!fits || std::ceil(std::sqrt((double)want)) > dbgk::kMaxD1, "cap %llu refused",
              (unsigned long long)cap);
        return;
    }
    CHECK(d1 >= 1 && d1 <= dbgk::kMaxD1, "cap %llu d1 %u", (unsigned long long)cap, d1);
    CHECK(fan >= 1 && fan <= dbgk::kMaxFan, "cap %llu fan %u", (unsigned long long)cap, fan);
    CHECK(parts == (uint64_t)d1 * fan, "cap %llu parts %llu", (unsigned long long)cap, (unsigned long long)parts);
    CHECK(parts >= want, "cap %llu: %llu segments for %llu wanted", (unsigned long long)cap,
          (unsigned long long)parts, (unsigned long long)want);
    // no whole bucket of spare segments, and fan never exceeds what d1 requires
    CHECK((uint64_t)(d1 - 1) * fan < want, "cap %llu: d1 %u fan %u over %llu", (unsigned long long)cap, d1, fan,
          (unsigned long long)want);
    CHECK((uint64_t)d1 * (fan - 1) < want, "cap %llu: fan %u larger than needed", (unsigned long long)cap, fan);
}

// A table has the same slots whatever its build's route, and the geometry found
// from its slots again is its own (dbg_build_device_static sizes by it).
static void check_table_geometry() {
    uint32_t d[3], f[3];
    uint64_t p[3];
    for (uint64_t s = 1; s <= 70000; s += s < 1100 ? 1 : 7) {
        const uint64_t cap = s * dbgk::kSegSlots - s % 2;
        CHECK(dbgrt::binned_geometry(cap, &d[0], &f[0], &p[0]) && dbgrt::table_geometry(cap, false, &d[1], &f[1], &p[1]) &&
                  dbgrt::table_geometry(cap, true, &d[2], &f[2], &p[2]), "%llu segments refused", (unsigned long long)s);
        CHECK(p[1] == p[0] && d[1] == d[0] && f[1] == f[0], "%llu segments: shaped", (unsigned long long)s);
        CHECK(p[2] == p[0] && (uint64_t)d[2] * f[2] == p[2], "%llu segments: %llu in two levels, %llu", (unsigned long long)s,
              (unsigned long long)p[0], (unsigned long long)p[2]);
        CHECK((f[2] == 1 && d[2] <= dbgk::kSingleParts) || p[2] > dbgk::kSingleParts, "%llu segments: levels", (unsigned long long)s);
        uint32_t d2, f2;
        uint64_t p2;
        CHECK(dbgrt::binned_geometry(p[2] * dbgk::kSegSlots, &d2, &f2, &p2) && p2 == p[0] && d2 == d[0] && f2 == f[0],
              "%llu segments: not found again", (unsigned long long)s);
    }
}

// What the kernels of a pass by sorted tiles address stays within the capacities
// and byte sizes reserved for it (sort_caps, SortSizes), for random tables,
// inputs and skew: the tiles and groups of level 1, transposed offsets and group
// sums of the two-level instances, and each bucket's tiles and records on whole
// lines in level 2, with a pair of records stored at an odd end.
static void check_sorted(std::mt19937_64 &rng) {
    for (int round = 0; round < 4000; ++round) {
        const uint32_t m = 1 + (uint32_t)(rng() % (round % 3 ? 6 : 200));
        const uint64_t len = 64 + rng() % (round % 4 ? (1ull << 23) : (1ull << 32));
        std::vector<Instance> in(m);
        for (Instance &x : in) {
            x = Instance{};
            uint64_t parts = 0;
            const uint64_t want = 1 + rng() % (rng() % 3 ? 3000 : 300000);
            if (!dbgrt::table_geometry(want * dbgk::kSegSlots, rng() % 8 != 0, &x.d1, &x.fan, &parts)) continue;
            x.parts = (uint32_t)parts;
            x.k = m == 1 && round % 2 ? 45 : 21;
            x.entry_words = x.k > 32 ? 4 : 3;
        }
        dbgk::BuildShape shape{256, 4, 0, 0};
        const dbgrt::PassKey k = dbgrt::pass_key(m, 1 + rng() % len, len, shape, true, in.data(), dbgrt::PassOpts{});
        CHECK(k.sorted, "round %d", round);
        dbgk::SortBuffers sb{};
        dbgrt::sort_caps(k, sb);
        const dbgrt::SortSizes z(k, sb);
        uint64_t tiles = 0, groups = 0, offt = 0, gsum = 0, buckets = 0, tiles2 = 0, at2 = 0, end2 = 0, left = len;
        for (uint32_t i = 0; i < m; ++i) {
            const uint64_t w = i + 1 == m ? left : (left ? rng() % (left + 1) : 0);  // its windows
            left -= w;
            const uint64_t t = (w + sb.tile1 - 1) / sb.tile1;
            tiles += t;
            CHECK(in[i].d1 + 1 <= sb.row1 && in[i].d1 <= sb.d1_max && in[i].fan + 1 <= sb.row2, "round %d: rows", round);
            if (in[i].fan == 1) continue;
            CHECK(sb.two_level && in[i].d1 <= k.d1_two_cap, "round %d: levels", round);
            const uint64_t g = (t + dbgk::kSortGroup - 1) / dbgk::kSortGroup;
            groups += g;
            offt += t * in[i].d1;
            gsum += g * in[i].d1;
            buckets += in[i].d1;
            uint64_t records = w;
            for (uint32_t b = 0; b < in[i].d1; ++b) {
                const uint64_t n = b + 1 == in[i].d1 ? records : std::min(records, rng() % (2 * (w / in[i].d1) + 2));
                records -= n;
                tiles2 += (n + sb.tile2 - 1) / sb.tile2;
                end2 = std::max(end2, at2 + n + (n & 1));
                at2 += (n + 15) & ~15ull;
            }
        }
        CHECK(tiles <= sb.tiles1_cap && groups <= sb.groups_cap && buckets <= sb.buckets_cap && tiles2 <= sb.tiles2_cap,
              "round %d: %llu tiles, %llu groups, %llu buckets, %llu tiles", round, (unsigned long long)tiles,
              (unsigned long long)groups, (unsigned long long)buckets, (unsigned long long)tiles2);
        CHECK(8 * tiles <= z.tile_read && 2 * tiles * sb.row1 <= z.off1 && 8 * k.rw * tiles * sb.tile1 <= z.rec1, "round %d: level 1", round);
        CHECK(4 * offt <= z.offt && 4 * gsum <= z.gsum && 8 * gsum <= z.gpre, "round %d: between", round);
        CHECK(2 * tiles2 * sb.row2 <= z.off2 && 8 * k.rw * end2 <= z.rec2, "round %d: level 2", round);
        CHECK(buckets * sizeof(dbgk::SortBucket) <= z.buckets && (!buckets || 8 * (buckets + 1) <= z.tile2_base), "round %d: buckets", round);
    }
}

// The search times no build twice (with automatic shapes chunks and divisor do
// nothing), finds the best of what it times, and tunes the scatter's launch where
// set shapes are the best.
static void check_tuner(std::mt19937_64 &rng) {
    for (int round = 0; round < 400; ++round) {
        std::vector<dbgrt::Cand> seen;
        double least = 1e300, at_half = 0;
        bool twice = false;
        const int favour = round % 3;  // automatic shapes, set ones, neither
        const auto consider = [&](const dbgrt::Cand &c) {
            const bool shaped = c.bin_shape1 || c.bin_shape2;
            for (const auto &x : seen)
                twice |= x.lf == c.lf && x.bin_shape1 == c.bin_shape1 && x.bin_shape2 == c.bin_shape2 &&
                         (!shaped || (x.bin_chunks == c.bin_chunks && x.bin_div == c.bin_div));
            seen.push_back(c);
            double ms = 1.0 + (double)(rng() % 1000) / 1000;
            if (favour == 0 && !shaped) ms /= 4;
            if (favour == 1 && shaped) ms /= 4;
            if (rng() % 20 == 0) ms = 1e300;
            least = std::min(least, ms);
            if (seen.size() == 1) at_half = ms;
            return ms;
        };
        double best_ms = 0, default_ms = 0;
        const dbgrt::Cand best = dbgrt::search_binned(consider, &best_ms, &default_ms);
        CHECK(!twice, "round %d: a build timed twice", round);
        CHECK(best_ms == least && default_ms == at_half, "round %d: %g of %g", round, best_ms, least);
        const bool shaped = best.bin_shape1 || best.bin_shape2;
        CHECK(seen.size() == (shaped ? 16u : 9u) && (shaped || (!best.bin_chunks && !best.bin_div)), "round %d: %zu candidates",
              round, seen.size());
    }
}

// The scatter shapes that a pass by sorted tiles reports are those of the two
// levels that the same table has in a count-and-scatter launch, also where its
// own tables have one.
static void check_reported_shapes() {
    for (uint64_t s = 1; s <= 600000; s += s < 1100 ? 1 : 997) {
        Instance one[2] = {}, two[2] = {};
        uint64_t parts = 0;
        for (int i = 0; i < 2; ++i) {
            const uint64_t cap = (i ? s : s / 3 + 1) * dbgk::kSegSlots;
            if (!dbgrt::table_geometry(cap, true, &one[i].d1, &one[i].fan, &parts)) return;
            one[i].parts = (uint32_t)parts;
            if (!dbgrt::binned_geometry(cap, &two[i].d1, &two[i].fan, &parts)) return;
            two[i].parts = (uint32_t)parts;
        }
        uint32_t most = 1;
        for (const Instance &x : two) most = std::max(most, x.d1);
        const uint32_t d1 = (uint32_t)std::min<uint64_t>(dbgrt::size_class(most, 16), dbgk::kMaxD1);
        CHECK(dbgrt::scatter_d1(one, 2) == d1, "%llu segments: %u, not %u", (unsigned long long)s, dbgrt::scatter_d1(one, 2), d1);
        CHECK(dbgk::auto_shapes(1, dbgrt::scatter_d1(one, 2)) == (d1 > 384 ? 0x304u : 0x303u), "%llu segments", (unsigned long long)s);
        CHECK(dbgk::auto_shapes(2, dbgrt::scatter_d1(one, 2)) == (d1 > 384 ? 0x303u : 0x301u), "%llu segments", (unsigned long long)s);
    }
}

static void check_size_class() {
    uint64_t prev = 0;
    for (uint64_t x = 0; x < 300000; ++x) {
        const uint64_t s = dbgrt::size_class(x, 64);
        CHECK(s >= x && s >= 64, "size_class(%llu) = %llu", (unsigned long long)x, (unsigned long long)s);
        CHECK(s >= prev, "size_class not monotone at %llu", (unsigned long long)x);
        // at most one eighth of the next power of two above x
        CHECK(x < 64 || s - x < std::max<uint64_t>(x / 4, 1), "size_class(%llu) = %llu too coarse",
              (unsigned long long)x, (unsigned long long)s);
        prev = s;
    }
    for (uint64_t x = 1; x < (1ull << 60); x = x * 5 / 3 + 1) {
        const uint64_t s = dbgrt::size_class(x, 1);
        CHECK(s >= x && s - x <= x / 4 + 1, "size_class(%llu) = %llu", (unsigned long long)x, (unsigned long long)s);
        CHECK(dbgrt::size_class(s, 1) == s, "size_class(%llu) not a fixed point", (unsigned long long)s);
    }
}

static void check_host_counts(std::mt19937_64 &rng) {
    for (int rep = 0; rep < 2000; ++rep) {
        const uint64_t n = rng() % 40;
        const uint32_t k = 2 + rng() % 63;
        std::vector<uint64_t> off(n + 1);
        off[0] = rng() % 1000;
        for (uint64_t i = 0; i < n; ++i) off[i + 1] = off[i] + (rng() % 4 == 0 ? rng() % 8 : rng() % 200);
        const bool decrease = n > 0 && rng() % 5 == 0;
        if (decrease) {
            const uint64_t i = 1 + rng() % n;
            if (off[i] > 0) off[i] = off[i - 1] - (off[i - 1] > 0 ? 1 : 0) * (1 + rng() % std::max<uint64_t>(1, off[i - 1]));
        }
        bool mono = true;
        uint64_t w = 0, e = 0;
        for (uint64_t i = 0; i < n; ++i) {
            if (off[i + 1] < off[i]) mono = false;
            else if (off[i + 1] - off[i] >= k) {
                w += off[i + 1] - off[i] - k + 2;  // windows: L - k + 2 vertices
                e += off[i + 1] - off[i] - k + 1;  // k-mers: L - k + 1 edges
            }
        }
        uint64_t hw = 12345, he = 6789;
        const bool ok = dbgrt::host_counts(off.data(), n, k, &hw, &he);
        CHECK(ok == mono, "rep %d: accepted %d, monotone %d", rep, (int)ok, (int)mono);
        if (ok && mono) CHECK(hw == w && he == e, "rep %d: %llu/%llu vs %llu/%llu", rep, (unsigned long long)hw,
                              (unsigned long long)he, (unsigned long long)w, (unsigned long long)e);
    }
}

// Chunk counts of the two partition passes stay within the capacities the
// runtime reserves (bin_caps): for random instance and bucket sizes, the
// chunk length max(1, floor(tiles / target)) that the plan kernels use gives
// at most chunks1_cap - 1 (pass 1) and chunks2_cap - 1 (pass 2) chunks, and
// the histograms fit.
static uint64_t chunks_of(const std::vector<uint64_t> &tiles, uint64_t target) {
    uint64_t all = 0;
    for (uint64_t t : tiles) all += t;
    const uint64_t chunk = std::max<uint64_t>(1, all / std::max<uint64_t>(target, 1));
    uint64_t n = 0;
    for (uint64_t t : tiles) n += (t + chunk - 1) / chunk;
    return n;
}

static void check_chunks(std::mt19937_64 &rng) {
    for (int round = 0; round < 3000; ++round) {
        const uint32_t m = 1 + (uint32_t)(rng() % (round % 3 ? 8 : 300));
        const uint64_t len = 4096 + rng() % (round % 5 ? (1ull << 24) : (1ull << 33));
        const uint32_t target = 1 + (uint32_t)(rng() % dbgk::kMaxChunkTarget);
        // windows of each instance: a random split of at most len
        std::vector<uint64_t> w(m), tiles(m);
        uint64_t left = len;
        for (uint32_t i = 0; i < m; ++i) {
            w[i] = i + 1 == m ? left : (left ? rng() % (left + 1) : 0);
            left -= w[i];
            tiles[i] = (w[i] + dbgk::kBinTile - 1) / dbgk::kBinTile;
        }
        dbgrt::PassKey k;
        k.binned = 1;
        k.m_cap = (uint32_t)dbgrt::size_class(m, 1);
        k.len_cap = dbgrt::size_class(len, 4096);
        const uint32_t d1 = 1 + (uint32_t)(rng() % dbgk::kMaxD1), fan = 1 + (uint32_t)(rng() % dbgk::kMaxFan);
        const uint64_t G = (uint64_t)m * d1;  // buckets over the launch
        k.buckets_cap = dbgrt::size_class(G, 64);
        k.d1_cap = (uint32_t)std::min<uint64_t>(dbgrt::size_class(d1, 16), dbgk::kMaxD1);
        k.fan_cap = (uint32_t)std::min<uint64_t>(dbgrt::size_class(fan, 16), dbgk::kMaxFan);
        dbgk::BinBuffers bb{};
        dbgrt::bin_caps(k, bb);
        const uint64_t c1 = chunks_of(tiles, target);
        CHECK(c1 + 1 <= bb.chunks1_cap, "pass 1: %llu chunks, cap %llu", (unsigned long long)c1,
              (unsigned long long)bb.chunks1_cap);
        CHECK((uint64_t)d1 * c1 <= bb.hist1_cap, "pass 1 histogram");
        // records (one per window) split over the G buckets
        std::vector<uint64_t> bt(G);
        uint64_t rec_left = len;
        for (uint64_t g = 0; g < G; ++g) {
            const uint64_t sz = g + 1 == G ? rec_left : (rec_left ? rng() % (2 * rec_left / (G - g) + 1) : 0);
            const uint64_t take = std::min(sz, rec_left);
            rec_left -= take;
            bt[g] = (take + dbgk::kRefTile - 1) / dbgk::kRefTile;
        }
        const uint64_t c2 = chunks_of(bt, target);
        CHECK(c2 + 1 <= bb.chunks2_cap, "pass 2: %llu chunks, cap %llu", (unsigned long long)c2,
              (unsigned long long)bb.chunks2_cap);
        CHECK((uint64_t)fan * c2 <= bb.hist2_cap, "pass 2 histogram");
    }
}

int main() {
    for (uint64_t cap = 0; cap < 200000; cap += 7) check_geometry(cap);
    for (uint64_t cap = 1; cap < (1ull << 45); cap = cap * 9 / 8 + 1) check_geometry(cap);
    // around every segment count near the square boundaries
    for (uint64_t s = 1; s <= 2048; ++s)
        for (int64_t d = -2; d <= 2; ++d) {
            const int64_t segs = (int64_t)(s * s) + d;
            if (segs > 0) check_geometry((uint64_t)segs * dbgk::kSegSlots);
        }
    check_table_geometry();
    check_reported_shapes();
    check_size_class();
    std::mt19937_64 rng(20240105);
    check_host_counts(rng);
    check_chunks(rng);
    check_tuner(rng);
    check_sorted(rng);
    if (failures) std::printf("%d failures\n", failures);
    else std::printf("ok\n");
    return failures > 100 ? 100 : failures;
}
