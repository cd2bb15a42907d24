// HIP kernels of the A-Bruijn graph build for gfx950 (MI355X).
//
// The per-k-mer work is the paper's makeGraph body (Methods, "Lock-free graph
// creation algorithm", Algorithms 2-4): look the source (k-1)-mer up, add it
// if absent, raise its counter for the k-mer's last letter; for the target
// (k-1)-mer only make sure it exists.  Both halves are expressed per window:
// window j of a read with L >= k is its (k-1)-mer at offset j, for
// j = 0 .. L-k+1; every window is found-or-claimed, and every window but the
// last also raises one counter.  Window j's target is window j+1 of the same
// read, so claiming every window is exactly "add left and right vertex".
//
// Differences from the paper's CPU structure, for the device:
//   * open addressing with linear probing instead of chained buckets: a slot
//     goes from empty to one key once, by a 64-bit compare-and-swap (the
//     paper's CAS, Algorithm 1), and never changes key afterwards, so a
//     non-empty value read once is final and no list has to be walked;
//   * the key is the packed (k-1)-mer itself, so the paper's string compare
//     (Algorithm 4) is one 64-bit compare and no read has to stay resident;
//   * the out-edge pointers are not stored: the target of (v, c) is
//     (v << 2 | c) masked to 2(k-1) bits;
//   * counters are uint32, not uint8 (255 is exceeded by repeat-rich inputs).
#include "dbg_device.h"

#include <algorithm>

namespace dbgk {
namespace {
// ---------------------------------------------------------------- begin

// The pass's argument block and instances, from pinned host memory (read once
// over the link: a copy command and this kernel's own launch take longer than
// the few hundred bytes do), its statuses and cursors, and the counters of its end.
constexpr uint32_t kInstWords = sizeof(Instance) / 8;
static_assert(sizeof(Instance) % 8 == 0, "copied in words");

__global__ void k_begin(const uint64_t *host, PassArgs *args, Instance *inst, InstStatus *st, CallState *cs,
                        uint64_t *done, uint32_t n_done) {
    const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    for (uint32_t i = x; i < n_done; i += stride) done[i] = 0;
    const PassArgs *a = host ? reinterpret_cast<const PassArgs *>(host) : args;
    const Instance *in = host ? reinterpret_cast<const Instance *>(host + kArgsBytes / 8) : inst;
    const uint32_t m = a->m;
    const uint64_t n = a->n_reads;
    const uint64_t *off = as_global(a->off);
    if (host) {
        if (x < sizeof(PassArgs) / 8) reinterpret_cast<uint64_t *>(args)[x] = host[x];
        for (uint32_t w = x; w < m * kInstWords; w += stride) {
            const uint32_t f = w % kInstWords;
            if (f == offsetof(Instance, byte_begin) / 8 || f == offsetof(Instance, byte_end) / 8) continue;
            reinterpret_cast<uint64_t *>(inst)[w] = host[kArgsBytes / 8 + w];
        }
    }
    for (uint32_t i = x; i < m; i += stride) {
        InstStatus s{};
        s.err = in[i].skip ? kErrSkip : 0u;
        st[i] = s;
        // byte range of the instance, relative to the first read's first byte
        uint64_t b0 = 0, b1 = 0;
        if (n) {
            const uint64_t off0 = off[0];
            b0 = off[min(in[i].read_begin, n)] - off0;
            b1 = off[min(in[i].read_end, n)] - off0;
        }
        inst[i].byte_begin = b0;
        inst[i].byte_end = b1;
    }
    if (x == 0) *cs = CallState{};
}

// Words for the host, in its pinned memory: a kernel behind another costs 5 us,
// the runtime's copy of a few bytes 10 to 20.
__global__ void k_store_words(const uint64_t *from, uint64_t *to, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        to[i] = from[i];
}

__global__ void k_fill_zero(uint64_t *__restrict__ words, uint64_t n_words) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t pairs = n_words >> 1;
    ulonglong2 *w2 = reinterpret_cast<ulonglong2 *>(words);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < pairs; i += stride)
        w2[i] = make_ulonglong2(0ull, 0ull);
    if ((n_words & 1) && blockIdx.x == 0 && threadIdx.x == 0) words[n_words - 1] = 0;
}

__global__ void k_gather_u64(const uint64_t *__restrict__ src, const uint64_t *__restrict__ idx, uint64_t n,
                             uint64_t *__restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = src[idx[i]];
}

// ---------------------------------------------------------------- pack

// One thread per output word: 32 bases, letter code (c >> 1) & 3, first base
// in bits 63..62.  Words past the input are zero (the build reads one word
// beyond the last base of a window).
__global__ __launch_bounds__(256) void k_pack(const PassArgs *__restrict__ args,
                                             uint64_t *__restrict__ packed,
                                             const Instance *__restrict__ inst, InstStatus *st) {
    const uint8_t *__restrict__ ascii = as_global(args->reads);
    const uint64_t n = args->reads_len;
    const uint64_t n_words = packed_words(n);
    const uint32_t m = args->m;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const bool aligned = (reinterpret_cast<uintptr_t>(ascii) & 15) == 0;
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < n_words; w += stride) {
        const uint64_t b0 = w * 32;
        uint64_t v = 0;
        uint32_t bad = 0;  // bit i: byte b0 + i is not a letter
        if (aligned && b0 + 32 <= n) {
            const uint4 *src = reinterpret_cast<const uint4 *>(ascii + b0);
            const uint4 lo = src[0], hi = src[1];
            const uint32_t q[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const uint32_t c = (q[i >> 2] >> (8 * (i & 3))) & 0xffu;
                v |= (uint64_t)((c >> 1) & 3u) << (62 - 2 * i);
                bad |= (valid_letter(c) ? 0u : 1u) << i;
            }
        } else {
            for (int i = 0; i < 32; ++i) {
                if (b0 + i >= n) break;
                const uint32_t c = ascii[b0 + i];
                v |= (uint64_t)((c >> 1) & 3u) << (62 - 2 * i);
                bad |= (valid_letter(c) ? 0u : 1u) << i;
            }
        }
        packed[w] = v;
        while (bad) {
            const int i = __builtin_ctz(bad);
            bad &= bad - 1;
            const uint32_t t = (m == 1) ? 0u : instance_of_byte(inst, m, b0 + i);
            atomic_or_u32(&st[t].err, kErrBase);
        }
    }
}

// ---------------------------------------------------------------- scan

// Windows and k-mers of one read.  A read with bad offsets has none (the
// instance is flagged and the build skips it).
struct ReadCount {
    uint64_t windows, kmers;
    bool bad;
};

// Read r lies at [a, b).
__device__ __forceinline__ ReadCount count_read(uint64_t a, uint64_t b, uint64_t off0, uint64_t r, uint64_t n,
                                                uint64_t len, bool check_ends, uint32_t k) {
    ReadCount rc{0, 0, false};
    if (b < a || a < off0 || b - off0 > len) {
        rc.bad = true;
        return rc;
    }
    if (check_ends && r + 1 == n && b - off0 != len) rc.bad = true;
    const uint64_t L = b - a;
    if (L >= k) {
        rc.windows = L - k + 2;
        rc.kmers = L - k + 1;
    }
    return rc;
}

// Offsets that overlap can sum to anything: a block's sum stops here, above any
// valid total and low enough for the sum of all blocks not to wrap.
constexpr uint64_t kMostOfBlock = 1ull << 40;

// Sum of v over the block's threads (each gets it).
__device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t *s_wave) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0;
    for (uint32_t i = 0; i < kScanBlock / 64; ++i) v += s_wave[i];
    __syncthreads();
    return v;
}

// Windows per read and their exclusive prefix, the first read of every tile,
// the k-mers and windows of each instance, and the plan of a one-instance pass
// by sorted tiles.  One launch counts (a pair of sums per block of 8192 reads),
// a second scans, each block adding up the sums before its own; reads that fit
// one block take a single launch that does both.
// In a batch, a block whose reads all belong to one instance, as they almost
// always do, adds its totals to it with one atomic (one for each wavefront: 114
// us instead of 32 for 16 sets), else a wavefront or a lane.  Valid offsets give at most
// one window per byte, which is what the buffers are sized for; overlapping
// (malformed) offsets can exceed that, and then every instance is flagged
// invalid and no window is processed.
// Bound by latency: a lane's loads are issued together, a row of 64 reads at a
// time.  20 us for 0.93 million reads and 61 for 2.2 million of which one in ten
// has no window (count, map and tile map were four launches of 57 and 73 us with
// their gaps).  A single launch over all blocks that hands out tickets and looks
// back at the blocks before took 19 and 57 us, but 158 against 89 for a batch of
// 48 sets: each ticket and each look at a watched line takes its turn.
template <bool COUNT, bool WRITE>
__global__ __launch_bounds__(kScanBlock) void k_scan(
    const PassArgs *__restrict__ args, const Instance *__restrict__ inst, InstStatus *st,
    uint64_t *__restrict__ ws, uint64_t *sums, uint64_t *__restrict__ tile_read, CallState *cs,
    SortPlan *__restrict__ plan, SortTotals *__restrict__ tot) {
    __shared__ uint64_t s_wave[kScanBlock / 64];
    __shared__ uint32_t s_inst[kScanBlock / 64];
    const uint64_t *__restrict__ off = as_global(args->off);
    const uint8_t *__restrict__ ascii = as_global(args->reads);
    const uint64_t n = args->n_reads, len = args->reads_len, tile_cap = args->tile_cap;
    const uint32_t m = args->m, check_ends = args->check_ends, tile = args->tile;
    const uint64_t block = blockIdx.x, rb = block * kScanReads;
    if (rb >= n) {  // grid sized for the capacity
        if (WRITE && n == 0 && block == 0 && threadIdx.x == 0 && plan) {
            *plan = SortPlan{};
            *tot = SortTotals{};
        }
        return;
    }
    const bool last_block = rb + kScanReads >= n, single = m == 1;
    const uint64_t off0 = off[0];
    // A wavefront has 64 * kScanPerThread reads, a lane every 64th of them.
    const uint64_t first = rb + (uint64_t)(threadIdx.x & ~63u) * kScanPerThread, r0 = first + (threadIdx.x & 63);
    uint64_t at[kScanPerThread], to[kScanPerThread];  // where the reads lie: all loads first
#pragma unroll
    for (uint32_t i = 0; i < kScanPerThread; ++i) {
        at[i] = off[min(r0 + 64 * i, n - 1)];
        to[i] = off[min(r0 + 64 * i, n - 1) + 1];
    }
    uint64_t before = 0, kbefore = 0;  // the blocks before
    if (WRITE && !COUNT) {
        for (uint64_t i = threadIdx.x; i < block; i += kScanBlock) {
            before += sums[2 * i];
            if (last_block) kbefore += sums[2 * i + 1];
        }
        before = block_sum(before, s_wave);
        if (last_block) kbefore = block_sum(kbefore, s_wave);
    }
    const uint32_t t0 = single ? 0u : instance_of_read(inst, m, min(first, n - 1));
    const bool uniform = single || t0 + 1 == m || inst[t0 + 1].read_begin >= min(first + 64 * kScanPerThread, n);
    const uint32_t t1 = uniform ? t0 : instance_of_read(inst, m, min(first + 64 * kScanPerThread, n) - 1);
    const uint32_t k0 = inst[t0].k;
    uint64_t w[kScanPerThread];
    uint64_t tw = 0, tk = 0;
    uint32_t bad = 0, bare = 0;  // bit i: this read's offsets are bad, it has no window
#pragma unroll
    for (uint32_t i = 0; i < kScanPerThread; ++i) {
        const uint64_t r = r0 + 64 * i;
        const uint32_t k = uniform ? k0 : inst[instance_of_read(inst, t0, t1 + 1, min(r, n - 1))].k;
        const ReadCount rc = count_read(at[i], to[i], off0, r, n, len, check_ends != 0, k);
        const bool in = r < n;
        w[i] = in ? rc.windows : 0;
        const uint64_t kmers = in ? rc.kmers : 0;
        tw += w[i];
        tk += kmers;
        if (!COUNT) continue;
        bad |= in && rc.bad ? 1u << i : 0u;
        bare |= in && !rc.bad && !rc.windows ? 1u << i : 0u;
    }
    if (COUNT) {
        if (bad)
            for (uint32_t i = 0; i < kScanPerThread; ++i)
                if (bad >> i & 1) atomic_or_u32(&st[single ? 0u : instance_of_read(inst, m, r0 + 64 * i)].err, kErrInval);
        if (plan && bare)  // no tile covers these
            for (uint32_t i = 0; i < kScanPerThread; ++i)
                if (bare >> i & 1) {
                    bool good = true;
                    const uint64_t q0 = off[r0 + 64 * i] - off0, q1 = off[r0 + 64 * i + 1] - off0;
                    for (uint64_t q = q0; q < q1; q += 16)
#pragma unroll
                        for (uint32_t j = 0; j < 16; ++j) good &= valid_letter(ascii[min(q + j, q1 - 1)]);
                    if (!good) atomic_or_u32(&st[0].err, kErrBase);
                }
        bool one = true;  // the block's reads are of one instance
        if (!single) {
            if ((threadIdx.x & 63) == 0) s_inst[threadIdx.x >> 6] = uniform ? t0 : m;
            __syncthreads();
            for (uint32_t i = 0; i < kScanBlock / 64; ++i) one &= s_inst[i] == s_inst[0];
            one &= s_inst[0] < m;
        }
        if (!single && one) {
            const uint64_t bw = block_sum(tw, s_wave), bk = block_sum(tk, s_wave);
            if (threadIdx.x == 0 && bw) {
                atomic_add_u64(&st[t0].windows, bw);
                atomic_add_u64(&st[t0].inserts, bk);
            }
        }
        if (!one && uniform) {
            uint64_t sw = tw, sk = tk;
            for (int d = 32; d >= 1; d >>= 1) {
                sw += __shfl_xor(sw, d, 64);
                sk += __shfl_xor(sk, d, 64);
            }
            if ((threadIdx.x & 63) == 0 && sw) {
                atomic_add_u64(&st[t0].windows, sw);
                atomic_add_u64(&st[t0].inserts, sk);
            }
        }
        if (!uniform)  // the last lane of each instance in a row adds what the row has of it
            for (uint32_t i = 0; i < kScanPerThread; ++i) {
                const uint64_t r = r0 + 64 * i;
                const uint32_t t = r < n ? instance_of_read(inst, t0, t1 + 1, r) : m, lane = threadIdx.x & 63;
                ReadCount rc{0, 0, false};
                if (r < n) rc = count_read(off[r], off[r + 1], off0, r, n, len, check_ends != 0, inst[t].k);
                const uint64_t sw = wave_inclusive_scan(rc.windows), sk = wave_inclusive_scan(rc.kmers);
                const uint32_t next = __shfl_down(t, 1, 64);
                const uint64_t ends = __ballot(lane == 63 || next != t), lower = ends & ((1ull << lane) - 1);
                const int prev = lower ? 63 - __builtin_clzll(lower) : 0;
                const uint64_t pw = __shfl(sw, prev, 64), pk = __shfl(sk, prev, 64);
                if ((ends >> lane & 1) && t < m) {
                    atomic_add_u64(&st[t].windows, sw - (lower ? pw : 0));
                    atomic_add_u64(&st[t].inserts, sk - (lower ? pk : 0));
                }
            }
        if (WRITE && bad) __threadfence();  // the plan looks at the error bits
    }
    if (!WRITE) {
        const uint64_t total = min(block_sum(tw, s_wave), kMostOfBlock), ktotal = min(block_sum(tk, s_wave), kMostOfBlock);
        if (threadIdx.x == 0) {
            sums[2 * block] = total;
            sums[2 * block + 1] = ktotal;
        }
        return;
    }
    uint64_t total;
    uint64_t pre = block_exclusive_scan(tw, &total);
    pre = __shfl(pre, 0, 64) + before;  // before this wavefront's reads
    const bool narrow = !__any(tw >> 26);  // a row's sums fit 32 bits
    const uint32_t shift = tile & (tile - 1) ? 0u : (uint32_t)__builtin_ctz(tile);
#pragma unroll
    for (uint32_t i = 0; i < kScanPerThread; ++i) {
        const uint64_t r = r0 + 64 * i;
        const uint64_t inc = narrow ? wave_scan((uint32_t)w[i]) : wave_inclusive_scan(w[i]);
        const uint64_t a = pre + inc - w[i], z = pre + inc;
        pre += narrow ? (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)inc, 63) : __shfl(inc, 63, 64);
        if (r >= n) continue;
        ws[r] = a;
        if (r + 1 == n) ws[n] = z;
        // tiles whose first window falls inside this read start here
        if (tile_read && w[i])
            for (uint64_t tt = shift ? (a + tile - 1) >> shift : (a + tile - 1) / tile; tt * tile < z && tt < tile_cap; ++tt)
                tile_read[tt] = r;
    }
    if (!last_block) return;
    // the totals
    const uint64_t W = before + min(total, kMostOfBlock);
    uint64_t K = 0;
    if (single) K = kbefore + min(block_sum(tk, s_wave), kMostOfBlock);
    if (W > args->max_windows)
        for (uint32_t i = threadIdx.x; i < m; i += kScanBlock) atomic_or_u32(&st[i].err, kErrInval);
    if (threadIdx.x != 0) return;
    cs->windows = W > args->max_windows ? 0 : W;
    if (!single) return;
    st[0].windows = W;
    st[0].inserts = K;
    if (!plan) return;
    __threadfence();
    const Instance &in = inst[0];
    const uint32_t e = __hip_atomic_load(&st[0].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!(e & kErrRange) && in.prior_inserts + K > 0xffffffffull) atomic_or_u32(&st[0].err, kErrRange);
    SortPlan pl{};
    pl.w_end = W;
    pl.valid = !(e & (kErrInval | kErrSkip)) && W <= args->max_windows && in.parts;
    pl.tiles = pl.valid ? (W + tile - 1) / tile : 0;
    pl.groups = in.fan > 1 ? (pl.tiles + kSortGroup - 1) / kSortGroup : 0;
    *plan = pl;
    *tot = SortTotals{pl.tiles, in.fan > 1 ? in.d1 : 0u, pl.groups};
}

// ---------------------------------------------------------------- build

// Find the slot of `key` in the table, claiming an empty one if the key is
// absent (paper Algorithms 3 and 4 in open-addressing form).  A relaxed load
// first: a non-empty value is final, so most lookups of an existing vertex
// never issue an atomic.  An empty value (possibly stale) is resolved by the
// CAS, whose returned value says whether this lane claimed the slot, another
// lane claimed it for the same key, or another key took it.
//
// Returns kAllOnes when no empty slot lies within kMaxProbe slots of the home
// slot (or within the whole table when it is smaller), or when another lane
// has already reported this table full.  At the load factors the table is
// sized for (<= 0.9) linear-probing clusters stay orders of magnitude shorter
// than kMaxProbe, so this only fires on a table that is full in practice.
constexpr uint64_t kMaxProbe = 1ull << 16;

// Home slot of a key in the direct table: the mixed key's range reduction,
// or, with the test hash, the key's low 3 bits (cap >= 64), which sends
// every key of the table down the same probe chain.
__device__ __forceinline__ uint64_t direct_home(uint64_t key_bits, uint64_t h, uint64_t cap, uint32_t test_hash) {
    return test_hash ? (key_bits & 7u) : home_slot(h, cap);
}

template <bool STATS>
__device__ __forceinline__ uint64_t find_or_claim(uint64_t *table, uint32_t ew, uint64_t cap,
                                                  uint64_t key, uint64_t h, bool &claimed,
                                                  uint32_t *err, uint32_t test_hash, ProbeStats &ps) {
    const uint64_t tag = key | kOccupied;
    const uint64_t limit = cap < kMaxProbe ? cap : kMaxProbe;
    uint64_t s = direct_home(key, h, cap, test_hash);
    for (uint64_t probe = 0; probe < limit; ++probe) {
        uint64_t *kp = table + s * ew;
        const uint64_t cur = __hip_atomic_load(kp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == tag) {
            if (STATS) ps.lookup((uint32_t)min<uint64_t>(probe + 1, 0xffffffffu));
            return s;
        }
        if (cur == 0) {
            uint64_t expected = 0;
            const bool won = __hip_atomic_compare_exchange_strong(kp, &expected, tag, __ATOMIC_RELAXED,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (STATS) {
                ++ps.cas;
                ps.lost += won ? 0u : 1u;
            }
            if (won || expected == tag) {
                claimed = won;
                if (STATS) ps.lookup((uint32_t)min<uint64_t>(probe + 1, 0xffffffffu));
                return s;
            }
        }
        s = (s + 1 == cap) ? 0 : s + 1;
        if ((probe & 255) == 255 &&
            (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrFull))
            return kAllOnes;
    }
    return kAllOnes;
}

__device__ __forceinline__ void add_count(uint64_t *table, uint32_t ew, uint64_t s, uint32_t letter,
                                          uint32_t inc) {
    uint32_t *cnt = reinterpret_cast<uint32_t *>(table + s * ew + 1);
    __hip_atomic_fetch_add(cnt + letter, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr uint32_t kMergeSlots = 128;
constexpr uint32_t kMaxWaves = 16;

struct Window {
    uint64_t key;
    uint32_t letter;
    uint32_t inst;
    bool valid;  // a window of a read of an instance without errors
    bool sink;   // last window of its read: vertex only, no counter
};

// Instance of read r for a batched launch, with bit 31 set when its windows
// must be skipped: its input failed validation, its k-mer total would
// overflow a counter (every workgroup evaluates the same test, so the whole
// instance is skipped), or its table is already full.
__device__ __forceinline__ uint32_t instance_state(const Instance *inst, uint32_t m, InstStatus *st,
                                                   uint64_t r) {
    const uint32_t t = instance_of_read(inst, m, r);
    uint32_t e = __hip_atomic_load(&st[t].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!(e & kErrRange) && inst[t].prior_inserts + st[t].inserts > 0xffffffffull) {
        atomic_or_u32(&st[t].err, kErrRange);
        e |= kErrRange;
    }
    return (e & (kErrBase | kErrInval | kErrRange | kErrFull | kErrSkip)) ? (t | 0x80000000u) : t;
}

template <bool SINGLE, bool MERGE, bool STATS>
__global__ __launch_bounds__(1024) void k_build(const PassArgs *__restrict__ args,
                                               const Instance *__restrict__ inst,
                                               const uint64_t *__restrict__ packed,
                                               const uint64_t *__restrict__ ws,
                                               const uint64_t *__restrict__ tile_read,
                                               InstStatus *st, CallState *cs, uint32_t wpt) {
    const uint64_t *__restrict__ off = as_global(args->off);
    const uint64_t n = args->n_reads;
    const uint32_t m = args->m;
    __shared__ uint64_t s_ws[kMapReads + 1];
    __shared__ uint64_t s_delta[kMapReads];
    __shared__ uint32_t s_inst[kMapReads];  // instance index, bit 31 = skip
    __shared__ uint64_t s_tile;
    __shared__ uint64_t s_claims;
    __shared__ uint32_t s_slot[MERGE ? kMaxWaves * kMergeSlots : 1];
    __shared__ uint32_t s_cnt[MERGE ? kMaxWaves * 64 * 4 : 1];

    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t W = cs->windows;
    const uint64_t off0 = n ? off[0] : 0;
    const uint64_t T = (uint64_t)blockDim.x * wpt;
    const uint64_t ntiles = (W + T - 1) / T;

    // Single-graph launch: the graph's parameters stay in registers, and the
    // whole launch stops at once if validation failed or the k-mer count
    // would overflow a counter (every workgroup evaluates the same test).
    uint64_t *tab0 = nullptr;
    uint64_t cap0 = 0;
    uint32_t ew0 = 3, km1_0 = 0;
    if (SINGLE) {
        tab0 = as_global(inst[0].table);
        cap0 = inst[0].cap;
        ew0 = inst[0].entry_words;
        km1_0 = inst[0].k - 1;
        if (inst[0].prior_inserts + st[0].inserts > 0xffffffffull) {
            if (tid == 0) atomic_or_u32(&st[0].err, kErrRange);
            return;
        }
        if (__hip_atomic_load(&st[0].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
            (kErrBase | kErrInval | kErrRange | kErrSkip))
            return;
    }

    uint64_t my_claims = 0;  // SINGLE: flushed once at the end
    if (tid == 0) s_claims = 0;
    const uint32_t test_hash = args->test_hash;
    ProbeStats ps;

    for (;;) {
        if (tid == 0) {
            s_tile = __hip_atomic_fetch_add(&cs->cursor, 1ull, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
            // a full single table stops the whole launch
            if (SINGLE && (__hip_atomic_load(&st[0].err, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT) & kErrFull))
                s_tile = ntiles;
        }
        __syncthreads();
        const uint64_t tile = s_tile;
        if (tile >= ntiles) break;
        const uint64_t w0 = tile * T;
        const uint64_t w1 = min(w0 + T, W);
        const uint64_t r0 = tile_read[tile];
        const uint32_t R = (uint32_t)min((uint64_t)kMapReads, n - r0);

        // Stage the tile's reads: window prefix, base offset, instance.
        for (uint32_t i = tid; i <= R; i += blockDim.x) {
            const uint64_t r = r0 + i;
            const uint64_t wr = ws[r];
            s_ws[i] = wr;
            if (i < R) {
                s_delta[i] = off[r] - off0 - wr;
                s_inst[i] = SINGLE ? 0u : instance_state(inst, m, st, r);
            }
        }
        __syncthreads();

        uint32_t tile_inst0 = s_inst[0] & 0x7fffffffu;
        uint64_t tile_claims = 0;

        for (uint32_t it = 0; it < wpt; ++it) {
            const uint64_t w = w0 + (uint64_t)it * blockDim.x + tid;
            Window win{0, 0, 0, false, false};
            if (w < w1) {
                uint64_t wr, wr1, delta;
                uint32_t tinfo;
                if (w < s_ws[R]) {
                    uint32_t lo = 0, hi = R;  // s_ws[lo] <= w < s_ws[hi]
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (s_ws[mid] <= w) lo = mid; else hi = mid;
                    }
                    wr = s_ws[lo];
                    wr1 = s_ws[lo + 1];
                    delta = s_delta[lo];
                    tinfo = s_inst[lo];
                } else {
                    // The tile spans more reads than were staged.
                    uint64_t lo = r0 + R, hi = n;  // ws[lo] <= w < ws[hi]
                    while (hi - lo > 1) {
                        const uint64_t mid = (lo + hi) >> 1;
                        if (ws[mid] <= w) lo = mid; else hi = mid;
                    }
                    wr = ws[lo];
                    wr1 = ws[lo + 1];
                    delta = off[lo] - off0 - wr;
                    tinfo = SINGLE ? 0u : instance_state(inst, m, st, lo);
                }
                (void)wr;
                win.valid = (tinfo & 0x80000000u) == 0;
                win.inst = tinfo & 0x7fffffffu;
                win.sink = (w + 1 == wr1);
                if (win.valid) {
                    const uint32_t km1 = SINGLE ? km1_0 : inst[win.inst].k - 1;
                    const uint64_t b = bases_at(packed, w + delta);
                    win.key = b >> (64 - 2 * km1);
                    win.letter = (uint32_t)(b >> (62 - 2 * km1)) & 3u;
                }
            }
            uint64_t *tab = tab0;
            uint64_t cap = cap0;
            uint32_t ew = ew0;
            if (!SINGLE && win.valid) {
                tab = as_global(inst[win.inst].table);
                cap = inst[win.inst].cap;
                ew = inst[win.inst].entry_words;
            }
            const uint64_t h = mix64(win.key);

            uint32_t inc[4] = {0, 0, 0, 0};
            bool leader = win.valid;
            if (MERGE) {
                // Merge equal vertices of this wavefront: every lane writes
                // its lane id into a slot chosen by the key; the lane whose
                // id survives leads all lanes with the same key, which add
                // their letters into the leader's LDS counters.  A key whose
                // slot another key won simply stays on its own.
                uint32_t *slot = s_slot + wave * kMergeSlots;
                uint32_t *cnt = s_cnt + wave * 256;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    __hip_atomic_store(cnt + lane * 4 + c, 0u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
                const uint32_t sl = (uint32_t)h & (kMergeSlots - 1);
                if (win.valid)
                    __hip_atomic_store(slot + sl, lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                uint32_t winner = lane;
                if (win.valid)
                    winner = __hip_atomic_load(slot + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                const uint64_t wkey = __shfl(win.key, (int)winner, 64);
                const uint32_t winst = __shfl(win.inst, (int)winner, 64);
                const uint32_t lead = (win.valid && wkey == win.key && winst == win.inst) ? winner : lane;
                if (win.valid && !win.sink)
                    __hip_atomic_fetch_add(cnt + lead * 4 + win.letter, 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WAVEFRONT);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                leader = win.valid && lead == lane;
                if (leader) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        inc[c] = __hip_atomic_load(cnt + lane * 4 + c, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WAVEFRONT);
                }
            } else if (win.valid && !win.sink) {
                inc[win.letter] = 1;
            }

            if (leader) {
                bool claimed = false;
                const uint64_t s =
                    find_or_claim<STATS>(tab, ew, cap, win.key, h, claimed, &st[win.inst].err, test_hash, ps);
                if (s == kAllOnes) {
                    atomic_or_u32(&st[win.inst].err, kErrFull);
                } else {
                    if (MERGE) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (inc[c]) add_count(tab, ew, s, (uint32_t)c, inc[c]);
                    } else if (!win.sink) {
                        add_count(tab, ew, s, win.letter, 1u);
                    }
                    if (claimed) {
                        if (SINGLE) {
                            ++my_claims;
                        } else {
                            ++tile_claims;
                            if (win.inst != tile_inst0) {
                                // rare: tile crosses into another graph
                                atomic_add_u64(&st[win.inst].claimed, 1);
                                --tile_claims;
                            }
                        }
                    }
                }
            }
        }
        if (!SINGLE) {
            // claims of the tile's first graph: one atomic per workgroup
            for (int d = 32; d >= 1; d >>= 1) tile_claims += __shfl_xor(tile_claims, d, 64);
            if (lane == 0 && tile_claims)
                __hip_atomic_fetch_add(&s_claims, tile_claims, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            __syncthreads();
            if (tid == 0 && s_claims) {
                atomic_add_u64(&st[tile_inst0].claimed, s_claims);
                s_claims = 0;
            }
        }
        __syncthreads();
    }
    if (STATS) ps.flush(args->stats);
    if (SINGLE) {
        for (int d = 32; d >= 1; d >>= 1) my_claims += __shfl_xor(my_claims, d, 64);
        if (lane == 0 && my_claims)
            __hip_atomic_fetch_add(&s_claims, my_claims, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        if (tid == 0 && s_claims) atomic_add_u64(&st[0].claimed, s_claims);
    }
}

// ---------------------------------------------------------------- build, long k

// For 32 < k <= 64 the (k-1)-mer K has 64 to 126 bits and takes two words of
// a 32-byte entry: word 0 = kOccupied | K >> 63, word 1 = kWritten | (K mod
// 2^63), then the four counters.  A slot is claimed by the CAS of word 0
// alone; the claimer then stores word 1 once.  A lane that finds word 0
// equal to its own but word 1 still zero has met a claim in flight and reads
// the slot again (the claimer waits for nothing between its CAS and that
// store, so the wait ends); a word 1 of another key sends it on to the next
// slot.  Words are written once each, so no ordering between the two words
// is needed beyond each word's own atomicity.
constexpr uint64_t kWritten = 1ull << 63;
constexpr uint64_t kLow63 = kWritten - 1;
constexpr uint32_t kMaxInFlight = 1u << 20;  // re-reads of one claim in flight

template <bool STATS>
__device__ __forceinline__ uint64_t find_or_claim_wide(uint64_t *table, uint64_t cap, uint64_t tag0,
                                                       uint64_t tag1, uint64_t h, bool &claimed,
                                                       uint32_t *err, uint32_t test_hash, ProbeStats &ps) {
    const uint64_t limit = cap < kMaxProbe ? cap : kMaxProbe;
    uint64_t s = direct_home(tag1, h, cap, test_hash);
    uint64_t probes = 0;
    uint32_t waits = 0;
    for (;;) {
        uint64_t *e = table + s * 4;
        uint64_t cur = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == 0) {
            uint64_t expected = 0;
            const bool won = __hip_atomic_compare_exchange_strong(e, &expected, tag0, __ATOMIC_RELAXED,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (STATS) {
                ++ps.cas;
                ps.lost += won ? 0u : 1u;
            }
            if (won) {
                __hip_atomic_store(e + 1, tag1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                claimed = true;
                if (STATS) ps.lookup((uint32_t)min<uint64_t>(probes + 1, 0xffffffffu));
                return s;
            }
            cur = expected;
        }
        if (cur == tag0) {
            const uint64_t w1 = __hip_atomic_load(e + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (w1 == tag1) {
                if (STATS) ps.lookup((uint32_t)min<uint64_t>(probes + 1, 0xffffffffu));
                return s;
            }
            if (w1 == 0) {  // a claim in flight: read this slot again
                if (++waits > kMaxInFlight) return kAllOnes;
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
        }
        if (++probes >= limit) return kAllOnes;
        s = (s + 1 == cap) ? 0 : s + 1;
        if ((probes & 255) == 255 &&
            (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrFull))
            return kAllOnes;
    }
}

// Plain (one-graph) build for 32 < k <= 64; same tiles and window map as
// k_build, one window per thread per step, no merging.
template <bool STATS>
__global__ __launch_bounds__(1024) void k_build_wide(const PassArgs *__restrict__ args,
                                                    const Instance *__restrict__ inst,
                                                    const uint64_t *__restrict__ packed,
                                                    const uint64_t *__restrict__ ws,
                                                    const uint64_t *__restrict__ tile_read,
                                                    InstStatus *st, CallState *cs, uint32_t wpt) {
    const uint64_t *__restrict__ off = as_global(args->off);
    const uint64_t n = args->n_reads;
    __shared__ uint64_t s_ws[kMapReads + 1];
    __shared__ uint64_t s_delta[kMapReads];
    __shared__ uint64_t s_tile;
    __shared__ uint64_t s_claims;

    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint64_t W = cs->windows;
    const uint64_t off0 = n ? off[0] : 0;
    const uint64_t T = (uint64_t)blockDim.x * wpt;
    const uint64_t ntiles = (W + T - 1) / T;
    uint64_t *tab = as_global(inst[0].table);
    const uint64_t cap = inst[0].cap;
    const uint32_t km1 = inst[0].k - 1;
    if (inst[0].prior_inserts + st[0].inserts > 0xffffffffull) {
        if (tid == 0) atomic_or_u32(&st[0].err, kErrRange);
        return;
    }
    if (__hip_atomic_load(&st[0].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
        (kErrBase | kErrInval | kErrRange | kErrSkip))
        return;

    uint64_t my_claims = 0;
    if (tid == 0) s_claims = 0;
    const uint32_t test_hash = args->test_hash;
    ProbeStats ps;
    for (;;) {
        if (tid == 0) {
            s_tile = __hip_atomic_fetch_add(&cs->cursor, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__hip_atomic_load(&st[0].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrFull)
                s_tile = ntiles;
        }
        __syncthreads();
        const uint64_t tile = s_tile;
        if (tile >= ntiles) break;
        const uint64_t w0 = tile * T;
        const uint64_t w1 = min(w0 + T, W);
        const uint64_t r0 = tile_read[tile];
        const uint32_t R = (uint32_t)min((uint64_t)kMapReads, n - r0);
        for (uint32_t i = tid; i <= R; i += blockDim.x) {
            const uint64_t rr = r0 + i;
            const uint64_t wr = ws[rr];
            s_ws[i] = wr;
            if (i < R) s_delta[i] = off[rr] - off0 - wr;
        }
        __syncthreads();

        for (uint32_t it = 0; it < wpt; ++it) {
            const uint64_t w = w0 + (uint64_t)it * blockDim.x + tid;
            if (w >= w1) continue;
            uint64_t wr1, delta;
            if (w < s_ws[R]) {
                uint32_t lo = 0, hi = R;  // s_ws[lo] <= w < s_ws[hi]
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_ws[mid] <= w) lo = mid; else hi = mid;
                }
                wr1 = s_ws[lo + 1];
                delta = s_delta[lo];
            } else {
                uint64_t lo = r0 + R, hi = n;  // ws[lo] <= w < ws[hi]
                while (hi - lo > 1) {
                    const uint64_t mid = (lo + hi) >> 1;
                    if (ws[mid] <= w) lo = mid; else hi = mid;
                }
                wr1 = ws[lo + 1];
                delta = off[lo] - off0 - ws[lo];
            }
            const bool sink = (w + 1 == wr1);
            uint64_t x0, x1, khi, klo;
            uint32_t letter;
            bases128_at(packed, w + delta, x0, x1);
            wide_window(x0, x1, km1, khi, klo, letter);
            const uint64_t a = (khi << 1) | (klo >> 63);
            const uint64_t tag0 = a | kOccupied, tag1 = (klo & kLow63) | kWritten;
            const uint64_t h = mix64(tag1 ^ mix64(a));
            bool claimed = false;
            const uint64_t s = find_or_claim_wide<STATS>(tab, cap, tag0, tag1, h, claimed, &st[0].err, test_hash, ps);
            if (s == kAllOnes) {
                atomic_or_u32(&st[0].err, kErrFull);
                continue;
            }
            if (!sink)
                __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(tab + s * 4 + 2) + letter, 1u,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            my_claims += claimed ? 1u : 0u;
        }
        __syncthreads();
    }
    if (STATS) ps.flush(args->stats);
    for (int d = 32; d >= 1; d >>= 1) my_claims += __shfl_xor(my_claims, d, 64);
    if (lane == 0 && my_claims)
        __hip_atomic_fetch_add(&s_claims, my_claims, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (tid == 0 && s_claims) atomic_add_u64(&st[0].claimed, s_claims);
}

// ---------------------------------------------------------------- extract

constexpr uint32_t kExtractBlock = 256;
constexpr uint32_t kExtractPerThread = 4;

// Compact occupied slots into (key, counts) records; one atomic per block
// reserves the output range.  Record order is unspecified.
template <bool WRITE>
__global__ __launch_bounds__(kExtractBlock) void k_extract(const uint64_t *__restrict__ table,
                                                          uint32_t ew, uint64_t cap,
                                                          uint64_t *__restrict__ okeys,
                                                          uint32_t *__restrict__ ocnt,
                                                          uint64_t ocap, uint64_t *out_n) {
    __shared__ uint64_t s_base;
    const uint64_t chunk = (uint64_t)kExtractBlock * kExtractPerThread;
    for (uint64_t base = (uint64_t)blockIdx.x * chunk; base < cap; base += (uint64_t)gridDim.x * chunk) {
        uint64_t tags[kExtractPerThread];
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t i = 0; i < kExtractPerThread; ++i) {
            const uint64_t s = base + (uint64_t)i * kExtractBlock + threadIdx.x;
            tags[i] = s < cap ? table[s * ew] : 0;
            mine += tags[i] != 0;
        }
        uint64_t total;
        uint64_t pre = block_exclusive_scan(mine, &total);
        if (threadIdx.x == 0) s_base = total ? atomicAdd((unsigned long long *)out_n, (unsigned long long)total) : 0;
        __syncthreads();
        if (WRITE) {
            uint64_t idx = s_base + pre;
#pragma unroll
            for (uint32_t i = 0; i < kExtractPerThread; ++i) {
                if (!tags[i]) continue;
                const uint64_t s = base + (uint64_t)i * kExtractBlock + threadIdx.x;
                if (idx < ocap) {
                    okeys[idx] = tags[i] & ~kOccupied;
                    const uint32_t *c = reinterpret_cast<const uint32_t *>(table + s * ew + 1);
                    uint4 v = make_uint4(c[0], c[1], c[2], c[3]);
                    *reinterpret_cast<uint4 *>(ocnt + 4 * idx) = v;
                }
                ++idx;
            }
        }
        __syncthreads();
    }
}

// Long-k table: each record's key as two words (K >> 64, K mod 2^64).
__global__ __launch_bounds__(kExtractBlock) void k_extract_wide(const uint64_t *__restrict__ table,
                                                               uint64_t cap, uint64_t *__restrict__ okeys,
                                                               uint32_t *__restrict__ ocnt, uint64_t ocap,
                                                               uint64_t *out_n) {
    __shared__ uint64_t s_base;
    const uint64_t chunk = (uint64_t)kExtractBlock * kExtractPerThread;
    for (uint64_t base = (uint64_t)blockIdx.x * chunk; base < cap; base += (uint64_t)gridDim.x * chunk) {
        uint64_t tags[kExtractPerThread];
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t i = 0; i < kExtractPerThread; ++i) {
            const uint64_t s = base + (uint64_t)i * kExtractBlock + threadIdx.x;
            tags[i] = s < cap ? table[s * 4] : 0;
            mine += tags[i] != 0;
        }
        uint64_t total;
        uint64_t pre = block_exclusive_scan(mine, &total);
        if (threadIdx.x == 0) s_base = total ? atomicAdd((unsigned long long *)out_n, (unsigned long long)total) : 0;
        __syncthreads();
        uint64_t idx = s_base + pre;
#pragma unroll
        for (uint32_t i = 0; i < kExtractPerThread; ++i) {
            if (!tags[i]) continue;
            const uint64_t s = base + (uint64_t)i * kExtractBlock + threadIdx.x;
            if (idx < ocap) {
                const ulonglong2 e = *reinterpret_cast<const ulonglong2 *>(table + s * 4);
                const uint4 c = *reinterpret_cast<const uint4 *>(table + s * 4 + 2);
                const uint64_t a = e.x & ~kOccupied, b = e.y & kLow63;
                okeys[2 * idx] = a >> 1;
                okeys[2 * idx + 1] = (a << 63) | b;
                *reinterpret_cast<uint4 *>(ocnt + 4 * idx) = c;
            }
            ++idx;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- roofline

// Random-access microbenchmark over `words` uint64 words: indices come from
// mix64 of the operation number, so no index array is read.
__global__ __launch_bounds__(1024) void k_roofline(uint64_t *mem, uint64_t words, uint64_t n_ops,
                                                  uint32_t kind, uint64_t seed, uint64_t *sink) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t acc = 0;
    const uint64_t entries = words / 3;
    for (uint64_t op = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; op < n_ops; op += stride) {
        const uint64_t h = mix64(seed + op);
        if (kind == 0) {
            acc += __hip_atomic_load(mem + home_slot(h, words), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        } else if (kind == 1) {
            uint32_t *m32 = reinterpret_cast<uint32_t *>(mem);
            __hip_atomic_fetch_add(m32 + home_slot(h, words * 2), 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        } else if (kind == 2) {
            uint64_t expected = 0;
            __hip_atomic_compare_exchange_strong(mem + home_slot(h, words), &expected, h | 1,
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            acc += expected;
        } else {
            uint64_t *e = mem + home_slot(h, entries) * 3;
            const uint64_t k = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t *c = reinterpret_cast<uint32_t *>(e + 1);
            __hip_atomic_fetch_add(c + (k & 3), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (acc == 0x5eed5eed5eed5eedull) sink[0] = acc;
}

// Streaming copy of the first half of mem onto the second, 16 bytes per
// load and store: a plain copy of known size for scaling traffic counters.
__global__ __launch_bounds__(1024) void k_stream_copy(uint64_t *mem, uint64_t words) {
    const uint64_t half = (words / 2) & ~1ull;
    const ulonglong2 *src = reinterpret_cast<const ulonglong2 *>(mem);
    ulonglong2 *dst = reinterpret_cast<ulonglong2 *>(mem + half);
    const uint64_t n = half / 2, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

template <typename K>
uint32_t grid_for(K kernel, int device, uint32_t block) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        cus <= 0)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, (int)block, 0) != hipSuccess ||
        per <= 0)
        per = 1;
    return (uint32_t)(cus * per);
}

}  // namespace

// ---------------------------------------------------------------- launchers

hipError_t launch_begin(const void *host, PassArgs *args, Instance *inst, InstStatus *st, CallState *cs,
                        uint64_t *done, uint32_t m_cap, hipStream_t s) {
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(((uint64_t)m_cap * kInstWords + 255) / 256, 64);
    hipLaunchKernelGGL(k_begin, dim3(blocks), dim3(256), 0, s, static_cast<const uint64_t *>(host), args, inst, st, cs,
                       done, done ? kDoneWords : 0u);
    return hipGetLastError();
}

hipError_t launch_store_words(const uint64_t *from, uint64_t *to, uint64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_store_words, dim3((uint32_t)std::min<uint64_t>((n + 255) / 256, 256)), dim3(256), 0, s, from, to, n);
    return hipGetLastError();
}

hipError_t launch_gather_u64(const uint64_t *src, const uint64_t *idx, uint64_t n, uint64_t *out, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_gather_u64, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, src, idx, n, out);
    return hipGetLastError();
}

hipError_t launch_fill_zero(uint64_t *words, uint64_t n_words, hipStream_t s) {
    if (!n_words) return hipSuccess;
    const uint64_t pairs = (n_words + 1) / 2;
    const uint64_t want = (pairs + 255) / 256;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(want, 256 * 64);
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, s, words, n_words);
    return hipGetLastError();
}

hipError_t launch_pack(const PassArgs *args, uint64_t *packed, const Instance *inst, InstStatus *st,
                       uint64_t len_cap, hipStream_t s) {
    const uint64_t n_words = packed_words(len_cap);
    const uint64_t want = (n_words + 255) / 256;
    const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(want, 256 * 64));
    hipLaunchKernelGGL(k_pack, dim3(blocks), dim3(256), 0, s, args, packed, inst, st);
    return hipGetLastError();
}

hipError_t launch_scan(const PassArgs *args, const Instance *inst, InstStatus *st, uint64_t *ws, uint64_t *sums,
                       uint64_t *tile_read, CallState *cs, SortPlan *plan, SortTotals *tot, uint64_t n_cap,
                       hipStream_t s) {
    const dim3 g((uint32_t)std::max<uint64_t>(1, scan_blocks(n_cap))), b(kScanBlock);
    if (g.x == 1) {
        hipLaunchKernelGGL((k_scan<true, true>), g, b, 0, s, args, inst, st, ws, sums, tile_read, cs, plan, tot);
    } else {
        hipLaunchKernelGGL((k_scan<true, false>), g, b, 0, s, args, inst, st, ws, sums, tile_read, cs, plan, tot);
        hipLaunchKernelGGL((k_scan<false, true>), g, b, 0, s, args, inst, st, ws, sums, tile_read, cs, plan, tot);
    }
    return hipGetLastError();
}

hipError_t launch_build(const PassArgs *args, const Instance *inst, const uint64_t *packed,
                        const uint64_t *ws, const uint64_t *tile_read, InstStatus *st, CallState *cs,
                        BuildShape shape, bool single, bool stats, hipStream_t s) {
    const dim3 g(shape.grid), b(shape.block);
#define DBG_LAUNCH_BUILD(SINGLE, MERGE, STATS)                                                                    \
    hipLaunchKernelGGL((k_build<SINGLE, MERGE, STATS>), g, b, 0, s, args, inst, packed, ws, tile_read, st, cs, \
                       shape.wpt)
    if (stats) {
        if (single) {
            if (shape.merge) DBG_LAUNCH_BUILD(true, true, true); else DBG_LAUNCH_BUILD(true, false, true);
        } else {
            if (shape.merge) DBG_LAUNCH_BUILD(false, true, true); else DBG_LAUNCH_BUILD(false, false, true);
        }
    } else {
        if (single) {
            if (shape.merge) DBG_LAUNCH_BUILD(true, true, false); else DBG_LAUNCH_BUILD(true, false, false);
        } else {
            if (shape.merge) DBG_LAUNCH_BUILD(false, true, false); else DBG_LAUNCH_BUILD(false, false, false);
        }
    }
#undef DBG_LAUNCH_BUILD
    return hipGetLastError();
}

hipError_t launch_build_wide(const PassArgs *args, const Instance *inst, const uint64_t *packed,
                             const uint64_t *ws, const uint64_t *tile_read, InstStatus *st, CallState *cs,
                             BuildShape shape, bool stats, hipStream_t s) {
    if (stats)
        hipLaunchKernelGGL(k_build_wide<true>, dim3(shape.grid), dim3(shape.block), 0, s, args, inst, packed, ws,
                           tile_read, st, cs, shape.wpt);
    else
        hipLaunchKernelGGL(k_build_wide<false>, dim3(shape.grid), dim3(shape.block), 0, s, args, inst, packed, ws,
                           tile_read, st, cs, shape.wpt);
    return hipGetLastError();
}

namespace {

// round-half-up(c * genome / total) = floor((2 c genome + total) / (2 total)),
// exactly: the 128-bit numerator is divided 16 bits at a time (the divisor
// 2 total is below 2^34, so a partial remainder shifted by 16 stays below
// 2^50); saturated at 2^32 - 1.
__device__ __forceinline__ uint32_t normalized(uint32_t c, uint64_t genome, uint64_t total) {
    if (!genome || !total) return c;
    uint64_t lo = (uint64_t)c * genome;
    uint64_t hi = __umul64hi((uint64_t)c, genome);
    hi = (hi << 1) | (lo >> 63);
    lo <<= 1;
    const uint64_t lo2 = lo + total;
    hi += lo2 < lo ? 1u : 0u;
    lo = lo2;
    const uint64_t d = 2 * total;
    uint64_t q = 0, r = 0;
    for (int i = 7; i >= 0; --i) {
        const uint64_t limb = (i >= 4 ? hi >> (16 * (i - 4)) : lo >> (16 * i)) & 0xffffu;
        const uint64_t cur = (r << 16) | limb;
        const uint64_t qd = cur / d;
        r = cur - qd * d;
        if (q >> 48) return 0xffffffffu;
        q = (q << 16) | qd;
    }
    return q > 0xffffffffull ? 0xffffffffu : (uint32_t)q;
}

__global__ __launch_bounds__(256) void k_normalize(uint32_t *counts, uint64_t n, uint64_t genome, uint64_t total,
                                                   uint8_t *out8) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t v = normalized(counts[i], genome, total);
        if (out8) out8[i] = (uint8_t)(v > 255u ? 255u : v);
        else counts[i] = v;
    }
}

}  // namespace

hipError_t launch_normalize(uint32_t *counts, uint64_t n, uint64_t genome, uint64_t total, uint8_t *out8,
                            hipStream_t s) {
    if (!n) return hipSuccess;
    const uint32_t g = (uint32_t)std::min<uint64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_normalize, dim3(g), dim3(256), 0, s, counts, n, genome, total, out8);
    return hipGetLastError();
}

hipError_t launch_extract(const uint64_t *table, uint32_t ew, uint64_t cap, uint64_t *okeys,
                          uint32_t *ocnt, uint64_t ocap, uint64_t *out_n, hipStream_t s) {
    const uint64_t chunk = (uint64_t)kExtractBlock * kExtractPerThread;
    const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((cap + chunk - 1) / chunk, 256 * 32));
    hipLaunchKernelGGL((k_extract<true>), dim3(blocks), dim3(kExtractBlock), 0, s, table, ew, cap,
                       okeys, ocnt, ocap, out_n);
    return hipGetLastError();
}

hipError_t launch_extract_wide(const uint64_t *table, uint64_t cap, uint64_t *okeys, uint32_t *ocnt,
                               uint64_t ocap, uint64_t *out_n, hipStream_t s) {
    const uint64_t chunk = (uint64_t)kExtractBlock * kExtractPerThread;
    const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((cap + chunk - 1) / chunk, 256 * 32));
    hipLaunchKernelGGL(k_extract_wide, dim3(blocks), dim3(kExtractBlock), 0, s, table, cap, okeys, ocnt, ocap,
                       out_n);
    return hipGetLastError();
}

hipError_t launch_count(const uint64_t *table, uint32_t ew, uint64_t cap, uint64_t *out_n,
                        hipStream_t s) {
    const uint64_t chunk = (uint64_t)kExtractBlock * kExtractPerThread;
    const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((cap + chunk - 1) / chunk, 256 * 32));
    hipLaunchKernelGGL((k_extract<false>), dim3(blocks), dim3(kExtractBlock), 0, s, table, ew, cap,
                       nullptr, nullptr, 0, out_n);
    return hipGetLastError();
}

hipError_t launch_roofline(uint64_t *mem, uint64_t words, uint64_t n_ops, uint32_t kind, uint64_t seed,
                           uint32_t block, uint64_t *sink, hipStream_t s) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    if (kind == 4) {
        const uint32_t grid = grid_for(k_stream_copy, dev, block);
        hipLaunchKernelGGL(k_stream_copy, dim3(grid), dim3(block), 0, s, mem, words);
        return hipGetLastError();
    }
    const uint32_t grid = grid_for(k_roofline, dev, block);
    hipLaunchKernelGGL(k_roofline, dim3(grid), dim3(block), 0, s, mem, words, n_ops, kind, seed, sink);
    return hipGetLastError();
}

uint32_t build_grid_wide(int device, uint32_t block) { return grid_for(k_build_wide<false>, device, block); }

uint32_t build_grid(int device, uint32_t block) {
    // the instantiations share the same resource shape up to LDS; the
    // merging one uses the most LDS and registers, so size from it (the
    // statistics kernels may fit fewer workgroups: tiles come from a cursor,
    // so extra workgroups simply start later)
    return grid_for(k_build<false, true, false>, device, block);
}

}  // namespace dbgk
