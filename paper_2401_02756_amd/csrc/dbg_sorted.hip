// The binned build's partition by sorted tiles (automatic scatter shapes).
//
// Records reach their table segment without any count pass: a workgroup sorts
// a tile of records by digit in LDS and stores the whole tile as it lies
// there, one contiguous run, beside a row of 16-bit offsets (where each digit
// starts in the tile).  Whoever needs the records of one digit gathers that
// digit's pieces, one per tile.
//
//   k_sort_windows  reads -> tiles of window records, sorted by level-1
//                   bucket.  The tile's bases are packed from ASCII into LDS
//                   here (and checked), so no packed copy of the reads exists.
//   k_sort_bucket   the pieces of one bucket -> tiles sorted by the bucket's
//                   segments (tables of up to kSingleParts segments skip this:
//                   their buckets are segments)
//   k_reduce_pieces the pieces of each segment -> claims and counts in LDS ->
//                   the table (and the caller's arrays)
//
// Against one histogram per chunk, flat scans and scattered runs (dbg_binned.hip)
// the records are read once less per level, every record line is stored
// whole, and a single-level build is two kernels after the window scan.
// Measured, a reset and a fused build and extraction (ms): 13.3 M reads of
// 150 bases, k = 31, 504 M vertices 30.2 -> 21.6; 1 M reads of 150 bases,
// 36 M vertices 2.05 -> 1.61 (k = 51: 3.85 -> 2.97); 1.7 M reads of 15-75 bases
// 1.50 -> 0.68; 40 k reads of 100 bases 0.168 -> 0.109.  By kernel at the
// largest: windows 10.2 -> 6.0 (with the packing and the count), level 2
// 11.2 -> 5.7, reduce 9.2 -> 10.2: a piece of 23 records covers 2.4 lines
// where it fills 1.4, so the reduce and level 2 read almost twice the records'
// bytes, at 4.9 and 5.4 TB/s.
#include "dbg_records.h"

#include <algorithm>

namespace dbgk {
namespace {

// ---------------------------------------------------------------- scans

// Exclusive scan over the block, one barrier; s_w[BLOCK / 64] is free again
// after the caller's next barrier.
template <uint32_t BLOCK>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *s_w, uint32_t *total) {
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t inc = wave_scan(v);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    const uint32_t x = lane < BLOCK / 64 ? s_w[lane] : 0u, waves = wave_scan(x);
    *total = __builtin_amdgcn_readlane(waves, 63);
    return __builtin_amdgcn_readlane(waves - x, wave) + inc - v;
}

// ---------------------------------------------------------------- tiles

// A tile: BLOCK threads, PER records each.  Tags are digit << RB | rank.
constexpr uint32_t log2_of(uint32_t x) { return x <= 1 ? 0 : 1 + log2_of(x / 2); }

template <uint32_t BLOCK, uint32_t PER>
struct Tile {
    static constexpr uint32_t n = BLOCK * PER, rb = log2_of(n);
    static_assert((1u << rb) == n && n <= 32768, "a tile's offsets fit 16 bits");
};

// After the tagged counts (s_cnt[j] = (j << RB) + count of digit j): s_cnt[j]
// becomes digit j's start in the sorted tile, and row[0 .. digits] the tile's
// offsets (row[digits] = n).  Whole block; a barrier inside, none after.
template <uint32_t BLOCK, uint32_t RB>
__device__ __forceinline__ void digit_starts(uint32_t *s_cnt, uint32_t digits, uint32_t n, uint32_t *s_w,
                                             uint16_t *__restrict__ row) {
    const uint32_t per = (digits + BLOCK - 1) / BLOCK;
    const uint32_t j0 = threadIdx.x * per;
    uint32_t sum = 0;
    for (uint32_t q = 0; q < per; ++q)
        if (j0 + q < digits) sum += s_cnt[j0 + q] - ((j0 + q) << RB);
    uint32_t total;
    uint32_t pre = block_scan<BLOCK>(sum, s_w, &total);
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t j = j0 + q;
        if (j < digits) {
            const uint32_t c = s_cnt[j] - (j << RB);
            s_cnt[j] = pre;
            row[j] = (uint16_t)pre;
            pre += c;
        }
    }
    if (threadIdx.x == 0) row[digits] = (uint16_t)n;
}

// The room a tile's records take in LDS while they are put in order: all of
// them, or (WORDS) one 32-bit word of each at a time, so that a tile of twice
// the records fits, or two workgroups a CU.
__host__ __device__ constexpr uint32_t tile_room(uint32_t tile, uint32_t rw, bool words) {
    return (words ? 4u : 8u * rw) * tile;
}

// Put the thread's tagged records in order and store the tile.
template <uint32_t BLOCK, uint32_t PER, uint32_t RB, bool WORDS, typename R>
__device__ __forceinline__ void place_and_store(R (&rec)[PER], uint32_t (&tag)[PER], const uint32_t *s_cnt,
                                                uint32_t digits, void *s_room, uint32_t n, R *__restrict__ out) {
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {  // tags become places
        const uint32_t d = tag[q] >> RB;
        tag[q] = d != digits ? s_cnt[d] + (tag[q] & ((1u << RB) - 1)) : ~0u;
    }
    if constexpr (!WORDS) {
        R *s_rec = reinterpret_cast<R *>(s_room);
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q)
            if (tag[q] != ~0u) s_rec[tag[q]] = rec[q];
        __syncthreads();
        const ulonglong2 *src = reinterpret_cast<const ulonglong2 *>(s_rec);
        ulonglong2 *dst = reinterpret_cast<ulonglong2 *>(out);
        const uint32_t pairs = (n * (uint32_t)(sizeof(R) / 8) + 1) / 2;
        for (uint32_t j = threadIdx.x; j < pairs; j += BLOCK) dst[j] = src[j];
    } else {
        // word by word through LDS; a thread takes each word of two records in a row (one of 16 bytes)
        constexpr uint32_t W = sizeof(R) / 4, EACH = 4 / W;
        uint32_t *s_word = reinterpret_cast<uint32_t *>(s_room);
        uint4 res[PER / EACH];
#pragma unroll
        for (uint32_t w = 0; w < W; ++w) {
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q)
                if (tag[q] != ~0u) {
                    uint64_t v;
                    if constexpr (W == 2) v = rec[q];
                    else v = w < 2 ? rec[q].x : rec[q].y;
                    s_word[tag[q]] = (uint32_t)(w & 1 ? v >> 32 : v);
                }
            __syncthreads();
#pragma unroll
            for (uint32_t o = 0; o < PER / EACH; ++o) {
                const uint32_t at = (o * BLOCK + threadIdx.x) * EACH;
                if constexpr (EACH == 2) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(s_word + at);
                    if (w == 0) res[o].x = v.x, res[o].z = v.y;
                    else res[o].y = v.x, res[o].w = v.y;
                } else {
                    const uint32_t v = s_word[at];
                    if (w == 0) res[o].x = v;
                    else if (w == 1) res[o].y = v;
                    else if (w == 2) res[o].z = v;
                    else res[o].w = v;
                }
            }
            if (w + 1 < W) __syncthreads();
        }
#pragma unroll
        for (uint32_t o = 0; o < PER / EACH; ++o) {
            const uint32_t at = (o * BLOCK + threadIdx.x) * EACH;
            if (at < n) *reinterpret_cast<uint4 *>(out + at) = res[o];
        }
    }
}

// ---------------------------------------------------------------- plan

// Per instance: its windows and tiles, and, when its segments need a second
// level, the bases of its transposed offsets, groups and buckets.  One block.
__global__ __launch_bounds__(1024) void k_sort_plan(const PassArgs *__restrict__ args, const Instance *inst,
                                                    const uint64_t *ws, InstStatus *st, SortPlan *plan,
                                                    SortTotals *tot, uint32_t tile) {
    const uint32_t m = args->m;
    uint64_t base[5] = {0, 0, 0, 0, 0};  // tiles, offT entries, buckets, groups, group sums
    for (uint32_t i0 = 0; i0 < m; i0 += blockDim.x) {
        const uint32_t i = i0 + threadIdx.x;
        SortPlan pl{};
        uint64_t v[5] = {0, 0, 0, 0, 0};
        if (i < m) {
            const Instance &in = inst[i];
            const uint32_t e = __hip_atomic_load(&st[i].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!(e & kErrRange) && in.prior_inserts + st[i].inserts > 0xffffffffull)
                atomic_or_u32(&st[i].err, kErrRange);
            pl.w_begin = ws[in.read_begin];
            pl.w_end = ws[in.read_end];
            pl.valid = !(e & (kErrInval | kErrSkip)) && in.parts;
            if (pl.valid) pl.tiles = (pl.w_end - pl.w_begin + tile - 1) / tile;
            v[0] = pl.tiles;
            if (in.fan > 1) {
                pl.groups = (pl.tiles + kSortGroup - 1) / kSortGroup;
                v[1] = pl.tiles * in.d1;
                v[2] = in.d1;
                v[3] = pl.groups;
                v[4] = pl.groups * in.d1;
            }
        }
        uint64_t ex[5];
        for (int q = 0; q < 5; ++q) {
            uint64_t total;
            ex[q] = base[q] + block_exclusive_scan(v[q], &total);
            base[q] += total;
        }
        if (i < m) {
            pl.tile_base = ex[0];
            pl.offt_base = ex[1];
            pl.bucket_base = ex[2];
            pl.group_base = ex[3];
            pl.gsum_base = ex[4];
            plan[i] = pl;
        }
    }
    if (threadIdx.x == 0) {
        tot->tiles = base[0];
        tot->buckets = base[2];
        tot->groups = base[3];
    }
}

// First read of every tile: read r writes the tiles whose first window falls
// among its windows.  The bytes of a read without a window are checked here
// (k_sort_windows checks those that its windows cover).
__global__ void k_sort_tile_reads(const PassArgs *__restrict__ args, const Instance *__restrict__ inst,
                                  const uint64_t *__restrict__ ws, const SortPlan *__restrict__ plan, InstStatus *st,
                                  uint64_t *__restrict__ tile_read, uint32_t tile) {
    const uint32_t m = args->m;
    const uint64_t n = args->n_reads;
    const uint64_t *__restrict__ off = as_global(args->off);
    const uint8_t *__restrict__ ascii = as_global(args->reads);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const uint64_t a = ws[r], z = ws[r + 1];
        const uint32_t i = m == 1 ? 0u : instance_of_read(inst, m, r);
        const SortPlan &pl = plan[i];
        if (!pl.valid) continue;  // instance not built in this launch
        if (z == a) {
            bool good = true;
            for (uint64_t q = off[r] - off[0]; q < off[r + 1] - off[0]; ++q) good &= valid_letter(ascii[q]);
            if (!good) atomic_or_u32(&st[i].err, kErrBase);
            continue;
        }
        for (uint64_t t = (a - pl.w_begin + tile - 1) / tile; pl.w_begin + t * tile < z; ++t)
            tile_read[pl.tile_base + t] = r;
    }
}

// ---------------------------------------------------------------- level 1

// Codes of four letters (first in the low byte) as 8 bits, first letter on
// top; *bad has a nonzero byte for each byte outside ACGTacgt.
__device__ __forceinline__ uint32_t pack4(uint32_t x, uint32_t *bad) {
    const uint32_t c = (x >> 1) & 0x03030303u;
    *bad |= __builtin_amdgcn_perm(0u, 0x67746361u, c) ^ (x | 0x20202020u);  // the letter of each code: a c t g
    return (c * 0x40100401u) >> 24;
}

__device__ __forceinline__ uint32_t pack16(uint4 v, uint32_t *bad) {
    return pack4(v.x, bad) << 24 | pack4(v.y, bad) << 16 | pack4(v.z, bad) << 8 | pack4(v.w, bad);
}

// n <= 80 bases from byte p of the reads on, as packed words, sixteen bytes at a
// time while these lie in the reads (len bytes); bad: a byte of the n outside
// ACGTacgt.
struct Bases {
    uint64_t x[3];
    bool bad;
};
using Bytes16 = uint32_t __attribute__((ext_vector_type(4), aligned(1), may_alias));

__device__ __forceinline__ Bases ascii_bases(const uint8_t *ascii, uint64_t len, uint64_t p, uint32_t n) {
    uint32_t v[6] = {0, 0, 0, 0, 0, 0};
    bool good = true;
#pragma unroll
    for (uint32_t c = 0; c < 5; ++c) {
        if (16 * c >= n) break;
        const uint8_t *at = ascii + p + 16 * c;
        uint32_t bad = 1;
        if (p + 16 * c + 16 <= len) {
            const Bytes16 q = *reinterpret_cast<const Bytes16 *>(at);
            bad = 0;
            v[c] = pack16(make_uint4(q.x, q.y, q.z, q.w), &bad);
        }
        if (bad) {  // the n bytes one by one (a byte behind them is not looked at)
            v[c] = 0;
            for (uint32_t i = 0; i < min(16u, n - 16 * c); ++i) {
                good &= valid_letter(at[i]);
                v[c] |= (((uint32_t)at[i] >> 1) & 3u) << (30 - 2 * i);
            }
        }
    }
    return Bases{{(uint64_t)v[0] << 32 | v[1], (uint64_t)v[2] << 32 | v[3], (uint64_t)v[4] << 32}, !good};
}

// The read of window w, which starts it, behind read r (ws[r + 1] == w): the
// last of those up to r1 that start at w, as reads shorter than k have no window.
__device__ __forceinline__ uint64_t next_read(const uint64_t *__restrict__ ws, uint64_t r, uint64_t r1, uint64_t w) {
    uint64_t step = 1;
    for (++r; r + step <= r1 && ws[r + step] <= w; step *= 2) r += step;
    for (; step; step /= 2)
        if (r + step <= r1 && ws[r + step] <= w) r += step;
    return r;
}

template <uint32_t RW>
__device__ __forceinline__ typename RecOf<RW>::T record_of(uint64_t x0, uint64_t x1, uint32_t km1, uint64_t sink) {
    if constexpr (RW == 1) {
        return (key_image(x0 >> (64 - 2 * km1)) << 3) | sink | ((uint32_t)(x0 >> (62 - 2 * km1)) & 3u);
    } else {
        uint64_t kh, kl, ih, il;
        uint32_t letter;
        wide_window(x0, x1, km1, kh, kl, letter);
        wide_image(kh, kl, ih, il);
        return make_ulonglong2((ih << 3) | sink | letter, il);
    }
}

// Dynamic LDS: s_cnt[d1_max + 1], then room for the tile's records; until the
// records are placed, it holds the tile's reads (window and base of each) and
// its packed bases, half each.
__host__ __device__ inline uint32_t sort_lds_bytes(uint32_t digits_max, uint32_t room) {
    return align16(4 * (digits_max + 1)) + room;
}

template <uint32_t RW, uint32_t BLOCK, uint32_t PER, bool WORDS>
__global__ __launch_bounds__(BLOCK) void k_sort_windows(const PassArgs *__restrict__ args,
                                                        const Instance *__restrict__ inst,
                                                        const uint64_t *__restrict__ ws,
                                                        const SortPlan *__restrict__ plan,
                                                        const uint64_t *__restrict__ tile_read, InstStatus *st,
                                                        uint64_t *__restrict__ rec1w, uint16_t *__restrict__ off1,
                                                        uint32_t row_len, uint32_t d1_max) {
    using R = typename RecOf<RW>::T;
    constexpr uint32_t T = Tile<BLOCK, PER>::n, RB = Tile<BLOCK, PER>::rb;
    constexpr uint32_t kRoom = tile_room(T, RW, WORDS);
    constexpr uint32_t kReads = kRoom / 16 - 1;  // staged reads (8 bytes each, one more for the end)
    constexpr uint32_t kWords = kRoom / 16;      // packed words of 32 bases
    __shared__ uint32_t s_w[BLOCK / 64];
    __shared__ uint64_t s_roll[16];
    extern __shared__ __align__(16) unsigned char s_dyn[];
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s_dyn);
    unsigned char *s_room = s_dyn + align16(4 * (d1_max + 1));
    uint2 *s_read = reinterpret_cast<uint2 *>(s_room);  // x: the read's first window in the tile, y: its base
    uint64_t *s_word = reinterpret_cast<uint64_t *>(s_room) + kReads + 1;
    const uint32_t tid = threadIdx.x, m = args->m;
    const uint64_t tile = blockIdx.x;
    const uint32_t i = m == 1 ? 0u : (uint32_t)last_le(m, tile, [&](uint64_t j) { return plan[j].tile_base; });
    const SortPlan &pl = plan[i];
    const uint64_t t = tile - pl.tile_base;
    if (t >= pl.tiles) return;
    const Instance &in = inst[i];
    const uint64_t *__restrict__ off = as_global(args->off);
    const uint64_t off0 = off[0], len = args->reads_len;
    const uint8_t *__restrict__ ascii = as_global(args->reads);
    const uint32_t k = in.k, d1 = in.d1;
    const uint64_t w0 = pl.w_begin + t * T;
    const uint32_t n_in = (uint32_t)min<uint64_t>(T, pl.w_end - w0);
    const bool last = t + 1 == pl.tiles;
    const uint64_t r0 = tile_read[tile];
    const uint64_t r1 = last ? in.read_end - 1 : tile_read[tile + 1];  // at or after the read of the last window
    // the bytes from the tile's first window to the end of its last one (or to read r1)
    const uint64_t p0 = off[r0] + (w0 - ws[r0]) - off0;
    const uint64_t p1 = (last ? off[r1 + 1]
                         : ws[r1] < w0 + T ? min(off[r1] + (w0 + T - ws[r1]) + k - 1, off[r1 + 1])
                                           : off[r1]) - off0;
    const int64_t pa = (int64_t)p0 - (int64_t)((reinterpret_cast<uintptr_t>(ascii) + p0) & 15);
    const uint64_t words = ((uint64_t)((int64_t)p1 - pa) + 31) / 32;
    const uint32_t n_reads = (uint32_t)min<uint64_t>(kReads, r1 - r0 + 1);

    for (uint32_t j = tid; j <= d1; j += BLOCK) s_cnt[j] = j << RB;
    if (RW == 1 && tid < 16) s_roll[tid] = roll_entry(tid, k);
    for (uint32_t j = tid; j <= n_reads; j += BLOCK) {
        const uint64_t wr = ws[r0 + j];
        const uint64_t skip = wr < w0 ? w0 - wr : 0;  // windows of the first read in earlier tiles
        uint2 e;
        e.x = (uint32_t)min<uint64_t>(wr + skip - w0, T + 1);
        e.y = j < n_reads ? (uint32_t)((int64_t)(off[r0 + j] - off0 + skip) - pa) : 0u;
        s_read[j] = e;
    }
    const bool fits = words + 3 <= kWords;  // (the words that a window's loads may touch past them included)
    for (uint32_t w = tid; fits && w < words; w += BLOCK) {
        const int64_t b = pa + 32 * (int64_t)w;
        uint64_t v;
        uint32_t bad = 0;
        if (b >= 0 && (uint64_t)b + 32 <= len) {
            const uint4 *src = reinterpret_cast<const uint4 *>(ascii + b);
            const uint4 lo = src[0], hi = src[1];
            v = (uint64_t)pack16(lo, &bad) << 32;
            v |= pack16(hi, &bad);
        } else {
            v = 0;
            bad = 1;
            for (int64_t q = 0; q < 32; ++q)
                if (b + q >= 0 && (uint64_t)(b + q) < len)
                    v |= (uint64_t)((ascii[b + q] >> 1) & 3u) << (62 - 2 * q);
        }
        s_word[w] = v;
        if (bad) {  // look at the tile's own bytes one by one
            const int64_t lo = max<int64_t>(b, (int64_t)p0), hi = min<int64_t>(b + 32, (int64_t)p1);
            for (int64_t q = lo; q < hi; ++q)
                if (!valid_letter(ascii[q])) {
                    atomic_or_u32(&st[i].err, kErrBase);
                    break;
                }
        }
    }
    __syncthreads();

    R rec[PER];
    uint32_t tag[PER];
    const uint32_t j0 = tid * PER;
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        rec[q] = RecOf<RW>::none();
        tag[q] = d1 << RB;
    }
    const bool staged = fits && s_read[n_reads].x >= n_in;  // all the tile's bases, and the reads of all its windows
    const uint32_t jend = min(j0 + PER, n_in);
    if (staged) {
        if (j0 < n_in) {
            uint32_t lo = 0, hi = n_reads;  // s_read[lo].x <= j0 < s_read[hi].x
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s_read[mid].x <= j0) lo = mid; else hi = mid;
            }
            const uint2 rd = s_read[lo];
            uint32_t e = s_read[lo + 1].x;  // the window that starts the next read
            if constexpr (RW == 1) {
                const uint32_t kshift = 64 - 2 * (k - 1);
                static_assert(PER <= 32, "F and L hold the bases of 32 windows");
                Roll cur = roll_at(s_word, rd.y + (j0 - rd.x), k, kshift);
                Roll next = cur;
                uint32_t e2 = e;
                // the state of the next read that starts among this thread's windows
                const auto prepare = [&]() {
                    do ++lo; while (s_read[lo + 1].x <= e2);  // reads shorter than k have no window
                    next = roll_at(s_word, s_read[lo].y, k, kshift);
                    e2 = s_read[lo + 1].x;
                };
                if (e < jend) prepare();
#pragma unroll
                for (uint32_t q = 0; q < PER; ++q) {
                    const uint32_t j = j0 + q;
                    const bool cross = j == e;
                    if (cross) cur = next;
                    e = cross ? e2 : e;
                    if (cross && e < jend) prepare();
                    const uint64_t img = cur.x ^ (cur.x >> 30);  // the key's image
                    rec[q] = (img << 3) | (j + 1 == e ? 4u : 0u) | (uint32_t)(cur.L >> 62);
                    const uint32_t b = bucket_of(image_top(img), d1);
                    tag[q] = lds_add32(&s_cnt[j < n_in ? b : d1], 1u);  // d1: past the tile's end
                    roll_next(cur, s_roll);
                }
            } else {
                uint32_t base = rd.y + (j0 - rd.x);
#pragma unroll
                for (uint32_t q = 0; q < PER; ++q) {
                    const uint32_t j = j0 + q;
                    if (j >= n_in) break;
                    if (j == e) {
                        do ++lo; while (s_read[lo + 1].x <= j);
                        base = s_read[lo].y;
                        e = s_read[lo + 1].x;
                    }
                    uint64_t x0, x1;
                    bases128_at(s_word, base, x0, x1);
                    rec[q] = record_of<RW>(x0, x1, k - 1, j + 1 == e ? 4u : 0u);
                    tag[q] = lds_add32(&s_cnt[bucket_of(image_top(RecOf<RW>::head(rec[q]) >> 3), d1)], 1u);
                    ++base;
                }
            }
        }
    } else {
        // More reads or bases than are staged: about two windows a read, or as many
        // reads without one.  Each thread takes the reads of its own windows from
        // the ASCII, and their records wait where the staging was.  Bound by the
        // latency of a few loads a read.  A build from 4 M reads of exactly k = 31
        // takes 0.40 ms (1.58 with each window found and decoded by itself, a byte at
        // a time), of 10-50 bases at k = 45 0.39 (1.22), from 60 M of exactly 21 4.4
        // (16.0).
        static_assert(!WORDS && PER + 62 <= 80, "room for the records; bases of a thread's windows of one read");
        R *s_rec = reinterpret_cast<R *>(s_room) + tid;
        __syncthreads();  // s_read has been looked at
        if (j0 < n_in) {
            bool bad = false;
            uint64_t w = w0 + j0, r = r0, hi = r1 + 1;  // ws[r] <= w < ws[hi]
            while (hi - r > 1) {
                const uint64_t mid = (r + hi) >> 1;
                if (ws[mid] <= w) r = mid; else hi = mid;
            }
            uint64_t at = off[r] - off0 + (w - ws[r]);
            for (uint32_t j = j0;;) {
                const uint64_t z = ws[r + 1];  // the window that starts the next read
                const uint32_t n = (uint32_t)min<uint64_t>(z - w, jend - j);
                Bases x = ascii_bases(ascii, len, at, (uint32_t)min<uint64_t>(n + k - 1, z - w + k - 2));
                bad |= x.bad;
                for (uint32_t i = 0; i < n; ++i) {
                    s_rec[(j++ - j0) * BLOCK] = record_of<RW>(x.x[0], x.x[1], k - 1, ++w == z ? 4u : 0u);
                    x.x[0] = x.x[0] << 2 | x.x[1] >> 62;
                    x.x[1] = x.x[1] << 2 | x.x[2] >> 62;
                    x.x[2] <<= 2;
                }
                if (j == jend) break;
                r = next_read(ws, r, r1, w);
                at = off[r] - off0;
            }
            if (bad) atomic_or_u32(&st[i].err, kErrBase);
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                if (j0 + q >= n_in) break;
                rec[q] = s_rec[q * BLOCK];
                tag[q] = lds_add32(&s_cnt[bucket_of(image_top(RecOf<RW>::head(rec[q]) >> 3), d1)], 1u);
            }
        }
    }
    __syncthreads();
    digit_starts<BLOCK, RB>(s_cnt, d1, n_in, s_w, off1 + tile * row_len);
    __syncthreads();
    place_and_store<BLOCK, PER, RB, WORDS>(rec, tag, s_cnt, d1, s_room, n_in, reinterpret_cast<R *>(rec1w) + tile * T);
}

// ---------------------------------------------------------------- between the levels

// Offsets of kSortGroup tiles, transposed: offT[bucket][tile] = start | count
// << 16, and each bucket's records in the group.  A workgroup per group and 64
// buckets.  Bound by latency: a wavefront's rows are loaded together (a
// workgroup of 256 threads per group, 64 buckets after the other and a load at a
// time, took 36 us for 121 million windows and 31 for 27 million; now 10.5 and 5.8).
constexpr uint32_t kTransBlock = 1024, kTransRows = kSortGroup / (kTransBlock / 64);

__global__ __launch_bounds__(kTransBlock) void k_sort_transpose(const PassArgs *__restrict__ args,
                                                                const Instance *__restrict__ inst,
                                                                const SortPlan *__restrict__ plan,
                                                                const uint16_t *__restrict__ off1, uint32_t row_len,
                                                                uint32_t *__restrict__ offt,
                                                                uint32_t *__restrict__ gsum) {
    __shared__ uint16_t s_off[kSortGroup][66];
    const uint32_t m = args->m, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t G = blockIdx.x;
    const uint32_t b0 = blockIdx.y * 64;
    const uint32_t i = m == 1 ? 0u : (uint32_t)last_le(m, G, [&](uint64_t j) { return plan[j].group_base; });
    const SortPlan &pl = plan[i];
    const uint64_t g = G - pl.group_base;
    const uint32_t d1 = inst[i].d1;
    if (g >= pl.groups || b0 >= d1) return;
    const uint64_t t0 = g * kSortGroup;
    const uint32_t nt = (uint32_t)min<uint64_t>(kSortGroup, pl.tiles - t0), nb = min(64u, d1 - b0);
    const uint16_t *rows = off1 + (pl.tile_base + t0) * row_len + b0;
    uint16_t v[kTransRows], end = 0;  // (row_len covers d1 + 1 offsets)
#pragma unroll
    for (uint32_t j = 0; j < kTransRows; ++j)
        v[j] = rows[(uint64_t)min(wave * kTransRows + j, nt - 1) * row_len + min(lane, nb)];
    if (threadIdx.x < nt) end = rows[(uint64_t)threadIdx.x * row_len + nb];
#pragma unroll
    for (uint32_t j = 0; j < kTransRows; ++j) s_off[wave * kTransRows + j][lane] = v[j];
    __syncthreads();
    if (threadIdx.x < nt) s_off[threadIdx.x][nb] = end;
    __syncthreads();
    for (uint32_t c = wave; c < nb; c += kTransBlock / 64) {
        uint32_t a = 0, n = 0;
        if (lane < nt) {
            a = s_off[lane][c];
            n = (uint32_t)s_off[lane][c + 1] - a;
            offt[pl.offt_base + (uint64_t)(b0 + c) * pl.tiles + t0 + lane] = a | n << 16;
        }
        const uint32_t sum = wave_scan(n);
        if (lane == 63) gsum[pl.gsum_base + (uint64_t)(b0 + c) * pl.groups + g] = sum;
    }
}
static_assert(kSortGroup == 64, "a lane per tile of a group");

// Per level-1 bucket: the records before each of its groups (gpre, 64 bits:
// a bucket may hold every window) and its size.  A workgroup per bucket.
__global__ __launch_bounds__(256) void k_sort_groups(const PassArgs *__restrict__ args,
                                                     const SortTotals *__restrict__ tot,
                                                     const SortPlan *__restrict__ plan,
                                                     const uint32_t *__restrict__ gsum, uint64_t *__restrict__ gpre,
                                                     SortBucket *__restrict__ buckets) {
    const uint64_t g = blockIdx.x;
    if (g >= tot->buckets) return;
    const uint32_t i = (uint32_t)last_le(args->m, g, [&](uint64_t j) { return plan[j].bucket_base; });
    const SortPlan &pl = plan[i];
    const uint32_t b = (uint32_t)(g - pl.bucket_base);
    const uint64_t row = pl.gsum_base + (uint64_t)b * pl.groups;
    uint64_t carry = 0;
    for (uint64_t x0 = 0; x0 < pl.groups; x0 += blockDim.x) {
        const uint64_t x = x0 + threadIdx.x;
        const uint64_t v = x < pl.groups ? gsum[row + x] : 0;
        uint64_t total;
        const uint64_t ex = block_exclusive_scan(v, &total);
        if (x < pl.groups) gpre[row + x] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        buckets[g].size = carry;
        buckets[g].inst = i;
        buckets[g].b = b;
    }
}

// Where each bucket's level-2 records start (whole 128-byte lines) and its
// first level-2 tile; tile2_base[buckets] is the number of tiles.  One block.
__global__ __launch_bounds__(1024) void k_sort_buckets(const SortTotals *__restrict__ tot,
                                                       SortBucket *__restrict__ buckets,
                                                       uint64_t *__restrict__ tile2_base, uint32_t tile2) {
    const uint64_t G = tot->buckets;
    uint64_t at = 0, tiles = 0;
    for (uint64_t g0 = 0; g0 < G; g0 += blockDim.x) {
        const uint64_t g = g0 + threadIdx.x;
        const uint64_t size = g < G ? buckets[g].size : 0;
        uint64_t ta, tt;
        const uint64_t ea = block_exclusive_scan((size + 15) & ~15ull, &ta);
        const uint64_t et = block_exclusive_scan((size + tile2 - 1) / tile2, &tt);
        if (g < G) {
            buckets[g].start = at + ea;
            tile2_base[g] = tiles + et;
        }
        at += ta;
        tiles += tt;
    }
    if (threadIdx.x == 0) tile2_base[G] = tiles;
}

// ---------------------------------------------------------------- level 2

// A level-2 tile takes records [s T, (s + 1) T) of its bucket, counted over
// the bucket's pieces in tile order.  The pieces that cover them are laid end
// to end: bit r of the tile's bitmap marks that a piece starts at record r, so
// record r belongs to the piece numbered (marks at or before r) - 1, and one
// table entry per piece leads from r to the record's place.
constexpr uint32_t kPieces = 2048;  // pieces of a tile kept in LDS

struct Level2Lds {
    uint32_t cnt, room, mark, base, piece, bytes;
};

__host__ __device__ inline Level2Lds level2_lds(uint32_t fan_max, uint32_t tile, uint32_t room) {
    Level2Lds o;
    o.cnt = 0;
    o.mark = align16(4 * (fan_max + 1));
    o.base = o.mark + tile / 8;
    o.room = o.base + tile / 64 * 4;
    o.piece = o.room;  // the pieces are done with before records are placed
    o.bytes = o.room + room;
    return o;
}

template <uint32_t RW, uint32_t BLOCK, uint32_t PER, bool WORDS>
__global__ __launch_bounds__(BLOCK) void k_sort_bucket(const SortTotals *__restrict__ tot,
                                                       const Instance *__restrict__ inst,
                                                       const SortPlan *__restrict__ plan,
                                                       const SortBucket *__restrict__ buckets,
                                                       const uint64_t *__restrict__ tile2_base,
                                                       const uint64_t *__restrict__ gpre,
                                                       const uint32_t *__restrict__ offt,
                                                       const uint64_t *__restrict__ rec1w,
                                                       uint64_t *__restrict__ rec2w, uint16_t *__restrict__ off2,
                                                       uint32_t row_len, uint32_t fan_max, uint32_t tile1) {
    using R = typename RecOf<RW>::T;
    constexpr uint32_t T = Tile<BLOCK, PER>::n, RB = Tile<BLOCK, PER>::rb;
    constexpr uint32_t Q = T / 64;  // words of the bitmap
    static_assert(Q <= BLOCK && kPieces * 8 <= tile_room(T, RW, WORDS), "bitmap and pieces");
    __shared__ uint32_t s_w[BLOCK / 64], s_w2[BLOCK / 64];
    __shared__ uint32_t s_at, s_over;
    __shared__ uint64_t s_group;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    const Level2Lds lay = level2_lds(fan_max, T, tile_room(T, RW, WORDS));
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s_dyn);
    uint64_t *s_mark = reinterpret_cast<uint64_t *>(s_dyn + lay.mark);
    uint32_t *s_base = reinterpret_cast<uint32_t *>(s_dyn + lay.base);
    uint64_t *s_piece = reinterpret_cast<uint64_t *>(s_dyn + lay.piece);
    const R *__restrict__ rec1 = reinterpret_cast<const R *>(rec1w);
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t tile = blockIdx.x, G = tot->buckets;
    if (G == 0 || tile >= tile2_base[G]) return;  // uniform
    for (uint64_t g = tid; g < G; g += BLOCK)
        if (tile2_base[g] <= tile && tile < tile2_base[g + 1]) s_at = (uint32_t)g;
    if (tid == 0) s_over = 0;
    if (tid < Q) s_mark[tid] = 0;
    __syncthreads();
    const SortBucket B = buckets[s_at];
    const Instance &in = inst[B.inst];
    const SortPlan &pl = plan[B.inst];
    const uint32_t d1 = in.d1, fan = min(in.fan, in.parts - B.b * in.fan);
    const uint64_t first = (tile - tile2_base[s_at]) * T;  // in the bucket
    const uint32_t n = (uint32_t)min<uint64_t>(T, B.size - first);
    const uint64_t *gp = gpre + pl.gsum_base + (uint64_t)B.b * pl.groups;
    for (uint64_t g = tid; g < pl.groups; g += BLOCK) {
        const uint64_t lo = gp[g], hi = g + 1 < pl.groups ? gp[g + 1] : B.size;
        if (lo <= first && first < hi) s_group = g;
    }
    for (uint32_t j = tid; j <= fan; j += BLOCK) s_cnt[j] = j << RB;
    __syncthreads();
    const uint32_t *pieces = offt + pl.offt_base + (uint64_t)B.b * pl.tiles;
    uint64_t pos = gp[s_group];  // records of the bucket before piece t0
    R rec[PER];
    for (uint64_t t0 = s_group * kSortGroup; t0 < pl.tiles && pos < first + n; t0 += BLOCK) {
        const uint64_t t = t0 + tid;
        const uint32_t u = t < pl.tiles ? pieces[t] : 0u;
        uint32_t len = u >> 16, total;
        const uint64_t p = pos + block_scan<BLOCK>(len, s_w, &total);
        const uint64_t a = max(p, first), z = min(p + len, first + n);  // its records in this tile
        const uint32_t r = (uint32_t)(a - first);
        const bool has = z > a;
        if (has) __hip_atomic_fetch_or(&s_mark[r >> 6], 1ull << (r & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        // marks before each word (those of later pieces follow)
        const uint32_t marks = tid < Q ? (uint32_t)__popcll(s_mark[tid]) : 0u;
        uint32_t all;
        const uint32_t before = block_scan<BLOCK>(marks, s_w2, &all);
        if (tid < Q) s_base[tid] = before;
        __syncthreads();
        if (has) {
            const uint32_t rank = s_base[r >> 6] + (uint32_t)__popcll(s_mark[r >> 6] & ((1ull << (r & 63)) - 1));
            if (rank < kPieces) s_piece[rank] = t * tile1 + (u & 0xffffu) + (a - p) - r;
            else s_over = 1;
        }
        pos += total;
    }
    __syncthreads();
    const uint64_t rec_base = pl.tile_base * tile1;
    if (!s_over) {
        const R *src = rec1 + rec_base;
#pragma unroll
        for (uint32_t it = 0; it < PER; ++it) {  // no branch: the loads follow each other
            const uint32_t q = it * (BLOCK / 64) + wave, r = q * 64 + lane;
            const uint32_t upto = s_base[q] + (uint32_t)__popcll(s_mark[q] & (~0ull >> (63 - lane)));
            const uint64_t at = s_piece[(upto - 1) & (kPieces - 1)] + r;
            rec[it] = src[r < n ? at : 0];
        }
    } else {
        // more pieces than fit (few records in many tiles): each thread walks
        // the tiles from its first record on
        const uint32_t r0 = tid * PER;
        if (r0 < n) {
            uint64_t g0 = s_group, g1 = pl.groups;
            while (g1 - g0 > 1) {
                const uint64_t mid = (g0 + g1) >> 1;
                if (gp[mid] <= first + r0) g0 = mid; else g1 = mid;
            }
            uint64_t t = g0 * kSortGroup, p = gp[g0];
            uint32_t u = pieces[t];
#pragma unroll
            for (uint32_t it = 0; it < PER; ++it) {
                if (r0 + it < n) {
                    const uint64_t x = first + r0 + it;
                    while (p + (u >> 16) <= x) {
                        p += u >> 16;
                        u = pieces[++t];
                    }
                    rec[it] = rec1[rec_base + t * tile1 + (u & 0xffffu) + (x - p)];
                }
            }
        }
    }
    uint32_t tag[PER];
#pragma unroll
    for (uint32_t it = 0; it < PER; ++it) {
        const uint32_t r = s_over ? tid * PER + it : (it * (BLOCK / 64) + wave) * 64 + lane;
        tag[it] = lds_add32(&s_cnt[r < n ? child_of(image_top(RecOf<RW>::head(rec[it]) >> 3), d1, fan) : fan], 1u);
    }
    __syncthreads();
    digit_starts<BLOCK, RB>(s_cnt, fan, n, s_w, off2 + tile * row_len);
    __syncthreads();
    place_and_store<BLOCK, PER, RB, WORDS>(rec, tag, s_cnt, fan, s_dyn + lay.room, n,
                                           reinterpret_cast<R *>(rec2w) + B.start + first);
}

// ---------------------------------------------------------------- reduce

// Where the pieces of a run of segments lie: piece s of segment gp holds
// records [row[0], row[1]) of tile s, with row = off + s * row_len + (gp - gp0).
// (Segments count from the workgroup's first one here and in Unit, in 32 bits.)
struct Source {
    const uint16_t *off;   // offsets of segment gp0 in tile 0
    const uint64_t *rec;   // tile 0's records
    int32_t gp0, gp1;      // the run of segments (it may have begun before the workgroup's first)
    uint32_t pieces;       // of a segment
    uint32_t pairs;        // pairs of units of a segment
    uint32_t units;        // units of a pair: 2, or 1 where a unit holds the segment
    uint32_t per_unit;     // pieces of a unit
    uint32_t row_len, tile;  // offsets a row, records a tile
    uint32_t rows;         // a segment's pieces are read in rows of 64 records, not in units
};

// A planned unit: consecutive pieces of one segment.
struct Unit {
    const uint64_t *rec;   // its first tile's records
    uint32_t gp, first;    // its segment, its first piece
    uint32_t n;            // its records
    uint32_t last;         // the segment ends with its pair
};

constexpr uint32_t kUnitPieces = 128;     // two a lane of the wavefront that plans the unit
constexpr uint32_t kUnitRounds = 4;       // records a thread takes from a unit
constexpr uint32_t kUnitRecords = kUnitRounds * kReduceBlock;  // a larger unit is read piece by piece
constexpr uint32_t kUnitTarget = 1800;    // records a unit is meant to have at most
constexpr uint32_t kStageUnits = 4;       // planned together

// Few segments and many tiles (a small genome read deeply): a segment is many
// pairs of units, and nothing of a pair's loads and planning hides behind a
// write-back.  Where its pieces have kRowPiece records or more on average they
// are read in rows of 64 instead, each wavefront its own, without a plan or a
// barrier.  Bound by the latency of the LDS probes, of which a wavefront has one
// row's under way.  ms of a reset and build, units / rows (count-and-scatter): 24 M
// windows in 6 segments 9.3 / 7.2 (6.7), 122 M in 25 14.1 / 11.7 (11.6), in 56
// 6.1 / 5.9 (5.7).  With shorter pieces a row's last lanes idle: 122 M in 110
// 3.5 / 4.1, 48 sets in a batch 6.6 / 7.2.  And where a workgroup has several
// segments, others of its CU and its next segment's loads hide the stalls: 1.67 M
// reads of 15-75 bases in 8300 segments 0.66 / 0.68.
constexpr uint32_t kRowPiece = 128, kRowsAtOnce = 8;

// The pass's end: the last workgroup to come here stores the statuses in the
// host's memory (a copy command after the kernel takes longer).  Whole block.
// The statuses are written and read by device-wide atomics alone, so all that a
// workgroup needs before it counts itself is that its own are done: a fence
// would write back its XCD's whole L2, the table just stored included (100 us
// more for a 5 Mbp genome at 30x; one counter instead of kDoneLines, 20).
__device__ __forceinline__ void finish_pass(const PassArgs *args, const InstStatus *st, uint64_t *done, uint32_t *s_last) {
    if (!done) return;  // uniform
    __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t line = blockIdx.x % kDoneLines, lines = min(gridDim.x, kDoneLines);
        const uint32_t on_line = (gridDim.x - line + kDoneLines - 1) / kDoneLines;
        const auto last = [&](uint32_t which, uint32_t of) {
            return __hip_atomic_fetch_add(done + which * kDoneStride, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                       1 == of;
        };
        *s_last = last(line, on_line) && last(kDoneLines, lines);
    }
    __syncthreads();
    if (!*s_last) return;
    const uint64_t *from = reinterpret_cast<const uint64_t *>(st);
    uint64_t *to = as_global(reinterpret_cast<uint64_t *>(args->host_status));
    const uint32_t words = args->m * (uint32_t)(sizeof(InstStatus) / 8);
    for (uint32_t i = threadIdx.x; i < words; i += kReduceBlock)
        to[i] = __hip_atomic_load(from + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
static_assert(sizeof(InstStatus) % 8 == 0, "copied in words");

using Offsets2 = uint32_t __attribute__((aligned(2), may_alias));  // two 16-bit offsets side by side

// One workgroup per run of segments.  A segment's records are its pieces laid
// end to end.  They are read in pairs of units, a unit being up to 128
// consecutive pieces that a wavefront plans (a scan of the lengths, a bitmap of
// the starts and a place per piece, as in k_sort_bucket); a segment of the
// usual size is one pair, and a stage plans two pairs; a segment of fewer records
// is one unit, and a stage plans four.  As nothing but LDS sits
// between a pair's records and the table, all of the next pair's records load
// while a segment is written back, and the next stage's offsets load a stage
// ahead; the planning itself goes where the write-back has its barriers anyway.
template <uint32_t EW, uint32_t RW, bool STATS>
__global__ __launch_bounds__(kReduceBlock) __attribute__((amdgpu_waves_per_eu(RW == 1 ? 6 : 4))) void k_reduce_pieces(
    const PassArgs *__restrict__ args, const Instance *__restrict__ inst, const SortPlan *__restrict__ plan,
    const SortBucket *__restrict__ buckets, const uint64_t *__restrict__ tile2_base, const uint16_t *__restrict__ off1,
    const uint16_t *__restrict__ off2, const uint64_t *__restrict__ rec1w, const uint64_t *__restrict__ rec2w,
    uint32_t row1, uint32_t row2, uint32_t tile1, uint32_t tile2, InstStatus *st, uint64_t *done) {
    using R = typename RecOf<RW>::T;
    static_assert(RW == 1 || EW == 4, "long keys take 32-byte entries");
    constexpr uint32_t Q = kUnitRecords / 64;
    __shared__ uint64_t s_key[kSegSlots * RW];  // RW = 2: hi words, then lo words
    __shared__ __align__(16) uint32_t s_cnt[kSegSlots * 4];
    __shared__ uint64_t s_mark[kStageUnits][Q];
    __shared__ uint32_t s_piece[kStageUnits][kUnitPieces];
    __shared__ uint8_t s_base[kStageUnits][Q];
    __shared__ Unit s_unit[kStageUnits];
    __shared__ Source s_src[2];  // of the stage being read, and of the next one when another run starts there
    __shared__ uint32_t s_wave_n[kReduceWaves], s_claims[kReduceWaves];
    __shared__ uint64_t s_xbase;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t m = args->m;
    const uint64_t parts_total = args->parts_total;
    const uint32_t home_mask = args->test_hash ? 7u : kSegSlots - 1;
    ProbeStats ps;
    const uint64_t per_block = (parts_total + gridDim.x - 1) / gridDim.x;
    const uint64_t gp0 = min((uint64_t)blockIdx.x * per_block, parts_total);
    const uint32_t n_gp = (uint32_t)(min(gp0 + per_block, parts_total) - gp0);  // the workgroup's segments
    const auto finish = [&]() { finish_pass(args, st, done, &s_claims[0]); };
    if (n_gp == 0) {
        finish();
        return;
    }
    // LDS starts zeroed and every write-back leaves it zeroed again
    for (uint32_t s = tid; s < kSegSlots; s += kReduceBlock) {
        s_key[s] = 0;
        reinterpret_cast<uint4 *>(s_cnt)[s] = make_uint4(0, 0, 0, 0);
    }
    const auto skipped = [&](uint32_t i) {
        return (__hip_atomic_load(&st[i].err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kSkipMask) != 0;
    };
    // the run of segments that holds the workgroup's segment rel
    const auto source_at = [&](uint32_t rel) {
        const uint64_t gp = gp0 + rel;
        uint64_t first;
        Source S;
        const uint32_t i = m == 1 ? 0u : (uint32_t)last_le(m, gp, [&](uint64_t j) { return inst[j].part_base; });
        const Instance &in = inst[i];
        const SortPlan &pl = plan[i];
        uint32_t width = in.parts;
        if (in.fan == 1) {
            first = in.part_base;
            S.pieces = (uint32_t)pl.tiles;
            S.off = off1 + pl.tile_base * row1;
            S.rec = rec1w + pl.tile_base * tile1 * RW;
            S.row_len = row1;
            S.tile = tile1;
        } else {
            const uint32_t b = (uint32_t)(gp - in.part_base) / in.fan;
            const uint64_t g = pl.bucket_base + b;
            width = min(in.fan, in.parts - b * in.fan);
            first = in.part_base + (uint64_t)b * in.fan;
            S.pieces = (uint32_t)(tile2_base[g + 1] - tile2_base[g]);
            S.off = off2 + tile2_base[g] * row2;
            S.rec = rec2w + buckets[g].start * RW;
            S.row_len = row2;
            S.tile = tile2;
        }
        if (skipped(i)) S.pieces = 0;
        S.gp0 = (int32_t)((int64_t)first - (int64_t)gp0);
        S.gp1 = S.gp0 + (int32_t)width;
        const uint32_t most = min(kUnitPieces, max(1u, (uint32_t)((uint64_t)kUnitTarget * width / S.tile)));
        S.pairs = max(1u, (S.pieces + 2 * most - 1) / (2 * most));
        S.rows = S.pairs > 1 && per_block == 1 && width * kRowPiece <= S.tile;
        S.units = S.rows || S.pieces <= most ? 1u : 2u;
        if (S.rows) S.pairs = 1;
        S.per_unit = S.units == 1 ? S.pieces : (S.pieces + 2 * S.pairs - 1) / (2 * S.pairs);
        return S;
    };
    // The next stage: its pairs, and this wavefront's unit of it with this
    // lane's two pieces: each one's first and last record in its tile, as they lie
    // in the row of offsets.  They are taken apart when the unit is planned: that
    // is where a wavefront is to wait for them, not here.
    uint32_t at = 0, at_pair = 0, cs = 0, ns = 0, next_pairs = 0, next_units = 0;  // cs, ns: s_src slots of this stage and the next
    Unit mine{};
    uint32_t ow[2] = {0, 0};
    const auto next_stage = [&]() {
        next_pairs = 0;
        if (at >= n_gp) return;
        if (at == 0 && at_pair == 0) {
            if (lane == 0) s_src[0] = source_at(at);
        } else if ((int32_t)at >= s_src[cs].gp1) {
            ns = cs ^ 1;
            if (lane == 0) s_src[ns] = source_at(at);  // every wavefront writes the same
        }
        __builtin_amdgcn_wave_barrier();
        const Source &S = s_src[ns];
        const uint32_t pairs = S.pairs, left = min((uint32_t)S.gp1, n_gp) - at;
        next_units = S.units;
        next_pairs = min(kStageUnits >> (next_units - 1), pairs == 1 ? left : pairs - at_pair);
        ow[0] = ow[1] = 0;
        if (wave < next_units * next_pairs) {
            const uint32_t x = wave >> (next_units - 1), pair = pairs == 1 ? 0u : at_pair + x;
            mine.gp = pairs == 1 ? at + x : at;
            mine.last = pair + 1 == pairs;
            mine.first = (next_units * pair + (wave & (next_units - 1))) * S.per_unit;
            mine.rec = S.rec + (uint64_t)mine.first * S.tile * RW;
            const uint16_t *o = as_global(S.off) + ((int32_t)mine.gp - S.gp0);
#pragma unroll
            for (uint32_t h = 0; h < 2; ++h) {
                const uint32_t p = 2 * lane + h, s = mine.first + p;
                if (p < S.per_unit && s < S.pieces) ow[h] = *reinterpret_cast<const Offsets2 *>(o + (uint64_t)s * S.row_len);
            }
        }
        if (pairs == 1) {
            at += next_pairs;
        } else {
            at_pair += next_pairs;
            if (at_pair == pairs) {
                at_pair = 0;
                ++at;
            }
        }
    };
    // plan this wavefront's unit of the next stage
    const auto plan_unit = [&]() {
        if (wave >= next_units * next_pairs) return;
        asm volatile("" : "+v"(ow[0]), "+v"(ow[1]));  // nothing of this is moved up to the loads
        const uint32_t oa[2] = {ow[0] & 0xffffu, ow[1] & 0xffffu};
        const uint32_t n0 = (ow[0] >> 16) - oa[0], n1 = (ow[1] >> 16) - oa[1];
        const uint32_t inc = wave_scan(n0 + n1), p0 = inc - n0 - n1, p1 = inc - n1;
        mine.n = __builtin_amdgcn_readlane(inc, 63);
        if (s_src[ns].rows) mine.n = ~0u;
        if (lane < Q) s_mark[wave][lane] = 0;
        __builtin_amdgcn_wave_barrier();
        if (mine.n <= kUnitRecords) {  // uniform
            const uint64_t some0 = __ballot(n0 != 0), some1 = __ballot(n1 != 0), below = (1ull << lane) - 1;
            const uint32_t rank = (uint32_t)(__popcll(some0 & below) + __popcll(some1 & below));
            const uint32_t tile = s_src[ns].tile;
            if (n0) {
                __hip_atomic_fetch_or(&s_mark[wave][p0 >> 6], 1ull << (p0 & 63), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                s_piece[wave][rank] = 2 * lane * tile + oa[0] - p0;
            }
            if (n1) {
                __hip_atomic_fetch_or(&s_mark[wave][p1 >> 6], 1ull << (p1 & 63), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                s_piece[wave][rank + (n0 ? 1u : 0u)] = (2 * lane + 1) * tile + oa[1] - p1;
            }
            __builtin_amdgcn_wave_barrier();
            const uint32_t c = lane < Q ? (uint32_t)__popcll(lds_load64(&s_mark[wave][lane])) : 0u;
            const uint32_t before = wave_scan(c) - c;
            if (lane < Q) s_base[wave][lane] = (uint8_t)before;
        }
        if (lane == 0) s_unit[wave] = mine;
    };
    // The block's records of the planned pair x, and how many each unit has
    // (none if it is read piece by piece).  Every load is issued, those past the
    // end at a place that is always there, so that they follow each other.
    R rv[2 * kUnitRounds];
    uint32_t n_rv[2] = {0, 0};
    const auto load_pair = [&](uint32_t units, uint32_t x) {
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
            const R *src[kUnitRounds];
            const uint32_t u = units * x + (h < units ? h : 0);
            n_rv[h] = __builtin_amdgcn_readfirstlane(h < units && s_unit[u].n <= kUnitRecords ? s_unit[u].n : 0u);
            const R *rec = reinterpret_cast<const R *>(as_global(s_unit[u].rec));
            const auto find = [&](uint32_t c) {
                const uint32_t q = c * kReduceWaves + wave, r = q * 64 + lane;
                const uint32_t upto = s_base[u][q] + (uint32_t)__popcll(s_mark[u][q] & (~0ull >> (63 - lane)));
                const uint32_t to = s_piece[u][(upto - 1) & (kUnitPieces - 1)] + r;
                if (r < n_rv[h]) src[c] = rec + to;
            };
#pragma unroll
            for (uint32_t c = 0; c < kUnitRounds; ++c) src[c] = reinterpret_cast<const R *>(rec1w);
            if (n_rv[h] > kReduceBlock) {
#pragma unroll
                for (uint32_t c = 0; c < kUnitRounds; ++c) find(c);
            } else if (n_rv[h]) {
                find(0);
            }
#pragma unroll
            for (uint32_t c = 0; c < kUnitRounds; ++c) rv[h * kUnitRounds + c] = *src[c];
        }
    };

    uint64_t my_claims = 0;  // this thread's in the segment
    bool full = false;
    // Pieces [s0, s1) of the workgroup's segment rel, read where they lie: rows of
    // 64 records, numbered over 64 pieces at a time, every eighth to a wavefront.
    const auto take_rows = [&](const Source &S, uint32_t rel, uint32_t s0, uint32_t s1) {
        const uint16_t *o = as_global(S.off) + ((int32_t)rel - S.gp0);
        const R *rec = reinterpret_cast<const R *>(as_global(S.rec));
        for (uint32_t g = s0; g < s1; g += 64) {
            uint32_t a = 0, n = 0;  // this lane's piece
            if (g + lane < s1) {
                a = o[(uint64_t)(g + lane) * S.row_len];
                n = o[(uint64_t)(g + lane) * S.row_len + 1] - a;
            }
            const uint32_t inc = wave_scan((n + 63) / 64), first = inc - (n + 63) / 64;
            const uint32_t total = __builtin_amdgcn_readlane(inc, 63);
            for (uint32_t q0 = wave; q0 < total; q0 += kRowsAtOnce * kReduceWaves) {
                R v[kRowsAtOnce];
                uint32_t left[kRowsAtOnce];  // records of the piece from the row on
#pragma unroll
                for (uint32_t c = 0; c < kRowsAtOnce; ++c) {
                    const uint32_t q = q0 + c * kReduceWaves;
                    const uint64_t at = __ballot(first <= q && q < inc);  // none past the last row
                    const uint32_t piece = at ? (uint32_t)__builtin_ctzll(at) : 0u;
                    const uint32_t r = (q - __builtin_amdgcn_readlane(first, piece)) * 64;
                    left[c] = at ? (uint32_t)__builtin_amdgcn_readlane(n, piece) - r : 0u;
                    const uint64_t to = (uint64_t)(g + piece) * S.tile + __builtin_amdgcn_readlane(a, piece) + r;
                    v[c] = lane < left[c] ? rec[to + lane] : RecOf<RW>::none();
                }
#pragma unroll
                for (uint32_t c = 0; c < kRowsAtOnce; ++c)
                    if (lane < left[c] && !reduce_record<STATS>(v[c], s_key, s_cnt, my_claims, home_mask, ps)) full = true;
            }
        }
    };

    uint32_t cur_inst = m == 1 ? 0u : (uint32_t)last_le(m, gp0, [&](uint64_t j) { return inst[j].part_base; });
    uint64_t next_base = cur_inst + 1 < m ? inst[cur_inst + 1].part_base : ~0ull;
    bool skip = skipped(cur_inst);
    uint64_t *const xkeys = args->xkeys;
    uint32_t *const xcounts = args->xcounts;
    const uint64_t xcap = args->xcap;
    uint64_t inst_claims = 0;  // thread 0: the block's of cur_inst, not yet flushed
    uint32_t n_old = 0;        // vertices that the segment held before
    next_stage();
    plan_unit();
    __syncthreads();
    load_pair(next_units, 0);
    for (;;) {  // stages
        const uint32_t pairs = next_pairs, units = next_units;
        cs = ns;
        next_stage();
        for (uint32_t x = 0; x < pairs; ++x) {
            const bool stage_end = x + 1 == pairs;
            const uint32_t u0 = units * x, rel = s_unit[u0].gp;
            const bool seg_end = s_unit[u0].last != 0;
            const uint64_t gp = gp0 + rel;
            if (s_unit[u0].first == 0) {  // a segment starts
                if (gp >= next_base) {  // uniform: the run enters the next instance
                    if (tid == 0 && inst_claims) atomic_add_u64(&st[cur_inst].claimed, inst_claims);
                    inst_claims = 0;
                    while (gp >= next_base) {
                        ++cur_inst;
                        next_base = cur_inst + 1 < m ? inst[cur_inst + 1].part_base : ~0ull;
                    }
                    skip = skipped(cur_inst);
                }
                const Instance &in = inst[cur_inst];
                // a skipped (rejected) instance has no records and its table is left untouched
                n_old = 0;
                if (!skip && !in.fresh) {
                    const uint64_t idx = gp - in.part_base;
                    n_old = min(as_global(in.seg_count)[idx], kSegSlots);
                    seg_reinsert<RW>(in.table + idx * (uint64_t)kSegSlots * EW, n_old, s_key, s_cnt, home_mask);
                    __syncthreads();
                }
            }
            const auto take = [&](uint32_t c) {
                if (((c % kUnitRounds) * kReduceWaves + wave) * 64 + lane < n_rv[c / kUnitRounds] &&
                    !reduce_record<STATS>(rv[c], s_key, s_cnt, my_claims, home_mask, ps))
                    full = true;
            };
#pragma unroll
            for (uint32_t h = 0; h < 2; ++h) {
                if (!n_rv[h]) continue;  // uniform, as is the next: a sparse segment is a round of instructions, not eight
                take(h * kUnitRounds);
                if (n_rv[h] <= kReduceBlock) continue;
#pragma unroll
                for (uint32_t c = 1; c < kUnitRounds; ++c) take(h * kUnitRounds + c);
            }
            if (max(s_unit[u0].n, s_unit[u0 + units - 1].n) > kUnitRecords) {
                const Source &S = s_src[cs];
                for (uint32_t u = u0; u < u0 + units; ++u)
                    if (s_unit[u].n > kUnitRecords) take_rows(S, rel, s_unit[u].first, min(s_unit[u].first + S.per_unit, S.pieces));
            }
            if (full) {
                atomic_or_u32(&st[cur_inst].err, kErrFull);
                full = false;
            }
            if (seg_end) {
                const uint32_t claims = wave_scan((uint32_t)my_claims);
                if (lane == 63) s_claims[wave] = claims;
                my_claims = 0;
            }
            if (seg_end || stage_end) __syncthreads();  // every record so far is in LDS, a stage's plan has been read
            uint64_t xbase = 0;
            if (seg_end && tid == 0) {
                // fused extraction: room in the caller's arrays for the segment's
                // vertices, asked for before anything that its latency can hide behind
                uint32_t claims = 0;
                for (uint32_t w = 0; w < kReduceWaves; ++w) claims += s_claims[w];
                inst_claims += claims;
                if (xkeys && !skip)
                    xbase = __hip_atomic_fetch_add(&st[cur_inst].emitted, (uint64_t)(n_old + claims), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            if (stage_end) {
                plan_unit();
                __syncthreads();
            }
            load_pair(stage_end ? next_units : units, stage_end ? 0 : x + 1);  // (after the last pair: a stale plan's, not used)
            if (!seg_end) continue;
            const uint32_t occupied = seg_count_slots(s_key, lane, wave);
            if (lane == 0) s_wave_n[wave] = occupied;
            // the reservation has arrived once only the pair's loads are behind it; said here for
            // every wavefront, so that no later use of a register waits for the loads as well
            __builtin_amdgcn_s_waitcnt(0xf70 | 2 * kUnitRounds);
            if (tid == 0) s_xbase = xbase;
            __syncthreads();
            if (!skip) {  // uniform; a skipped instance left LDS all zero
                const Instance &in = inst[cur_inst];
                const uint64_t idx = gp - in.part_base;
                const uint32_t total = seg_store<RW>(in.table + idx * (uint64_t)kSegSlots * EW, s_key, s_cnt, s_wave_n,
                                                     lane, wave, xkeys, xcounts, xcap, s_xbase);
                if (tid == 0) as_global(in.seg_count)[idx] = total;
            }
            __syncthreads();
        }
        if (!next_pairs) break;
    }
    if (tid == 0 && inst_claims) atomic_add_u64(&st[cur_inst].claimed, inst_claims);
    if (STATS) ps.flush(args->stats);
    finish();
}

// ---------------------------------------------------------------- launches

// The tile shapes, by their records (SortBuffers::tile1, tile2).  Level 1:
// small inputs take small tiles; otherwise 64 KB of records on 512 threads,
// two workgroups a CU (378 against 460 us for 128 KB tiles at 121 M windows and
// 189 buckets: a workgroup's loads and barriers hide behind the other's
// decode), and 128 KB tiles where a first level of many buckets would leave
// pieces of a dozen records, which the next level then reads in parts of
// lines.  Level 2 has no decode and fits two workgroups of 1024 threads a CU
// when it orders its records a word at a time: 5.7 ms for 1.6 G records in 713
// segments a bucket, 6.6 ms with whole records on one workgroup; tiles of
// 32768 records (one workgroup) take 7.1 ms and give 0.6 ms back in the reduce.
template <uint32_t BLOCK, uint32_t PER, bool WORDS> struct Shape {
    static constexpr uint32_t block = BLOCK, per = PER, tile = BLOCK * PER;
    static constexpr bool words = WORDS;
};
template <uint32_t RW> struct Shapes;
template <> struct Shapes<1> {
    using Small = Shape<256, 8, false>;
    using Mid = Shape<512, 16, false>;
    using Large = Shape<1024, 16, false>;
    using Level2 = Shape<1024, 16, true>;
};
template <> struct Shapes<2> {
    using Small = Shape<256, 8, false>;
    using Mid = Shape<512, 8, false>;
    using Large = Shape<1024, 8, false>;
    using Level2 = Shape<1024, 8, true>;
};

template <uint32_t RW, typename S>
constexpr auto windows_kernel() { return &k_sort_windows<RW, S::block, S::per, S::words>; }
template <uint32_t RW, typename S>
constexpr auto bucket_kernel() { return &k_sort_bucket<RW, S::block, S::per, S::words>; }
template <uint32_t RW, typename S>
constexpr uint32_t room_of() { return tile_room(S::tile, RW, S::words); }

template <uint32_t RW, typename S>
hipError_t sort_windows(const PassArgs *args, const Instance *inst, const uint64_t *ws, InstStatus *st,
                        const SortBuffers &sb, hipStream_t s) {
    hipLaunchKernelGGL((windows_kernel<RW, S>()), dim3((uint32_t)sb.tiles1_cap), dim3(S::block),
                       sort_lds_bytes(sb.d1_max, room_of<RW, S>()), s, args, inst, ws, sb.plan, sb.tile_read, st, sb.rec1,
                       sb.off1, sb.row1, sb.d1_max);
    return hipGetLastError();
}

template <uint32_t RW>
hipError_t launch_sorted_rw(const PassArgs *args, const Instance *inst, const uint64_t *ws, InstStatus *st,
                            const SortBuffers &sb, uint64_t n_cap, bool single, bool stats, hipStream_t s,
                            hipEvent_t *marks) {
    using Sh = Shapes<RW>;
    hipError_t e;
    const auto mark = [&](int i) {
        if (marks) (void)hipEventRecord(marks[i], s);
    };
    if (!single) {  // (the window scan planned a one-instance pass)
        hipLaunchKernelGGL(k_sort_plan, dim3(1), dim3(1024), 0, s, args, inst, ws, st, sb.plan, sb.totals, sb.tile1);
        const uint32_t g = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n_cap + 255) / 256, 8192));
        hipLaunchKernelGGL(k_sort_tile_reads, dim3(g), dim3(256), 0, s, args, inst, ws, sb.plan, st, sb.tile_read,
                           sb.tile1);
    }
    mark(0);
    mark(1);  // no count
    mark(2);
    if (sb.tile1 == Sh::Small::tile) e = sort_windows<RW, typename Sh::Small>(args, inst, ws, st, sb, s);
    else if (sb.tile1 == Sh::Mid::tile) e = sort_windows<RW, typename Sh::Mid>(args, inst, ws, st, sb, s);
    else if (sb.tile1 == Sh::Large::tile) e = sort_windows<RW, typename Sh::Large>(args, inst, ws, st, sb, s);
    else return hipErrorInvalidValue;
    if (e != hipSuccess) return e;
    mark(3);
    if (sb.two_level) {
        using L2 = typename Sh::Level2;
        if (sb.tile2 != L2::tile) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_sort_transpose, dim3((uint32_t)sb.groups_cap, (sb.d1_max + 63) / 64), dim3(kTransBlock), 0, s,
                           args, inst, sb.plan, sb.off1, sb.row1, sb.offt, sb.gsum);
        hipLaunchKernelGGL(k_sort_groups, dim3((uint32_t)sb.buckets_cap), dim3(256), 0, s, args, sb.totals, sb.plan,
                           sb.gsum, sb.gpre, sb.buckets);
        hipLaunchKernelGGL(k_sort_buckets, dim3(1), dim3(1024), 0, s, sb.totals, sb.buckets, sb.tile2_base, sb.tile2);
        mark(4);
        mark(5);  // no count
        mark(6);
        hipLaunchKernelGGL((bucket_kernel<RW, L2>()), dim3((uint32_t)sb.tiles2_cap), dim3(L2::block),
                           level2_lds(sb.fan_max, L2::tile, room_of<RW, L2>()).bytes, s, sb.totals, inst, sb.plan,
                           sb.buckets, sb.tile2_base, sb.gpre, sb.offt, sb.rec1, sb.rec2, sb.off2, sb.row2, sb.fan_max,
                           sb.tile1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        mark(4);
        mark(5);
        mark(6);
    }
    mark(7);
    mark(8);
#define DBG_LAUNCH_REDUCE(EW, STATS)                                                                              \
    hipLaunchKernelGGL((k_reduce_pieces<EW, RW, STATS>), dim3(sb.grid_reduce), dim3(kReduceBlock), 0, s, args, inst, \
                       sb.plan, sb.buckets, sb.tile2_base, sb.off1, sb.off2, sb.rec1, sb.rec2, sb.row1, sb.row2,  \
                       sb.tile1, sb.tile2, st, sb.done)
    if constexpr (RW == 2) {
        if (stats) DBG_LAUNCH_REDUCE(4, true); else DBG_LAUNCH_REDUCE(4, false);
    } else if (sb.entry_words == 4) {
        if (stats) DBG_LAUNCH_REDUCE(4, true); else DBG_LAUNCH_REDUCE(4, false);
    } else {
        if (stats) DBG_LAUNCH_REDUCE(3, true); else DBG_LAUNCH_REDUCE(3, false);
    }
#undef DBG_LAUNCH_REDUCE
    return hipGetLastError();
}

template <typename K>
uint32_t resident(K kernel, int device, uint64_t cap) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, (int)kReduceBlock, 0) != hipSuccess || per <= 0)
        per = 1;
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((uint64_t)cus * per, cap));
}

}  // namespace

hipError_t launch_sorted(const PassArgs *args, const Instance *inst, const uint64_t *ws, InstStatus *st,
                         const SortBuffers &sb, uint64_t n_cap, bool single, bool stats, hipStream_t s,
                         hipEvent_t *marks) {
    if (sb.rec_words == 2) return launch_sorted_rw<2>(args, inst, ws, st, sb, n_cap, single, stats, s, marks);
    return launch_sorted_rw<1>(args, inst, ws, st, sb, n_cap, single, stats, s, marks);
}

// Dynamic LDS limits of the kernels (process-wide, so always the most any
// table needs) and the reduce's resident grid.
namespace {
template <uint32_t RW, typename S>
void allow_windows() {
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(windows_kernel<RW, S>()),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)sort_lds_bytes(kMaxD1, room_of<RW, S>()));
}

template <uint32_t RW>
void allow_all() {
    using Sh = Shapes<RW>;
    using L2 = typename Sh::Level2;
    allow_windows<RW, typename Sh::Small>();
    allow_windows<RW, typename Sh::Mid>();
    allow_windows<RW, typename Sh::Large>();
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(bucket_kernel<RW, L2>()),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)level2_lds(kMaxFan, L2::tile, room_of<RW, L2>()).bytes);
}
}  // namespace

void sorted_grids(int device, SortBuffers &sb) {
    if (sb.rec_words == 2) {
        allow_all<2>();
        sb.grid_reduce = resident(k_reduce_pieces<4, 2, false>, device, sb.parts_cap);
    } else {
        allow_all<1>();
        sb.grid_reduce = sb.entry_words == 4 ? resident(k_reduce_pieces<4, 1, false>, device, sb.parts_cap)
                                             : resident(k_reduce_pieces<3, 1, false>, device, sb.parts_cap);
    }
}

}  // namespace dbgk
