// Window records of the binned build, their claims in an LDS segment, and the
// segment's way back to the table (internal header, shared by the partition
// kernels of dbg_binned.hip and dbg_sorted.hip).
#pragma once

#include "dbg_device.h"

namespace dbgk {

constexpr uint32_t kSkipMask = kErrBase | kErrInval | kErrRange | kErrSkip;
static_assert((kSegSlots & (kSegSlots - 1)) == 0, "segment size must be a power of two");

__device__ __forceinline__ uint64_t lds_load64(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint32_t lds_add32(uint32_t *p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Long keys (33 <= k <= 63, so K < 2^124) as (kh = K >> 64 < 2^60, kl):
// two Feistel rounds give the image (ih < 2^60, il): il = kl ^ mix64(kh),
// then ih = kh ^ (il * kWideMul) >> 4.  ih takes the place of a short key's
// image (its top bits are the segment digits) and il's low bits are the
// home slot; each round undoes itself given the other half.
constexpr uint64_t kWideMul = 0xD1B54A32D192ED03ull;  // odd

__device__ __forceinline__ void wide_image(uint64_t kh, uint64_t kl, uint64_t &ih, uint64_t &il) {
    il = kl ^ mix64(kh);
    ih = kh ^ ((il * kWideMul) >> 4);
}

__device__ __forceinline__ void wide_key(uint64_t ih, uint64_t il, uint64_t &kh, uint64_t &kl) {
    kh = ih ^ ((il * kWideMul) >> 4);
    kl = il ^ mix64(kh);
}

// A window record: RW = 1, one word image << 3 | sink << 2 | letter; RW = 2
// (long keys), that word built from ih, then il.  Both start with the word
// that carries the segment digits and the flags.
template <uint32_t RW> struct RecOf;
template <> struct RecOf<1> {
    using T = uint64_t;
    static __device__ __forceinline__ uint64_t head(uint64_t r) { return r; }
    static __device__ __forceinline__ uint64_t none() { return ~0ull; }
};
template <> struct RecOf<2> {
    using T = ulonglong2;
    static __device__ __forceinline__ uint64_t head(ulonglong2 r) { return r.x; }
    static __device__ __forceinline__ ulonglong2 none() { return make_ulonglong2(~0ull, 0); }
};


// Last index i in [0, n) with base(i) <= x, for a non-decreasing base.
template <typename F>
__device__ __forceinline__ uint64_t last_le(uint64_t n, uint64_t x, F base) {
    uint64_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint64_t mid = (lo + hi) >> 1;
        if (base(mid) <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// 64 bits starting `o` bits into the 192-bit big-endian word triple (o < 128).
__device__ __forceinline__ uint64_t funnel3(uint64_t a, uint64_t b, uint64_t c, uint32_t o) {
    if (o >= 64) {
        a = b;
        b = c;
        o -= 64;
    }
    return o ? (a << o) | (b >> (64 - o)) : a;
}

// Rolling window state of one-word keys (k <= 31).  Consecutive windows of a
// read share all but one base: the key of the next window is the key shifted
// by one base, with the window's letter shifted in and its first base shifted
// out.  The image multiplies the key by kKeyMul modulo 2^60, so with
// x = key * kKeyMul mod 2^60 the next window's x is
//   4 x + letter * kKeyMul - first * (4^(k-1) * kKeyMul)  (mod 2^60),
// one shift-add of a table entry indexed by (first base, letter).  F holds
// the 32 bases from the window's first on, L the 32 from its letter on, so a
// thread rolls through up to 32 windows of one read without touching the
// packed reads again.
struct Roll {
    uint64_t F, L, x;
};

// The state of the window whose first base is at position p of the packed
// reads.  kshift = 64 - 2 (k - 1).
__device__ __forceinline__ Roll roll_at(const uint64_t *__restrict__ packed, uint64_t p, uint32_t k,
                                        uint32_t kshift) {
    const uint64_t wb = p >> 5;
    const uint64_t a = packed[wb], b = packed[wb + 1], c = packed[wb + 2];
    const uint32_t o = (uint32_t)(p & 31) * 2;  // o + 2 (k - 1) <= 122: inside the triple
    const uint64_t F = funnel3(a, b, c, o);
    return Roll{F, funnel3(a, b, c, o + 2 * (k - 1)), ((F >> kshift) * kKeyMul) & kKey60};
}

// Table entry (first << 2 | letter): letter * kKeyMul - first * 4^(k-1) * kKeyMul, mod 2^60.
__device__ __forceinline__ uint64_t roll_entry(uint32_t e, uint32_t k) {
    const uint64_t out = (kKeyMul << (2 * (k - 1))) & kKey60;
    return ((uint64_t)(e & 3u) * kKeyMul - (uint64_t)(e >> 2) * out) & kKey60;
}

__device__ __forceinline__ void roll_next(Roll &r, const uint64_t *s_roll) {
    const uint32_t e = (uint32_t)(r.F >> 62) << 2 | (uint32_t)(r.L >> 62);
    r.F <<= 2;
    r.L <<= 2;
    r.x = ((r.x << 2) + s_roll[e]) & kKey60;
}

__host__ __device__ inline uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }

// Sum of v over the block; thread 0 adds it to *dst.  Whole block.
__device__ inline void flush_block_sum(uint64_t v, uint64_t *dst, uint64_t *s_sum) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (threadIdx.x == 0) *s_sum = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0 && v)
        __hip_atomic_fetch_add(s_sum, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (threadIdx.x == 0 && *s_sum) atomic_add_u64(dst, *s_sum);
    __syncthreads();
}

constexpr uint32_t kReducePrefetch = 8;  // records a thread loads before using them
constexpr uint64_t kNoRecord = ~0ull;     // no record: a record's first word stays below 2^63

// Find-or-claim one record's vertex in the LDS segment and count its letter.
// Returns false when the segment has no free slot for it.
// home_mask: kSegSlots - 1, or 7 with the test hash (every key of a segment
// then starts at one of its first eight slots).
template <bool STATS>
__device__ __forceinline__ bool reduce_record(uint64_t rec, uint64_t *s_key, uint32_t *s_cnt,
                                              uint64_t &claims, uint32_t home_mask, ProbeStats &ps) {
    const uint64_t img = rec >> 3;
    const uint64_t tagv = img | kOccupied;
    uint32_t s = seg_home(img) & home_mask;
    uint32_t q = 0;
    if constexpr (!STATS) {
        // Each probe is one compare-and-swap of an empty slot to this key: it
        // claims the slot if empty and otherwise returns the key it holds, so
        // the loop has one exit test and no nested branch (10 % less reduce
        // time than a load followed by a CAS on empty slots).  The statistics
        // build below keeps the load, so that a CAS it issues is one that
        // expected an empty slot and a failed one is a lost race.
        uint64_t old;
        for (;;) {
            old = 0;
            __hip_atomic_compare_exchange_strong(&s_key[s], &old, tagv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
            if (old == 0 || old == tagv) break;
            if (++q == kSegSlots) return false;
            s = (s + 1) & (kSegSlots - 1);
        }
        claims += old == 0 ? 1u : 0u;
        if (!(rec & 4)) lds_add32(&s_cnt[4 * s + (uint32_t)(rec & 3)], 1u);
        return true;
    }
    uint64_t cur = lds_load64(&s_key[s]);
    // probe until the slot holds this key (found, or claimed here); the count
    // is added once, after the loop
    for (;;) {
        if (cur == 0) {
            uint64_t expected = 0;
            __hip_atomic_compare_exchange_strong(&s_key[s], &expected, tagv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
            if (STATS) {
                ++ps.cas;
                ps.lost += expected != 0 ? 1u : 0u;
            }
            if (expected == 0) {
                ++claims;
                break;
            }
            cur = expected;
        }
        if (cur == tagv) break;
        if (++q == kSegSlots) return false;
        s = (s + 1) & (kSegSlots - 1);
        cur = lds_load64(&s_key[s]);
    }
    if (STATS) ps.lookup(q + 1);
    if (!(rec & 4)) lds_add32(&s_cnt[4 * s + (uint32_t)(rec & 3)], 1u);
    return true;
}

// Long keys: a slot's key is two LDS words, hi (ih | kOccupied) and lo (il).
// A slot is claimed by the CAS of hi; the claimer then stores lo and sets
// kReady in hi.  A lane that finds its own hi without kReady has met a claim
// in flight and reads the slot again (the claimer waits on nothing between
// its CAS and those stores); with kReady set, lo decides whether the slot
// is this key's.  Returns the slot, or kSegSlots when none is found.
constexpr uint64_t kReady = 1ull << 62;
constexpr uint32_t kMaxInFlightReads = 1u << 20;

template <bool STATS>
__device__ __forceinline__ uint32_t wide_slot(uint64_t tag, uint64_t lo, uint64_t *s_hi, uint64_t *s_lo,
                                              bool &claimed, uint32_t home_mask, ProbeStats &ps) {
    uint32_t s = seg_home(lo) & home_mask, waits = 0;
    for (uint32_t q = 0;;) {
        uint64_t cur = __hip_atomic_load(&s_hi[s], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == 0) {
            uint64_t expected = 0;
            __hip_atomic_compare_exchange_strong(&s_hi[s], &expected, tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
            if (STATS) {
                ++ps.cas;
                ps.lost += expected != 0 ? 1u : 0u;
            }
            if (expected == 0) {
                __hip_atomic_store(&s_lo[s], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_store(&s_hi[s], tag | kReady, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                claimed = true;
                if (STATS) ps.lookup(q + 1);
                return s;
            }
            cur = expected;
        }
        if ((cur & ~kReady) == tag) {
            if (!(cur & kReady)) {  // claim in flight: read the slot again
                if (++waits > kMaxInFlightReads) return kSegSlots;
                continue;
            }
            if (lds_load64(&s_lo[s]) == lo) {
                if (STATS) ps.lookup(q + 1);
                return s;
            }
        }
        if (++q == kSegSlots) return kSegSlots;
        s = (s + 1) & (kSegSlots - 1);
    }
}

template <bool STATS>
__device__ __forceinline__ bool reduce_record(ulonglong2 rec, uint64_t *s_key, uint32_t *s_cnt, uint64_t &claims,
                                              uint32_t home_mask, ProbeStats &ps) {
    bool claimed = false;
    const uint32_t s =
        wide_slot<STATS>((rec.x >> 3) | kOccupied, rec.y, s_key, s_key + kSegSlots, claimed, home_mask, ps);
    if (s == kSegSlots) return false;
    claims += claimed ? 1u : 0u;
    if (!(rec.x & 4)) lds_add32(&s_cnt[4 * s + (uint32_t)(rec.x & 3)], 1u);
    return true;
}

// ---------------------------------------------------------------- segments in LDS and in the table

static_assert(kSegSlots % kReduceBlock == 0 && kReduceBlock % 64 == 0, "slot ranges per wavefront");
constexpr uint32_t kReduceWaves = kReduceBlock / 64;
constexpr uint32_t kWaveSlots = kSegSlots / kReduceWaves;  // slots compacted by one wavefront

// Put the n_old vertices that the table's segment holds back into the LDS
// slots (not counted in any probe statistics).  Whole block, no barrier.
template <uint32_t RW>
__device__ __forceinline__ void seg_reinsert(const uint64_t *seg, uint32_t n_old, uint64_t *s_key, uint32_t *s_cnt,
                                             uint32_t home_mask) {
    seg = as_global(seg);
    for (uint32_t e = threadIdx.x; e < n_old; e += kReduceBlock) {
        // distinct keys: each claims its own slot, and nobody else touches
        // that slot's counters before the next barrier
        const uint64_t tagv = seg[e];
        const uint4 cv = seg_counts<RW>(seg)[e];
        if constexpr (RW == 2) {
            bool claimed = false;
            ProbeStats none;
            const uint32_t s =
                wide_slot<false>(tagv, seg[kSegSlots + e], s_key, s_key + kSegSlots, claimed, home_mask, none);
            if (s < kSegSlots) reinterpret_cast<uint4 *>(s_cnt)[s] = cv;
            continue;
        }
        uint32_t s = seg_home(tagv) & home_mask;
        for (uint32_t q = 0; q < kSegSlots; ++q) {
            uint64_t expected = 0;
            if (__hip_atomic_compare_exchange_strong(&s_key[s], &expected, tagv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP)) {
                reinterpret_cast<uint4 *>(s_cnt)[s] = cv;
                break;
            }
            s = (s + 1) & (kSegSlots - 1);
        }
    }
}

// Occupied slots in this wavefront's range of the segment.
__device__ __forceinline__ uint32_t seg_count_slots(const uint64_t *s_key, uint32_t lane, uint32_t wave) {
    uint32_t mine = 0;
    for (uint32_t c = 0; c < kWaveSlots; c += 64)
        mine += (uint32_t)__popcll(__ballot(s_key[wave * kWaveSlots + c + lane] != 0));
    return mine;
}

// Two key words of the caller's, whose array may start at any word.
using Keys2 = uint64_t __attribute__((ext_vector_type(2), aligned(8)));

// Write this wavefront's occupied slots to the table's segment, packed, and
// zero them; with xkeys also, as keys and counters, to the caller's arrays from
// xbase on, which the caller has reserved for the whole segment.  s_wave_n:
// seg_count_slots of every wavefront, behind a barrier.  Returns the segment's
// vertices.  No barrier; the next use of the LDS slots waits on one.
template <uint32_t RW>
__device__ __forceinline__ uint32_t seg_store(uint64_t *seg, uint64_t *s_key, uint32_t *s_cnt, const uint32_t *s_wave_n,
                                              uint32_t lane, uint32_t wave, uint64_t *__restrict__ xkeys,
                                              uint32_t *__restrict__ xcnt, uint64_t xcap, uint64_t xbase) {
    seg = as_global(seg);
    xkeys = as_global(xkeys);
    uint4 *__restrict__ xcounts = reinterpret_cast<uint4 *>(as_global(xcnt));
    const uint32_t nw = lane < kReduceWaves ? s_wave_n[lane] : 0u, waves = wave_scan(nw);
    const uint32_t total = __builtin_amdgcn_readlane(waves, 63);
    uint32_t out = __builtin_amdgcn_readlane(waves - nw, __builtin_amdgcn_readfirstlane(wave));
#pragma unroll
    for (uint32_t c = 0; c < kWaveSlots; c += 64) {
        const uint32_t s = wave * kWaveSlots + c + lane;
        const uint64_t tagv = s_key[s];
        const uint64_t mask = __ballot(tagv != 0);
        if (tagv) {
            const uint32_t to = out + (uint32_t)__popcll(mask & ((1ull << lane) - 1));
            const uint4 cnt = reinterpret_cast<const uint4 *>(s_cnt)[s];
            uint64_t low = 0;
            if constexpr (RW == 2) low = s_key[kSegSlots + s];
            s_key[s] = 0;
            reinterpret_cast<uint4 *>(s_cnt)[s] = make_uint4(0, 0, 0, 0);
            seg[to] = tagv & ~kReady;
            if constexpr (RW == 2) seg[kSegSlots + to] = low;
            seg_counts<RW>(seg)[to] = cnt;
            const uint64_t o = xbase + to;
            if (xkeys && o < xcap) {
                if constexpr (RW == 1) {
                    xkeys[o] = key_of_image(tagv & ~kOccupied);
                } else {  // two key words per record: K >> 64, K mod 2^64
                    uint64_t kh, kl;
                    wide_key(tagv & ~(kOccupied | kReady), low, kh, kl);
                    *reinterpret_cast<Keys2 *>(xkeys + 2 * o) = Keys2{kh, kl};
                }
                xcounts[o] = cnt;
            }
        }
        out += (uint32_t)__popcll(mask);
    }
    return total;
}

}  // namespace dbgk
