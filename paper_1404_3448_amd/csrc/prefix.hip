// Suffix array by sorting prefixes, for the texts of the library on gfx950.
//
// DC3 sorts a text of any structure in O(n), but on DNA nearly every suffix
// is told from all others by a few dozen symbols, and DC3 still pays for its
// levels: about two dozen passes over (shrinking) arrays, a gather per merged
// suffix and a read-back per level. Here the same (unique) order is built as
//   keys   : the first K symbols of every suffix packed in at most 32 bits;
//   sort   : LSD radix passes over (key, position), 1 to 4 of them;
//   resolve: suffixes with equal keys are neighbours now. A group of up to
//            kSmall of them is ordered inside one workgroup: 8 more text
//            bytes per member are gathered into LDS and a member's place is
//            the number of smaller ones; runs that still agree stay open;
//   groups : larger groups (short tandem repeats, mostly) are collected and
//            radix sorted by a key that sees through a repeat. Let t be the
//            period of the group's K symbols and e the first place where a
//            suffix breaks that period. Of two suffixes of the group the one
//            that breaks first is smaller if it breaks downwards (to a smaller
//            symbol than the period asks for) and larger otherwise; of two
//            that break at the same place and in the same direction the
//            symbols from there on decide. So (direction and e, next symbols)
//            orders a repeat of any length in one sort.
//   settle : the members of open runs compare their texts.
// Suffixes that come within K symbols of their sequence's separator ("near"
// suffixes, at most K per sequence) would need keys with separators in them;
// they are left out of the sort and merged in afterwards (k_merge).
//
// Measured against DC3 on the same texts (whole call, SA + LCP + ISA +
// overlap): two sequences of 600 and 431 bases 1.34 -> 0.16 ms, 50k + 50k
// 2.60 -> 0.19 ms, 8M + 8M noncoding-like 7.45 -> 1.71 ms, 16 x 2^26
// 248 -> 83 ms. Of the 83 ms the key passes stream 20 (4.1 TB/s), and random
// reads, at the 45 to 55 G/s that they reach, take 10 here and 19 in the LCP.
//
// Suffixes that still agree after kDeep symbols (long exact or nearly exact
// copies) are ordered by doubling: by the rank of the suffix h symbols on, h
// doubling from round to round. Two sequences of 2M bases with 0.1% mutations
// take 1.3 ms (DC3 4.2 ms), two identical ones 2.7 ms (6.4 ms).
//
// Groups that stay large (words with more than kSmall copies) are doubled as well,
// by sorts of (group, rank of the suffix h symbols on).
//
// Texts whose suffixes are mostly in large groups (one repeat all through) or
// would take more sorts than DC3 is worth, and workspaces that do not hold them,
// are DC3's: the caller then runs it. 2M + 2M equal bases: 4.6 ms (4.7 ms by DC3
// alone).
#include <stdio.h>

#include <algorithm>
#include <memory>
#include <new>

#include "lor_internal.hpp"

namespace lor {

namespace {

constexpr int kWordAbort = 6;      // header words of this file (see WsHeader)
constexpr int kWordTied = 3;       // suffixes in large groups
constexpr int kWordHeads = 4;      // large groups (next to kWordTied: cleared together)
constexpr int kWordOpen = 7;       // suffixes still equal to their neighbour, after resolve
constexpr int kWordRound = 8;      // the same after rounds of doubling
constexpr int kWordItems = 14;     // items of the run list
constexpr int kWordSpent = 5;      // comparison budget used, in units of kUnit steps

constexpr uint32_t kSmall = 64;               // largest group resolved in a workgroup
// Ranks per thread of the resolve kernels: few per thread for small inputs,
// whose time is one workgroup's chain of waits (and its instruction fetches).
constexpr int kResItems = 4, kResItemsSmall = 1;
constexpr uint32_t kResSmall = 1u << 18;      // inputs up to here count as small
constexpr uint32_t kDeep = 256;               // symbols that k_settle compares: many open suffixes,
constexpr uint32_t kSettle = 2048;            // and few
constexpr uint32_t kUnit = 32;                // 32-byte comparison steps per budget unit
constexpr uint32_t kCodeBits = 15;
constexpr uint32_t kExtent = (1u << (kCodeBits - 1)) - 1u;   // longest repeat a key describes
constexpr uint32_t kRepeatSymbols = (64 - kCodeBits) / 3;    // next symbols of resolve's repeat keys
constexpr uint32_t kRepeat = 16;              // symbols of a repeat bit, less one (see mark_runs)
constexpr uint32_t kKeyTile = 2048;           // positions per workgroup of the key kernels
// Texts up to here take every slot as an item and settle without waiting to
// hear whether anything is open: a read-back and the list's three launches cost
// more than looking at 2^21 run bits (10 us).
constexpr uint32_t kIdentityItems = 1u << 21;
constexpr uint32_t kDirectRanks = 1u << 24;   // ranks as plain stores up to here (see kDirectIsa)
constexpr int kMaxRounds = 4;                 // sorts of large groups by their next symbols, at most
// What the sorts of large groups may cost before DC3 takes over, counted in sorted
// suffixes (see Spend): one per member, and kRoundCost for a round's launches.
constexpr uint64_t kRoundCost = 1u << 19, kLeastSpend = 3u << 23;
constexpr int kMaxK = 16;
constexpr uint32_t kScan = 4;                 // group members read from LDS together

// ------------------------------------------------------------ text access

using dev::Bytes16;
struct __attribute__((packed, aligned(1))) Bytes8 {
    uint32_t x, y;
};

__device__ __forceinline__ uint64_t be64(uint32_t a, uint32_t b, uint8_t) {
    return ((uint64_t)__builtin_bswap32(a) << 32) | __builtin_bswap32(b);
}
__device__ __forceinline__ uint64_t be64(uint32_t a, uint32_t b, uint16_t) {
    return ((uint64_t)((a << 16) | (a >> 16)) << 32) | ((b << 16) | (b >> 16));
}

// 16 text bytes from symbol i on, in comparison order (first symbol most
// significant); symbols past the end read 0.
template <typename CH>
__device__ __forceinline__ void window(const CH *__restrict__ t, uint32_t n, uint32_t i, uint64_t *hi, uint64_t *lo) {
    constexpr uint32_t W = 16 / sizeof(CH);
    if (i < n && W <= n - i) {
        const Bytes16 v = *reinterpret_cast<const Bytes16 *>(t + i);
        *hi = be64(v.x, v.y, CH());
        *lo = be64(v.z, v.w, CH());
        return;
    }
    uint64_t h = 0, l = 0;
    for (uint32_t c = 0; c < W; ++c) {
        const uint64_t x = (i < n && c < n - i) ? (uint64_t)t[i + c] : 0ull;
        if (c < W / 2) h = (h << (8 * sizeof(CH))) | x;
        else l = (l << (8 * sizeof(CH))) | x;
    }
    *hi = h;
    *lo = l;
}

// The first 8 of those bytes.
template <typename CH>
__device__ __forceinline__ uint64_t window8(const CH *__restrict__ t, uint32_t n, uint32_t i) {
    constexpr uint32_t W = 8 / sizeof(CH);
    if (i < n && W <= n - i) {
        const Bytes8 v = *reinterpret_cast<const Bytes8 *>(t + i);
        return be64(v.x, v.y, CH());
    }
    uint64_t h = 0;
    for (uint32_t c = 0; c < W; ++c) h = (h << (8 * sizeof(CH))) | ((i < n && c < n - i) ? (uint64_t)t[i + c] : 0ull);
    return h;
}

// A budget for long comparisons: every kUnit steps a lane draws one unit, and
// gives up when they are spent (the call then goes to DC3).
struct Budget {
    uint32_t *hdr;
    uint32_t units;
    uint32_t steps = 0;
    __device__ bool operator()() {
        if ((++steps % kUnit) != 0) return false;
        const uint64_t m = __ballot(1);
        const int lead = __builtin_ctzll(m);
        uint32_t got = 0;
        if ((int)dev::lane_id() == lead) got = atomicAdd(&hdr[kWordSpent], (uint32_t)__popcll(m));
        got = (uint32_t)__shfl((int)got, lead, kWave);
        if (got > units) {
            hdr[kWordAbort] = 1;
            return true;
        }
        return __hip_atomic_load(&hdr[kWordAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
};

// Refines classes of equal suffixes in LDS, one slot per thread: thread l has
// slot l, whose suffix val[l] is in a group of slots [f, f + size). cls[l] is the
// first place of its class, which lies inside the group, key[l] >> 32 the symbols
// that the class shares. In every step the members of a class compare their texts
// with its first member: a member that differs after L symbols comes before it,
// the shorter L the earlier, or after it, the shorter L the later; equal (L,
// direction) form the classes of the next step. One comparison per member and
// step, instead of one per pair: members of one tandem repeat all part in the
// first step. A member that shares max(deep, shared + 64) symbols with the first
// stays in its class for good. All threads of the workgroup call this; `again`:
// whether the thread's slot is in a class to refine.
template <typename CH>
__device__ __forceinline__ void refine(const CH *__restrict__ t, uint32_t n, uint32_t deep, uint32_t f, uint32_t size,
                                       const uint32_t *val, uint64_t *key, uint16_t *cls, bool again) {
    constexpr uint32_t kEqual = 0x40000000u, kTop = 0x7fffffffu;
    const uint32_t l = threadIdx.x;
    while (__syncthreads_or(again)) {
        uint16_t c = 0;
        uint32_t mine = 0;
        if (again) {
            c = cls[l];
            uint32_t first = l;
            for (uint32_t q = f; q < l; q += kScan) {
                uint16_t x[kScan];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) x[i] = cls[min(q + i, l)];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i)
                    if (x[i] == c) first = min(first, min(q + i, l));
                if (first < l) break;
            }
            mine = kEqual;
            if (first != l) {
                const uint32_t p = val[l], q = val[first], h = (uint32_t)(key[l] >> 32), cap = max(deep, h + 64u);
                const uint32_t L = dev::extend<CH, 2>(t, n, p, q, h, cap);
                if (L < cap) {
                    const bool less = L >= n - max(p, q) ? p > q : t[p + L] < t[q + L];
                    mine = less ? L : kTop - L;
                }
            }
            key[l] = (key[l] & 0xffffffff00000000ull) | mine;
        }
        __syncthreads();
        uint32_t less = 0, same = 0;
        if (again) {
            for (uint32_t q = f; q < f + size; q += kScan) {
                uint16_t x[kScan];
                uint32_t y[kScan];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) {
                    const uint32_t o = min(q + i, f + size - 1u);
                    x[i] = q + i < f + size ? cls[o] : (uint16_t)0xffffu;
                    y[i] = (uint32_t)key[o];
                }
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) {
                    less += x[i] == c && y[i] < mine;
                    same += x[i] == c && y[i] == mine;
                }
            }
        }
        __syncthreads();
        if (again) {
            cls[l] = (uint16_t)(c + less);
            if (mine != kEqual) key[l] = (uint64_t)(mine < kEqual ? mine : kTop - mine) << 32;
            again = same > 1 && mine != kEqual;
        }
    }
}

// ------------------------------------------------------------------ texts
// What the kernels need to know of a text: its symbols, how a suffix's first
// K symbols make a key, and where its near suffixes are.
//
// Joined: up to kMaxSeqs sequences, unique separators above every base. Key:
//   two bits per base.
// Tagged: the batched path's text (symbol = 8 * pair + code; codes 1..4 bases,
//   5 and 6 separators). Key: the pair, then two bits per base.
// Shared: a reference and its queries, one separator symbol for all, so a
//   suffix reads on past it. Key: K symbols base 5; no near suffixes.
struct Joined {
    using CH = uint8_t;
    const uint8_t *t;
    uint32_t n;
    int K;
    uint32_t k;                          // sequences
    uint32_t near;                       // near suffixes in total
    int32_t start[kMaxSeqs + 1];         // joined start of every sequence, plus n
    uint32_t *rep;                       // repeat bits (see mark_runs)
    static constexpr bool kRepeatBits = true;
};
struct Tagged {
    using CH = uint16_t;
    const uint16_t *t;
    uint32_t n;
    int K;
    uint32_t k;                          // pairs
    uint32_t near;
    const int32_t *start, *alen;         // joined start of every pair (plus n), |A|
    const uint32_t *below;               // near suffixes in the pairs before
    uint32_t *rep;
    static constexpr bool kRepeatBits = true;
};
struct Shared {
    using CH = uint8_t;
    const uint8_t *t;
    uint32_t n;
    int K;
    uint32_t *rep;   // none: its repeats may run through separators
    static constexpr bool kRepeatBits = false;
};

__host__ __device__ __forceinline__ uint32_t near_of(uint32_t len, int K) {   // of one sequence and its separator
    return (len < (uint32_t)K - 1u ? len : (uint32_t)K - 1u) + 1u;
}

// Order-keeping small codes of a symbol: 0 past the end, bases 1..4, separator 5.
__device__ __forceinline__ uint32_t code3(uint8_t c) { return c < 4u ? (uint32_t)c + 1u : 5u; }
__device__ __forceinline__ uint32_t code3(uint16_t c) { return min((uint32_t)c & 7u, 5u); }

// ------------------------------------------------------------------- keys
// One workgroup per kKeyTile positions. The tile's symbols are packed once
// into 2-bit words in LDS (16 symbols a word, first symbol on top), so a
// position's key is a funnel shift of two words; keys and positions leave in
// position order with the near suffixes left out.
constexpr uint32_t kKeyWords = kKeyTile / 16 + 2;

__device__ __forceinline__ uint32_t pack4(uint32_t w) {   // 4 byte symbols -> 8 bits, first on top
    return ((w & 0x03030303u) * 0x40100401u) >> 24;
}

// The packed tile, and its symbols' bits apart: symbol i of the tile has bit i
// of three planes (high bit, low bit, no base), for mark_runs().
struct KeyTile {
    uint32_t w[kKeyWords];
    alignas(8) uint16_t hi[kKeyWords], lo[kKeyWords], no[kKeyWords];
};

__device__ __forceinline__ uint32_t even_bits(uint32_t v) {   // bits 0, 2, 4.. -> 0, 1, 2..
    v &= 0x55555555u;
    v = (v | (v >> 1)) & 0x33333333u;
    v = (v | (v >> 2)) & 0x0f0f0f0fu;
    v = (v | (v >> 4)) & 0x00ff00ffu;
    return (v | (v >> 8)) & 0xffffu;
}

__device__ __forceinline__ void put_word(KeyTile *s, uint32_t i, uint32_t v, uint32_t no) {
    s->w[i] = v;
    const uint32_t r = __builtin_bitreverse32(v);   // the first symbol's high bit lowest
    s->hi[i] = (uint16_t)even_bits(r);
    s->lo[i] = (uint16_t)even_bits(r >> 1);
    s->no[i] = (uint16_t)no;
}

__device__ __forceinline__ void pack_tile(const Joined &x, uint32_t base, KeyTile *s) {
    for (uint32_t i = threadIdx.x; i < kKeyWords; i += kBlock) {
        const uint32_t p = base + 16 * i;
        uint32_t v = 0, no = 0;
        if (p < x.n && x.n - p >= 16) {   // p is a multiple of 16, the text 4-byte aligned
            const uint32_t *w = reinterpret_cast<const uint32_t *>(x.t + p);
            v = (pack4(w[0]) << 24) | (pack4(w[1]) << 16) | (pack4(w[2]) << 8) | pack4(w[3]);
            if ((w[0] | w[1] | w[2] | w[3]) & 0xfcfcfcfcu)
                for (uint32_t c = 0; c < 16; ++c) no |= ((w[c >> 2] >> (8 * (c & 3u))) & 0xfcu ? 1u : 0u) << c;
        } else {
            for (uint32_t c = 0; c < 16; ++c) {
                const uint32_t y = p < x.n && c < x.n - p ? x.t[p + c] : 4u;
                v = (v << 2) | (y & 3u);
                no |= (y > 3u ? 1u : 0u) << c;
            }
        }
        put_word(s, i, v, no);
    }
}

__device__ __forceinline__ void pack_tile(const Tagged &x, uint32_t base, KeyTile *s) {
    for (uint32_t i = threadIdx.x; i < kKeyWords; i += kBlock) {
        const uint32_t p = base + 16 * i;
        uint32_t v = 0, no = 0;
        if (p < x.n && x.n - p >= 16) {   // the text is 256-byte aligned
            const uint32_t *w = reinterpret_cast<const uint32_t *>(x.t + p);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t y0 = (w[c] & 7u) - 1u, y1 = (w[c] >> 16 & 7u) - 1u;
                v = (v << 4) | ((y0 & 3u) << 2) | (y1 & 3u);
                no |= (((y0 >> 2) & 1u) | ((y1 >> 1) & 2u)) << (2 * c);
            }
        } else {
            for (uint32_t c = 0; c < 16; ++c) {
                const uint32_t y = p < x.n && c < x.n - p ? (x.t[p + c] & 7u) - 1u : 4u;
                v = (v << 2) | (y & 3u);
                no |= ((y >> 2) & 1u) << c;
            }
        }
        put_word(s, i, v, no);
    }
}

// Repeat bits: bit p is set when the M + 1 symbols from p on are bases and have
// a period of at most M / 2, M = kRepeat. Two such periods of M symbols have
// their greatest common divisor as a period too (Fine and Wilf, 1965), so along
// a run of set bits the smallest period stays the same, and a suffix q whose
// first M symbols have a smallest period t <= M / 2 keeps it for exactly M + r
// symbols, r the number of set bits from q on. A word of 32 positions per thread
// and period, over bit planes; the waves take the periods in turn (1.85 -> 2.03 ms
// for the keys of 1G suffixes).
__device__ __forceinline__ uint64_t any_of(uint64_t d, uint32_t width) {   // bit i: any of bits i..i + width - 1
    uint32_t have = 1;
    for (; 2 * have <= width; have *= 2) d |= d >> have;
    return d | (d >> (width - have));
}

__device__ __forceinline__ void mark_runs(const KeyTile &s, uint32_t *s_rep, uint32_t n, uint32_t base,
                                          uint32_t *__restrict__ rep) {
    constexpr uint32_t kWords = kKeyTile / 32u, kWaves = kBlock / kWave;
    static_assert(kWords == kWave, "one lane per word");
    const uint32_t j = threadIdx.x % kWords;
    auto plane = [&](const uint16_t *a) {
        const uint32_t *w = reinterpret_cast<const uint32_t *>(a) + j;
        return ((uint64_t)w[1] << 32) | w[0];
    };
    const uint64_t hi = plane(s.hi), lo = plane(s.lo);
    uint32_t set = 0;
    for (uint32_t t = 1 + threadIdx.x / kWords; t <= kRepeat / 2u; t += kWaves)
        set |= ~(uint32_t)any_of((hi ^ (hi >> t)) | (lo ^ (lo >> t)), kRepeat + 1u - t);
    if (set) {
        set &= ~(uint32_t)any_of(plane(s.no), kRepeat + 1u);
        if (set) atomicOr(&s_rep[j], set);
    }
    __syncthreads();
    const uint32_t w = base / 32u + threadIdx.x;
    if (threadIdx.x < kWords && w < (n + 31u) / 32u) rep[w] = s_rep[threadIdx.x];
}

// Largest j in [0, count) with start[j] <= x.
__device__ __forceinline__ uint32_t seq_of(const int32_t *start, uint32_t count, uint32_t x) {
    uint32_t lo = 0, hi = count - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if ((uint32_t)start[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The kernels also clear the tile's words of the run bits (see RunList).
struct OpenBits {
    uint32_t *open, *was;   // was may be null
};
__device__ __forceinline__ void clear_open(const OpenBits &o, uint32_t n, uint32_t base) {
    const uint32_t i = base / 32u + threadIdx.x;
    if (threadIdx.x >= kKeyTile / 32u || i >= (n + 31u) / 32u) return;
    o.open[i] = 0;
    if (o.was) o.was[i] = 0;
}

__global__ __launch_bounds__(kBlock) void k_prefix_keys(Joined x, uint32_t *__restrict__ keys,
                                                        uint32_t *__restrict__ vals, OpenBits open) {
    __shared__ KeyTile s_tile;
    __shared__ uint32_t s_rep[kKeyTile / 32];
    __shared__ int32_t s_start[kMaxSeqs + 1];
    __shared__ uint32_t s_below[kMaxSeqs + 1];
    __shared__ uint32_t s_tmp[kBlock / kWave];
    const uint32_t base = blockIdx.x * kKeyTile, tid = threadIdx.x;
    static_assert(kMaxSeqs < kBlock, "one thread per sequence");
    uint32_t mine = 0, all;
    if (tid <= x.k) s_start[tid] = x.start[tid];
    if (tid < x.k) mine = near_of((uint32_t)(x.start[tid + 1] - x.start[tid]) - 1u, x.K);
    const uint32_t bel = dev::block_exclusive_sum(mine, s_tmp, &all);
    if (tid < x.k) s_below[tid] = bel;
    pack_tile(x, base, &s_tile);
    clear_open(open, x.n, base);
    if (tid < kKeyTile / 32) s_rep[tid] = 0;
    __syncthreads();
    mark_runs(s_tile, s_rep, x.n, base, x.rep);
    const uint32_t drop = 32u - 2u * (uint32_t)x.K;
    const uint32_t j0 = seq_of(s_start, x.k, base);
#pragma unroll
    for (int r = 0; r < (int)(kKeyTile / kBlock); ++r) {
        const uint32_t l = r * kBlock + tid, p = base + l;
        if (p >= x.n) continue;
        uint32_t j = j0;
        while (p >= (uint32_t)s_start[j + 1]) ++j;        // p < n = start[k]
        if (p + (uint32_t)x.K >= (uint32_t)s_start[j + 1]) continue;   // near: its separator is among its K symbols
        const uint32_t i = l >> 4, sh = (l & 15u) * 2u;
        const uint64_t ww = ((uint64_t)s_tile.w[i] << 32) | s_tile.w[i + 1];
        const uint32_t key = (uint32_t)((ww << sh) >> 32) >> drop;
        const uint32_t e = p - s_below[j];
        keys[e] = key;
        vals[e] = p;
    }
}

__global__ __launch_bounds__(kBlock) void k_prefix_keys_tagged(Tagged x, uint32_t *__restrict__ keys,
                                                               uint32_t *__restrict__ vals, OpenBits open) {
    const uint32_t m = x.n - x.near;
    __shared__ KeyTile s_tile;
    __shared__ uint32_t s_rep[kKeyTile / 32];
    const uint32_t base = blockIdx.x * kKeyTile, tid = threadIdx.x;
    pack_tile(x, base, &s_tile);
    clear_open(open, x.n, base);
    if (tid < kKeyTile / 32) s_rep[tid] = 0;
    __syncthreads();
    mark_runs(s_tile, s_rep, x.n, base, x.rep);
    const uint32_t drop = 32u - 2u * (uint32_t)x.K;
#pragma unroll
    for (int r = 0; r < (int)(kKeyTile / kBlock); ++r) {
        const uint32_t l = r * kBlock + tid, p = base + l;
        if (p >= x.n) continue;
        const uint32_t pair = min((uint32_t)x.t[p] >> 3, x.k - 1u);
        const uint32_t s0 = (uint32_t)x.start[pair], a = (uint32_t)x.alen[pair], s1 = (uint32_t)x.start[pair + 1];
        const uint32_t sep = s0 + a;                                  // separator of A
        const bool inb = p > sep;
        if (p + (uint32_t)x.K >= (inb ? s1 : sep + 1u)) continue;
        const uint32_t i = l >> 4, sh = (l & 15u) * 2u;
        const uint64_t ww = ((uint64_t)s_tile.w[i] << 32) | s_tile.w[i + 1];
        const uint32_t key = ((uint32_t)((ww << sh) >> 32) >> drop) | (uint32_t)((uint64_t)pair << (2 * x.K));
        const uint32_t e = p - x.below[pair] - (inb ? near_of(a, x.K) : 0u);
        if (e >= m) continue;   // a bad input base spoils the pair number; the call then fails
        keys[e] = key;
        vals[e] = p;
    }
}

// Base-5 keys, 8 consecutive positions per thread from the last to the first:
// key(p) = s_p 5^(K-1) + key(p+1) / 5.
constexpr int kShareRun = 8;
__global__ __launch_bounds__(kBlock) void k_prefix_keys_shared(Shared x, uint32_t top, uint32_t *__restrict__ keys,
                                                               OpenBits open) {
    static_assert(kBlock * kShareRun == kKeyTile, "clear_open covers a workgroup's positions");
    clear_open(open, x.n, blockIdx.x * kKeyTile);
    const uint32_t p0 = (blockIdx.x * kBlock + threadIdx.x) * kShareRun;
    if (p0 >= x.n) return;
    uint32_t s[kShareRun + kMaxK];
#pragma unroll
    for (int i = 0; i < (kShareRun + kMaxK) / 4; ++i) {
        const uint32_t p = p0 + 4 * i;
        uint32_t w = 0;
        if (p < x.n && x.n - p >= 4) w = *reinterpret_cast<const uint32_t *>(x.t + p);
        else
            for (uint32_t c = 0; c < 4; ++c) w |= (p < x.n && c < x.n - p ? (uint32_t)x.t[p + c] : 0u) << (8 * c);
#pragma unroll
        for (int c = 0; c < 4; ++c) s[4 * i + c] = min((w >> (8 * c)) & 255u, 4u);
    }
    uint32_t key = 0, out[kShareRun];
#pragma unroll
    for (int i = kShareRun + kMaxK - 1; i >= 0; --i) {
        key = s[i] * top + key / 5u;
        if (i < kShareRun) out[i] = key;
    }
    if (x.n - p0 >= (uint32_t)kShareRun) {
        *reinterpret_cast<uint4 *>(keys + p0) = make_uint4(out[0], out[1], out[2], out[3]);
        *reinterpret_cast<uint4 *>(keys + p0 + 4) = make_uint4(out[4], out[5], out[6], out[7]);
    } else {
#pragma unroll
        for (int i = 0; i < kShareRun; ++i)
            if (p0 + i < x.n) keys[p0 + i] = out[i];
    }
}

// ----------------------------------------------------------- near suffixes
// A near suffix w#.. (w of d < K bases, then the separator) follows every
// normal suffix that starts with w and precedes those that start with
// anything larger: its place among the normal ones is the number of keys not
// above w filled with the largest base. Near suffixes that fill to the same
// key order by d from long to short (at the shorter one's separator the other
// has a base), then by separator. One thread per (sequence, d); `places`
// receives the places in order, which is all that the resolve kernel needs to
// shift the normal suffixes apart.
__device__ __forceinline__ uint32_t keys_not_above(const uint32_t *__restrict__ keys, uint32_t m, uint32_t v) {
    uint32_t lo = 0, len = m;
    while (len > 0) {
        const uint32_t half = len >> 1;
        if (keys[lo + half] <= v) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    return lo;
}

__device__ __forceinline__ uint32_t base2(uint8_t c) { return c & 3u; }
__device__ __forceinline__ uint32_t base2(uint16_t c) { return ((c & 7u) - 1u) & 3u; }

// Fill key of the suffix d symbols before the separator at `sep`, then what
// orders equal fills: K - 1 - d.
template <typename CH>
__device__ __forceinline__ uint32_t near_fill(const CH *__restrict__ t, uint32_t sep, uint32_t d, int K) {
    uint32_t v = 0;
    for (uint32_t c = 0; c < (uint32_t)K; ++c) v = (v << 2) | (c < d ? base2(t[sep - d + c]) : 3u);
    return v;
}

__global__ __launch_bounds__(kBlock) void k_merge(Joined x, const uint32_t *__restrict__ keys, uint32_t m,
                                                  int32_t *__restrict__ sa, uint32_t *__restrict__ places) {
    extern __shared__ uint64_t s_key[];   // one per (sequence, d); ~0 where there is none
    const uint32_t slots = x.k * (uint32_t)x.K;
    for (uint32_t i = threadIdx.x; i < slots; i += kBlock) {
        const uint32_t j = i / (uint32_t)x.K, d = i % (uint32_t)x.K;
        const uint32_t len = (uint32_t)(x.start[j + 1] - x.start[j]) - 1u;
        uint64_t v = ~0ull;
        if (d <= len)
            v = ((uint64_t)near_fill(x.t, (uint32_t)x.start[j + 1] - 1u, d, x.K) << 12) |
                ((uint64_t)((uint32_t)x.K - 1u - d) << 8) | j;
        s_key[i] = v;
    }
    __syncthreads();
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= slots || s_key[i] == ~0ull) return;
    const uint64_t mine = s_key[i];
    uint32_t rank = 0;
    for (uint32_t q = 0; q < slots; ++q) rank += s_key[q] < mine;
    const uint32_t at = keys_not_above(keys, m, (uint32_t)(mine >> 12));
    const uint32_t j = i / (uint32_t)x.K, d = i % (uint32_t)x.K;
    sa[at + rank] = x.start[j + 1] - 1 - (int32_t)d;
    places[rank] = at;
}

// The same for pairs: the pair leads every key, so near suffixes only compare
// inside their pair.
__global__ __launch_bounds__(kBlock) void k_merge_tagged(Tagged x, const uint32_t *__restrict__ keys, uint32_t m,
                                                         int32_t *__restrict__ sa, uint32_t *__restrict__ places) {
    const uint32_t per = 2u * (uint32_t)x.K;
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    const uint32_t pair = i / per, q0 = i % per;
    if (pair >= x.k) return;
    const uint32_t s0 = (uint32_t)x.start[pair], a = (uint32_t)x.alen[pair], s1 = (uint32_t)x.start[pair + 1];
    auto key_of = [&](uint32_t q, uint32_t *pos) -> uint64_t {
        const uint32_t second = q >= (uint32_t)x.K, d = q - (second ? (uint32_t)x.K : 0u);
        const uint32_t len = second ? s1 - s0 - a - 2u : a, sep = second ? s1 - 1u : s0 + a;
        if (d > len) return ~0ull;
        *pos = sep - d;
        return ((uint64_t)near_fill(x.t, sep, d, x.K) << 12) | ((uint64_t)((uint32_t)x.K - 1u - d) << 8) | second;
    };
    uint32_t pos = 0, other;
    const uint64_t mine = key_of(q0, &pos);
    if (mine == ~0ull) return;
    uint32_t rank = x.below[pair];
    for (uint32_t q = 0; q < per; ++q) rank += key_of(q, &other) < mine;
    const uint32_t at = keys_not_above(keys, m, (uint32_t)((uint64_t)pair << (2 * x.K)) | (uint32_t)(mine >> 12));
    sa[at + rank] = (int32_t)pos;
    places[rank] = at;
}

// keys_not_above() for the `count` sorted entries of a, by a wave.
__device__ __forceinline__ uint32_t wave_not_above(const uint32_t *__restrict__ a, uint32_t count, uint32_t x) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo = 0, len = count;
    while (len > 0) {
        const uint32_t step = (len + 63u) / 64u, o = lane * step;
        const bool in = o < len && a[lo + o] <= x;
        const uint32_t c = (uint32_t)__popcll(__ballot(in));
        if (c == 0) return lo;
        const uint32_t first = (c - 1u) * step + 1u;       // entries up to lo + first - 1 are in
        const uint32_t next = min(len, first + step - 1u);
        lo += first;
        len = next - first;
    }
    return lo;
}

// ----------------------------------------------------------- repeat keys
// The `count` (at most 21) symbols from i on at 3 bits, first on top; symbols
// past the end read 0, and with `stop` so do those behind a separator.
template <typename CH>
__device__ __forceinline__ uint64_t codes(const CH *__restrict__ t, uint32_t n, uint32_t i, uint32_t count,
                                          bool stop) {
    constexpr uint32_t W = 16 / sizeof(CH);
    uint64_t v = 0;
    bool open = true;
    for (uint32_t c0 = 0; c0 < count; c0 += W) {
        uint64_t hi, lo;
        window(t, n, i + c0, &hi, &lo);
#pragma unroll
        for (uint32_t c = 0; c < W; ++c) {
            if (c0 + c >= count) continue;
            const uint64_t half = c < W / 2 ? hi : lo;
            const uint32_t at = (W / 2 - 1u - c % (W / 2)) * 8u * (uint32_t)sizeof(CH);
            const uint32_t k = open && i + c0 + c < n ? code3((CH)(half >> at)) : 0u;
            if (stop && k == 5u) open = false;
            v = (v << 3) | k;
        }
    }
    return v;
}

template <typename X> struct StopAtSep { static constexpr bool value = true; };
template <> struct StopAtSep<Shared> { static constexpr bool value = false; };

// Set bits of `rep` from bit q on, up to about `cap`; there is a clear one before
// the end of the text. 128 bits a step.
__device__ __forceinline__ uint32_t run_ones(const uint32_t *__restrict__ rep, uint32_t q, uint32_t cap) {
    const uint4 *a = reinterpret_cast<const uint4 *>(rep);
    uint32_t b = q >> 7;
    const uint32_t o = q & 127u;
    uint64_t below0 = o < 64u ? (1ull << o) - 1ull : ~0ull, below1 = o < 64u ? 0ull : (1ull << (o - 64u)) - 1ull;
    for (;;) {
        const uint4 v = a[b];
        const uint64_t z0 = ~(((uint64_t)v.y << 32) | v.x) & ~below0, z1 = ~(((uint64_t)v.w << 32) | v.z) & ~below1;
        if (z0) return b * 128u + (uint32_t)__builtin_ctzll(z0) - q;
        if (z1) return b * 128u + 64u + (uint32_t)__builtin_ctzll(z1) - q;
        ++b;
        if (b * 128u - q >= cap) return cap;
        below0 = below1 = 0;
    }
}

// Where and how the suffix at q leaves the smallest period t of its first K
// symbols (K when they have none): 15 bits, e when it breaks downwards,
// 2 kExtent + 1 - e when upwards, kExtent when it runs at least that far; then
// its next `ns` symbols at 3 bits (0 behind a unique separator, which decides).
// The first K symbols hold no unique separator, so symbols that repeat them hold
// none either. A period that lasts kRepeat symbols is followed over the repeat
// bits: two or three lines instead of some 30 for the 400 symbols that a tandem
// repeat has left on average, 3.28 -> 0.15 ms in k_group_keys for 9.2 M suffixes.
template <typename X>
__device__ __forceinline__ uint64_t repeat_key(const X &x, uint32_t q, uint32_t ns, uint32_t *hdr, uint32_t budget) {
    using CH = typename X::CH;
    const uint32_t K = (uint32_t)x.K;
    const uint64_t v = codes(x.t, x.n, q, kRepeat, false), first = v >> (3u * (kRepeat - K));
    uint32_t t = 1;
    while (t < K && ((first ^ (first >> (3u * t))) & ((1ull << (3u * (K - t))) - 1ull))) ++t;
    uint32_t code = kExtent, e = x.n - q;
    if (X::kRepeatBits && t <= kRepeat / 2u && ((v ^ (v >> (3u * t))) & ((1ull << (3u * (kRepeat - t))) - 1ull)) == 0) {
        e = min(e, min(kRepeat + run_ones(x.rep, q, kExtent), kExtent));
        if (e < kExtent) code = (q + e >= x.n || x.t[q + e] < x.t[q + e - t]) ? e : 2 * kExtent + 1u - e;
    } else if (q + t < x.n) {
        e = min(e, t + dev::extend<CH, 2>(x.t, x.n, q, q + t, K - t, kExtent - t, Budget{hdr, budget}));
        if (e < kExtent) code = (q + e >= x.n || x.t[q + e] < x.t[q + e - t]) ? e : 2 * kExtent + 1u - e;
    } else {
        code = e;
    }
    return ((uint64_t)code << (3 * ns)) | codes(x.t, x.n, q + e, ns, StopAtSep<X>::value);
}

// ---------------------------------------------------------------- resolve
// Sort keys of large groups: group number, then a repeat key of ns symbols
// taken off[group] symbols into the suffix (off == nullptr: 0).
struct GroupKey {
    uint32_t ns;
    const uint32_t *off;
    __device__ uint32_t shift() const { return kCodeBits + 3u * ns; }
    __device__ uint32_t offset(uint64_t key) const { return off ? off[key >> shift()] : 0u; }
    // do the next symbols hold a separator (5, the only code with bits 2 and 0)?
    __device__ bool at_sep(uint64_t key) const {
        const uint64_t v = key & ((1ull << (3u * ns)) - 1ull);
        return ((v >> 2) & v & 0x1249249249249249ull) != 0;
    }
    // symbols up to the break: what the members of a group of equal keys share at least
    __device__ uint32_t reach(uint64_t key) const {
        const uint32_t c = (uint32_t)(key >> (3u * ns)) & ((1u << kCodeBits) - 1u);
        return offset(key) + (c <= kExtent ? c : 2u * kExtent + 1u - c);
    }
};

// Groups of equal keys over sorted (key, position) pairs, 256 ITEMS
// ranks per workgroup. Head flags are ballots (a 64-bit word per 64 ranks), with the
// words beside the tile's, so every rank of a group of at most kSmall knows
// its whole group and works out its own place; members just outside the tile
// are looked at by both workgroups. 8 text bytes behind the known prefix are
// gathered into LDS for every tied rank; a rank's place is the number of
// smaller ones in its group. Members that agree there too stay neighbours in
// the order they came in and are marked in `open` (see RunList) for k_settle, so
// that the few of them do not hold up the many.
// Stage 0 (32-bit keys of the sort) writes places shifted by the near
// suffixes; stage 1 (64-bit keys of large groups) through `slots`. Larger
// groups are marked in `large` and counted, with their heads, per tile.
// Bound by the window reads of the tied ranks, near the rate of random reads: 9.8 ms
// at 2^30 suffixes, 0.19 ms at 2^24; with the comparisons of what stays open in
// here too, a few members of long repeats held up their workgroups: 14.5 and 0.42.
template <typename X, typename KT, int ITEMS>
__global__ __launch_bounds__(kBlock) void k_resolve(X x, GroupKey gk, const KT *__restrict__ keys,
                                                    const uint32_t *__restrict__ vals, uint32_t m,
                                                    int32_t *__restrict__ sa, const uint32_t *__restrict__ slots,
                                                    const uint32_t *__restrict__ places, uint32_t near,
                                                    uint64_t *__restrict__ large, uint32_t *__restrict__ tcount,
                                                    uint32_t *__restrict__ hcount, uint32_t *__restrict__ ocount,
                                                    uint32_t *__restrict__ open, uint32_t *__restrict__ was) {
    using CH = typename X::CH;
    constexpr bool kFirst = sizeof(KT) == 4;
    constexpr uint32_t kResTile = kBlock * ITEMS, kResWords = kResTile / 64;
    constexpr uint32_t kSlots = kResTile + 2 * kSmall;
    constexpr int kWaves = kBlock / kWave;
    __shared__ uint64_t s_head[kResWords + 2];
    __shared__ uint32_t s_val[kSlots];
    __shared__ uint64_t s_win[kSlots];
    __shared__ uint16_t s_cls[kSlots];
    __shared__ uint32_t s_shift[2], s_large, s_heads, s_open;
    const uint32_t base = blockIdx.x * kResTile, tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    // Round r < ITEMS: slot kSmall + 256 r + tid, rank base + 256 r + tid;
    // the last round: the ranks beside the tile, waves 0 (before) and 1 (after).
    auto slot_of = [&](int r) { return r < ITEMS ? kSmall + r * kBlock + tid : (w == 0 ? lane : kResTile + tid); };
    auto rank_of = [&](int r) { return base + slot_of(r) - kSmall; };   // wraps before rank 0: not below m then
    // Values are positions; after a bad input base some may be anything, and
    // no text read may leave the text.
#pragma unroll
    for (int r = 0; r <= ITEMS; ++r) {
        if (r == ITEMS && w >= 2) break;
        const uint32_t e = rank_of(r);
        const bool ok = e < m;
        const KT key = ok ? keys[e] : KT(0);
        const uint32_t val = ok ? min(vals[e], x.n - 1u) : 0u;
        KT prev;
        if constexpr (kFirst) {
            prev = (KT)__shfl_up((int)key, 1, kWave);
            if (lane == 0 && ok && e > 0) prev = keys[e - 1];
        } else {
            prev = (ok && e > 0) ? keys[e - 1] : KT(0);
        }
        const uint64_t h = __ballot(!ok || e == 0 || prev != key);   // past the end: heads, so groups end there
        if (lane == 0) s_head[r < ITEMS ? 1 + r * kWaves + w : (w == 0 ? 0 : kResWords + 1)] = h;
        s_val[slot_of(r)] = val;
    }
    if (kFirst && w >= 2) {
        const uint32_t a = wave_not_above(places, near,
                                          w == 2 ? (base > kSmall ? base - kSmall : 0u) : base + kResTile + kSmall);
        if (lane == 0) s_shift[w - 2] = a;
    }
    if (tid == 0) s_large = s_heads = s_open = 0;
    __syncthreads();

    // Group of a slot: first slot and size; size 0 when it is larger than kSmall.
    auto group = [&](uint32_t l, uint32_t *first) -> uint32_t {
        const uint32_t wd = l >> 6, b = l & 63u;
        const uint64_t upto = s_head[wd] & (~0ull >> (63u - b));
        uint32_t f, g;
        if (upto) f = wd * 64u + 63u - (uint32_t)__builtin_clzll(upto);
        else if (wd > 0 && s_head[wd - 1]) f = (wd - 1) * 64u + 63u - (uint32_t)__builtin_clzll(s_head[wd - 1]);
        else return 0;
        const uint64_t over = b == 63 ? 0ull : s_head[wd] & (~0ull << (b + 1u));
        if (over) g = wd * 64u + (uint32_t)__builtin_ctzll(over);
        else if (wd + 1 < kResWords + 2 && s_head[wd + 1]) g = (wd + 1) * 64u + (uint32_t)__builtin_ctzll(s_head[wd + 1]);
        else return 0;
        *first = f;
        return g - f <= kSmall ? g - f : 0u;
    };
    // Size of a slot's group when this workgroup has to look at it: every rank
    // of the tile, and those beside it whose group reaches into it.
    auto tied = [&](int r, uint32_t *first) -> uint32_t {
        if (r == ITEMS) {
            if (w >= 2) return 0;
            const uint64_t h = s_head[w == 0 ? 0 : kResWords + 1];
            const bool reach = w == 0 ? (lane == 63 || !(h >> (lane + 1u))) && !(s_head[1] & 1ull)
                                      : !(h & (~0ull >> (63u - lane)));
            if (!reach) return 0;
        }
        return rank_of(r) < m ? group(slot_of(r), first) : 0u;
    };

    // 8 text bytes of every tied rank, all gathers of a thread in flight at once
    uint64_t win[ITEMS + 1];
#pragma unroll
    for (int r = 0; r <= ITEMS; ++r) {
        uint32_t f;
        win[r] = 0;
        if (tied(r, &f) > 1) {
            const uint32_t l = slot_of(r);
            uint32_t h = (uint32_t)x.K;
            if constexpr (!kFirst) h = max(h, gk.reach(keys[rank_of(r)]));
            win[r] = window8(x.t, x.n, s_val[l] + h);
        }
    }
#pragma unroll
    for (int r = 0; r <= ITEMS; ++r)
        if (r < ITEMS || w < 2) s_win[slot_of(r)] = win[r];
    __syncthreads();
    // class of every tied rank: first place of those with its window
#pragma unroll
    for (int r = 0; r <= ITEMS; ++r) {
        uint32_t f;
        const uint32_t size = tied(r, &f);
        if (size > 1) {
            uint32_t less = f;
            for (uint32_t q = f; q < f + size; q += kScan) {
                uint64_t y[kScan];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) y[i] = s_win[min(q + i, f + size - 1u)];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) less += q + i < f + size && y[i] < win[r];
            }
            s_cls[slot_of(r)] = (uint16_t)less;
        }
    }
    __syncthreads();

    const uint32_t sh0 = kFirst ? s_shift[0] : 0u, sh1 = kFirst ? s_shift[1] : 0u;
    uint32_t lost = 0, heads = 0;
#pragma unroll 1
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t l = slot_of(r), e = rank_of(r);
        const bool valid = e < m;
        uint32_t f = 0;
        const uint32_t size = group(l, &f), v = s_val[l];
        bool big = valid && size == 0, kept = false;
        if constexpr (!kFirst && StopAtSep<X>::value) {
            // equal up to their separators: ordered by those, so by position,
            // which the stable sorts have kept
            if (big && gk.at_sep(keys[e])) {
                big = false;
                kept = true;
            }
        }
        const uint64_t bm = __ballot(big);
        if (lane == 0) {
            large[(size_t)blockIdx.x * kResWords + r * kWaves + w] = bm;
            lost += (uint32_t)__popcll(bm);
            heads += (uint32_t)__popcll(bm & s_head[l >> 6]);
        }
        if (!valid || big) continue;
        uint32_t place = l, same = 0;                       // same: equal ones placed before this rank
        if (size > 1 && !kept) {
            const uint16_t cls = s_cls[l];
            place = cls;
#pragma unroll 4
            for (uint32_t q = f; q < l; ++q) same += s_cls[q] == cls;
            place += same;
        }
        const uint32_t o = base + place - kSmall;           // place in the sorted order
        if (o >= m) continue;
        uint32_t slot;
        if constexpr (kFirst) {
            slot = o + sh0;
            if (sh0 != sh1) slot += keys_not_above(places + sh0, sh1 - sh0, o);
        } else {
            slot = slots[o];
        }
        sa[slot] = (int32_t)v;
        if (same) {
            atomicOr(&open[slot >> 5], 1u << (slot & 31u));
            if (was) atomicOr(&was[slot >> 5], 1u << (slot & 31u));
            atomicAdd(&s_open, 1u);
        }
    }
    if (lane == 0 && lost) {
        atomicAdd(&s_large, lost);
        atomicAdd(&s_heads, heads);
    }
    __syncthreads();
    if (tid == 0) {
        tcount[blockIdx.x] = s_large;
        hcount[blockIdx.x] = s_heads;
        ocount[blockIdx.x] = s_open;
    }
}

// Sums of the tiles' counts into the header. Atomics from every tile on three
// words would take their turns, some 30 ns each.
constexpr uint32_t kSumGroups = 64;
__global__ __launch_bounds__(kBlock) void k_resolve_totals(const uint32_t *__restrict__ tcount,
                                                           const uint32_t *__restrict__ hcount,
                                                           const uint32_t *__restrict__ ocount, uint32_t tiles,
                                                           uint32_t *__restrict__ hdr) {
    __shared__ uint32_t s_tmp[kBlock / kWave];
    uint32_t t = 0, h = 0, o = 0;
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < tiles; i += gridDim.x * kBlock) {
        t += tcount[i];
        h += hcount[i];
        o += ocount[i];
    }
    uint32_t st, sh, so;
    dev::block_exclusive_sum(t, s_tmp, &st);
    dev::block_exclusive_sum(h, s_tmp, &sh);
    dev::block_exclusive_sum(o, s_tmp, &so);
    if (threadIdx.x == 0) {
        if (st) atomicAdd(&hdr[kWordTied], st);
        if (sh) atomicAdd(&hdr[kWordHeads], sh);
        if (so) atomicAdd(&hdr[kWordOpen], so);
    }
}

// ----------------------------------------------------------- large groups
// The marked ranks in rank order: position, final slot, and the group number
// (the count of marked heads up to here); a group's head writes how many
// symbols further into the suffix the group's next keys start, so that the K
// symbols there end where the known prefix ends.
template <typename KT, int ITEMS>
__global__ __launch_bounds__(kBlock) void k_group_collect(GroupKey gk, int K, const KT *__restrict__ keys,
                                                          const uint32_t *__restrict__ vals, uint32_t m,
                                                          const uint64_t *__restrict__ large,
                                                          const uint32_t *__restrict__ tbase,
                                                          const uint32_t *__restrict__ hbase,
                                                          const uint32_t *__restrict__ places, uint32_t near,
                                                          const uint32_t *__restrict__ slots, uint32_t total,
                                                          uint32_t groups, uint64_t *__restrict__ tkeys,
                                                          uint32_t *__restrict__ tvals, uint32_t *__restrict__ tslots,
                                                          uint32_t *__restrict__ off) {
    constexpr bool kFirst = sizeof(KT) == 4;
    constexpr uint32_t kResTile = kBlock * ITEMS, kResWords = kResTile / 64;
    __shared__ uint32_t s_below[kResWords], s_hbelow[kResWords];
    __shared__ uint64_t s_bits[kResWords], s_head[kResWords];
    __shared__ uint32_t s_shift[2], s_none;
    const uint32_t base = blockIdx.x * kResTile, tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    static_assert(kResWords <= 64, "one lane per word");
    // most tiles hold no large group
    if (w == 0) {
        const uint64_t b = lane < kResWords ? large[(size_t)blockIdx.x * kResWords + lane] : 0ull;
        if (lane < kResWords) s_bits[lane] = b;
        if (lane == 0) s_none = 1;
        if (b) s_none = 0;
    }
    __syncthreads();
    if (s_none) return;
    KT key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t e = base + r * kBlock + tid;
        key[r] = e < m ? keys[e] : KT(0);
        const KT prev = (e > 0 && e < m) ? keys[e - 1] : KT(0);
        const uint64_t h = __ballot(e < m && (e == 0 || prev != key[r]));
        if (lane == 0) s_head[r * (kBlock / kWave) + w] = h;
    }
    if (kFirst && w >= 2) {
        const uint32_t a = wave_not_above(places, near, w == 2 ? base : base + kResTile);
        if (lane == 0) s_shift[w - 2] = a;
    }
    __syncthreads();
    if (w == 0) {
        const uint64_t b = lane < kResWords ? s_bits[lane] : 0ull;
        const uint32_t c = (uint32_t)__popcll(b), hc = lane < kResWords ? (uint32_t)__popcll(b & s_head[lane]) : 0u;
        const uint32_t inc = dev::wave_inclusive_sum(c), hinc = dev::wave_inclusive_sum(hc);
        if (lane < kResWords) {
            s_below[lane] = inc - c;
            s_hbelow[lane] = hinc - hc;
        }
    }
    __syncthreads();
    const uint32_t at = tbase[blockIdx.x], hat = hbase[blockIdx.x];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t l = r * kBlock + tid, e = base + l;
        const uint64_t b = s_bits[l >> 6], bit = 1ull << (l & 63u);
        if (e >= m || !(b & bit)) continue;
        const uint64_t heads = b & s_head[l >> 6];
        const uint32_t i = at + s_below[l >> 6] + (uint32_t)__popcll(b & (bit - 1ull));
        const uint32_t id = hat + s_hbelow[l >> 6] + (uint32_t)__popcll(heads & (bit | (bit - 1ull))) - 1u;
        if (i >= total || id >= groups) continue;   // never with consistent counts
        if constexpr (kFirst) {
            tslots[i] = e + s_shift[0] + keys_not_above(places + s_shift[0], s_shift[1] - s_shift[0], e);
        } else {
            tslots[i] = slots[e];
            if (heads & bit) off[id] = gk.reach(key[r]) + gk.ns - (uint32_t)K;
        }
        tkeys[i] = id;
        tvals[i] = vals[e];
    }
}

template <typename X>
__global__ __launch_bounds__(kBlock) void k_group_keys(X x, GroupKey gk, uint64_t *__restrict__ tkeys,
                                                       const uint32_t *__restrict__ tvals, uint32_t total,
                                                       uint32_t *__restrict__ hdr, uint32_t budget) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= total) return;
    const uint64_t id = tkeys[i];
    const uint32_t p = min(tvals[i], x.n - 1u);
    const uint32_t q = min(p + (gk.off ? gk.off[id] : 0u), x.n - 1u);
    tkeys[i] = (id << gk.shift()) | repeat_key(x, q, gk.ns, hdr, budget);
}

// -------------------------------------------------------------- open runs
// What resolve leaves open: runs of neighbouring slots (at most kSmall) whose
// suffixes agree as far as it looked. An item is a slot that is in a run, or in
// small texts any slot (RunList::slots is null then); bit i of `open`: item i
// agrees with item i - 1. k_settle compares texts; what is left then shares h
// symbols and is settled by doubling: with rank[p] the first slot of p's run,
// the suffixes of a run are ordered by rank[p + h], after which open runs share
// 2 h symbols, so a few rounds settle long exact or nearly exact copies that a
// comparison would walk through suffix by suffix. A workgroup owns the runs
// that start in its tile of items; `was` holds the bits of before the launch.
// Ranks only change between the rounds (k_run_ranks): all of a round's lookups
// see the same ranks.
struct RunList {
    const uint32_t *slots;   // slot of every item (null: the item itself)
    const uint32_t *count;   // device word: the number of items (null: cap)
    uint32_t cap;
    __device__ uint32_t items() const { return count ? min(*count, cap) : cap; }
    __device__ uint32_t slot(uint32_t i) const { return slots ? slots[i] : i; }
};

__device__ __forceinline__ bool open_bit(const uint32_t *open, uint32_t i, uint32_t items) {
    return i < items && ((open[i >> 5] >> (i & 31u)) & 1u);
}

// Slots in runs: those marked and those before a marked one.
__device__ __forceinline__ uint32_t run_members(const uint32_t *__restrict__ open, uint32_t words, uint32_t w) {
    if (w >= words) return 0;
    const uint32_t b = open[w], next = w + 1 < words ? open[w + 1] & 1u : 0u;
    return b | (b >> 1) | (next << 31);
}

// The items of a large text: the slots in runs, in slot order, so that the few
// of them fill their workgroups (one tile of slots in two holds a run on DNA
// texts of 16M bases, but few of them: 337 us in k_settle over slots, 60 over the
// list and 20 to make it).
constexpr uint32_t kOpenWords = 4 * kBlock;   // bitmap words per workgroup
__global__ __launch_bounds__(kBlock) void k_open_count(const uint32_t *__restrict__ open, uint32_t words,
                                                       uint32_t *__restrict__ count) {
    __shared__ uint32_t s_tmp[kBlock / kWave];
    uint32_t c = 0, all;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r)
        c += (uint32_t)__popc(run_members(open, words, blockIdx.x * kOpenWords + r * kBlock + threadIdx.x));
    dev::block_exclusive_sum(c, s_tmp, &all);
    if (threadIdx.x == 0) count[blockIdx.x] = all;
}

__global__ __launch_bounds__(kBlock) void k_open_list(const uint32_t *__restrict__ open, uint32_t words,
                                                      const uint32_t *__restrict__ first, uint32_t cap,
                                                      uint32_t *__restrict__ slots, uint32_t *__restrict__ bits) {
    __shared__ uint32_t s_tmp[kBlock / kWave];
    uint32_t base = first[blockIdx.x];
    for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t w = blockIdx.x * kOpenWords + r * kBlock + threadIdx.x;
        uint32_t m = run_members(open, words, w), all;
        uint32_t at = base + dev::block_exclusive_sum((uint32_t)__popc(m), s_tmp, &all);
        const uint32_t b = m ? open[w] : 0u;
        for (; m; m &= m - 1u, ++at) {
            const uint32_t i = (uint32_t)__builtin_ctz(m);
            if (at >= cap) break;   // never with consistent counts
            slots[at] = 32u * w + i;
            if ((b >> i) & 1u) atomicOr(&bits[at >> 5], 1u << (at & 31u));
        }
        base += all;
    }
}

__device__ __forceinline__ uint32_t run_head(const uint32_t *__restrict__ open, uint32_t i) {
    uint32_t wd = i >> 5;
    uint32_t z = ~open[wd] & (0xffffffffu >> (31u - (i & 31u)));
    while (!z && wd > 0) z = ~open[--wd];
    return z ? wd * 32u + 31u - (uint32_t)__builtin_clz(z) : 0u;
}

// rank of every suffix: the first slot of its run where the items are the
// slots, else its slot.
__global__ __launch_bounds__(kBlock) void k_ranks(uint32_t n, const int32_t *__restrict__ sa,
                                                  const uint32_t *__restrict__ open, uint32_t *__restrict__ rank) {
    for (uint32_t s = blockIdx.x * kBlock + threadIdx.x; s < n; s += gridDim.x * kBlock) {
        const uint32_t p = (uint32_t)sa[s];
        if (p < n) rank[p] = open ? run_head(open, s) : s;
    }
}

// Ranks of the suffixes that were in runs before the round: the slot of their
// run's first item now.
__global__ __launch_bounds__(kBlock) void k_run_ranks(RunList list, const uint32_t *__restrict__ open,
                                                      const uint32_t *__restrict__ was, uint32_t n,
                                                      const int32_t *__restrict__ sa, uint32_t *__restrict__ rank) {
    const uint32_t items = list.items();
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < items; i += gridDim.x * kBlock) {
        if (!open_bit(was, i, items) && !open_bit(was, i + 1, items)) continue;
        const uint32_t p = (uint32_t)sa[list.slot(i)];
        if (p < n) rank[p] = list.slot(run_head(open, i));
    }
}

__global__ __launch_bounds__(kBlock) void k_copy_words(const uint32_t *__restrict__ a, uint32_t *__restrict__ b,
                                                       uint32_t count) {
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < count; i += gridDim.x * kBlock) b[i] = a[i];
}

// Items per tile. k_settle: with the kSmall items after them one per thread, so
// the chains of waits run side by side. k_double, which waits little, has larger ones.
constexpr uint32_t kSettleTile = kBlock - kSmall, kDoubleTile = 4 * kBlock - kSmall;
// Workgroups of k_settle and of the (shorter) k_double: each may end in an
// atomic on the same word, about 30 ns apart.
constexpr uint32_t kSettleGroups = 8192, kDoubleGroups = 2048;
constexpr uint32_t kRepeatRun = 5;

// A tile's run bits (and those of the items after it) in LDS.
template <uint32_t TILE>
struct RunTile {
    static constexpr uint32_t kWords = (TILE + 2 * kSmall) / 32;
    const uint32_t *bits;   // kWords words
    // Item l of the tile or of the kSmall after it: first item and size of its
    // run, size 0 when the run is one suffix or starts in another tile.
    __device__ uint32_t run_of(uint32_t l, uint32_t *first) const {
        uint32_t wd = l >> 5;
        uint32_t z = ~bits[wd] & (0xffffffffu >> (31u - (l & 31u)));
        while (!z && wd > 0) z = ~bits[--wd];
        if (!z) return 0;
        const uint32_t f = wd * 32u + 31u - (uint32_t)__builtin_clz(z);
        uint32_t g = l + 1;
        wd = g >> 5;
        z = wd < kWords ? ~bits[wd] & (0xffffffffu << (g & 31u)) : 1u;
        while (!z && ++wd < kWords) z = ~bits[wd];
        g = wd < kWords ? wd * 32u + (uint32_t)__builtin_ctz(z) : TILE + 2 * kSmall;
        *first = f;
        return f < TILE && g - f > 1 && g - f <= kSmall ? g - f : 0u;
    }
    // Loads the bits of the tile that starts at item `base`; false (for the
    // whole workgroup) when no run is near.
    static __device__ bool load(const uint32_t *__restrict__ was, uint32_t items, uint32_t base, uint32_t *s_bits) {
        const uint32_t words = (items + 31u) / 32u, i = threadIdx.x, w = base / 32u + i;
        const uint32_t b = i < kWords && w < words ? was[w] : 0u;
        __syncthreads();   // the tile before is done with its bits
        if (i < kWords) s_bits[i] = b;
        return __syncthreads_or(b != 0) != 0;
    }
};

__global__ __launch_bounds__(kBlock) void k_double(RunList list, const uint32_t *__restrict__ was,
                                                   uint32_t *__restrict__ open, uint32_t n, uint32_t h,
                                                   const uint32_t *__restrict__ rank, int32_t *__restrict__ sa,
                                                   uint32_t *__restrict__ left) {
    using Tile = RunTile<kDoubleTile>;
    constexpr int kPer = (kDoubleTile + kSmall) / kBlock;
    static_assert(kPer * kBlock == kDoubleTile + kSmall, "whole items per thread");
    __shared__ uint32_t s_bits[Tile::kWords], s_rank[kPer * kBlock], s_left;
    const uint32_t tid = threadIdx.x, items = list.items();
    const Tile runs{s_bits};
    if (tid == 0) s_left = 0;
    for (uint32_t base = blockIdx.x * kDoubleTile; base < items; base += gridDim.x * kDoubleTile) {
        if (!Tile::load(was, items, base, s_bits)) continue;
        uint32_t val[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const uint32_t l = r * kBlock + tid;
            uint32_t f;
            val[r] = 0xffffffffu;
            if (base + l < items && runs.run_of(l, &f)) {
                const uint32_t p = (uint32_t)sa[list.slot(base + l)];
                val[r] = p;
                s_rank[l] = p < n && h < n - p ? rank[p + h] + 1u : 0u;   // the end of the text comes first
            }
        }
        __syncthreads();
        uint32_t mine_left = 0;
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const uint32_t l = r * kBlock + tid;
            if (val[r] == 0xffffffffu) continue;
            uint32_t f;
            const uint32_t size = runs.run_of(l, &f), mine = s_rank[l];
            uint32_t place = f, same = 0;
#pragma unroll 4
            for (uint32_t q = f; q < f + size; ++q) {
                const uint32_t o = s_rank[q];
                place += o < mine;
                same += o == mine && q < l;
            }
            place += same;
            const uint32_t to = base + place;
            if (to >= items) continue;
            sa[list.slot(to)] = (int32_t)val[r];
            if (same) ++mine_left;
            else if (place != f) atomicAnd(&open[to >> 5], ~(1u << (to & 31u)));
        }
        if (mine_left) atomicAdd(&s_left, mine_left);
    }
    __syncthreads();
    if (tid == 0 && s_left) atomicAdd(left, s_left);
}

// The same by comparing texts, up to `deep` symbols. Repeat keys come first: a
// tandem repeat inside one run would cost a long comparison per member and step
// otherwise. Runs of fewer than kRepeatRun, which have few steps, do without:
// the keys read as much as a comparison does (65,536 queries: 1.45 -> 0.48 ms).
// Runs share at least the K symbols of their sort key. Bound by the chain of
// waits of a run's members, so one item per thread and many workgroups: five
// per thread took 100 us longer on 64 pairs of 1,000 to 10,000 bases.
template <typename X>
__global__ __launch_bounds__(kBlock) void k_settle(X x, RunList list, const uint32_t *__restrict__ was,
                                                   uint32_t *__restrict__ open, int32_t *__restrict__ sa,
                                                   uint32_t deep, uint32_t *__restrict__ left,
                                                   uint32_t *__restrict__ hdr, uint32_t budget) {
    using Tile = RunTile<kSettleTile>;
    __shared__ uint32_t s_bits[Tile::kWords], s_val[kBlock], s_left;
    __shared__ uint64_t s_key[kBlock];
    __shared__ uint16_t s_cls[kBlock];
    const uint32_t l = threadIdx.x, items = list.items();
    const Tile runs{s_bits};
    if (hdr[kWordTied]) return;   // another round over large groups comes first: all is left as it is
    if (l == 0) s_left = 0;
    for (uint32_t base = blockIdx.x * kSettleTile; base < items; base += gridDim.x * kSettleTile) {
        if (!Tile::load(was, items, base, s_bits)) continue;
        uint32_t f = 0, place = 0, reach = 0;
        const uint32_t size = base + l < items ? runs.run_of(l, &f) : 0u;
        uint64_t k = 0;
        if (size) {
            const uint32_t p = min((uint32_t)sa[list.slot(base + l)], x.n - 1u);
            if (size >= kRepeatRun) k = repeat_key(x, p, kRepeatSymbols, hdr, budget);
            s_val[l] = p;
            s_key[l] = k;
        }
        __syncthreads();
        bool again = false;
        if (size) {
            uint32_t same = 0;
            place = f;
            for (uint32_t q = f; q < f + size; q += kScan) {
                uint64_t y[kScan];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) y[i] = s_key[min(q + i, f + size - 1u)];
#pragma unroll
                for (uint32_t i = 0; i < kScan; ++i) {
                    place += q + i < f + size && y[i] < k;
                    same += q + i < f + size && y[i] == k;
                }
            }
            const uint32_t c = (uint32_t)(k >> (3u * kRepeatSymbols));
            reach = max((uint32_t)x.K, c <= kExtent ? c : 2u * kExtent + 1u - c);
            again = same > 1;
        }
        // where few are open, as around one long copy, a longer comparison here saves a round
        const bool sparse = __syncthreads_count(again) <= (int)(kSettleTile / 8) && list.slots == nullptr;
        if (size) {
            s_cls[l] = (uint16_t)place;
            s_key[l] = (uint64_t)reach << 32;
        }
        refine(x.t, x.n, sparse ? kSettle : deep, f, size, s_val, s_key, s_cls, again);
        if (size) {
            uint32_t same = 0;
            const uint16_t c = s_cls[l];
#pragma unroll 4
            for (uint32_t q = f; q < l; ++q) same += s_cls[q] == c;
            const uint32_t to = base + c + same;
            if (to < items) {
                sa[list.slot(to)] = (int32_t)s_val[l];
                if (same) atomicAdd(&s_left, 1u);
                else if (to != base + f) atomicAnd(&open[to >> 5], ~(1u << (to & 31u)));
            }
        }
    }
    __syncthreads();
    if (l == 0 && s_left) atomicAdd(left, s_left);
}

// ----------------------------------------------------------- larger groups
// Groups that no workgroup holds and that their next symbols do not tell apart
// (words with more than kSmall copies) are doubled by sorting: their members (the
// pool) by (group, rank[p + h]), after which a group's members share 2 h symbols. A
// suffix alone with its key leaves the pool. Groups are numbered in slot order,
// so the i-th item of the sorted pool has the slot of the i-th before. Suffix arrays
// by this against those by DC3 alone: 65 copies of 100 bases in 1M 0.83 / 1.96 ms, in
// 16M 1.44 / 4.16 ms; 3,000 of 1,000 with 1% mutations in 16M 2.8 / 5.7 ms.
constexpr uint32_t kPoolItems = 4, kPoolTile = kBlock * kPoolItems;

struct PoolItems {   // the pool after a sort
    const uint64_t *keys;
    const uint32_t *vals, *slots;
    uint32_t m;
    __device__ bool head(uint32_t i) const { return i == 0 || i >= m || keys[i] != keys[i - 1]; }
};

// Items of a tile that stay in the pool, and the heads of their groups.
__global__ __launch_bounds__(kBlock) void k_pool_count(PoolItems x, uint32_t *__restrict__ tcount,
                                                       uint32_t *__restrict__ hcount) {
    __shared__ uint32_t s_tmp[kBlock / kWave];
    uint32_t c = 0, all;   // members, and heads above them
#pragma unroll
    for (uint32_t r = 0; r < kPoolItems; ++r) {
        const uint32_t i = blockIdx.x * kPoolTile + r * kBlock + threadIdx.x;
        if (i >= x.m) continue;
        if (!x.head(i)) c += 1u;
        else if (!x.head(i + 1)) c += 0x10001u;
    }
    static_assert(kPoolTile < 0x10000u, "two counts in a word");
    dev::block_exclusive_sum(c, s_tmp, &all);
    if (threadIdx.x == 0) {
        tcount[blockIdx.x] = all & 0xffffu;
        hcount[blockIdx.x] = all >> 16;
    }
}

// SA takes the sorted order, suffixes that leave the pool their ranks; the others
// go on with their group's new number, and every group with its first slot.
__global__ __launch_bounds__(kBlock) void k_pool_collect(PoolItems x, const uint32_t *__restrict__ tbase,
                                                         const uint32_t *__restrict__ hbase, uint32_t cap, uint32_t n,
                                                         int32_t *__restrict__ sa, uint32_t *__restrict__ rank,
                                                         uint64_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                         uint32_t *__restrict__ slots, uint32_t *__restrict__ first) {
    __shared__ uint32_t s_tmp[kBlock / kWave];
    uint32_t at = tbase[blockIdx.x], group = hbase[blockIdx.x];
    for (uint32_t r = 0; r < kPoolItems; ++r) {
        const uint32_t i = blockIdx.x * kPoolTile + r * kBlock + threadIdx.x;
        const bool head = i < x.m && x.head(i), member = i < x.m && !(head && x.head(i + 1));
        uint32_t all;
        const uint32_t below = dev::block_exclusive_sum(member ? (head ? 0x10001u : 1u) : 0u, s_tmp, &all);
        const uint32_t o = at + (below & 0xffffu), id = group + (below >> 16) - (head ? 0u : 1u);
        at += all & 0xffffu;
        group += all >> 16;
        if (i >= x.m) continue;
        const uint32_t slot = x.slots[i], p = x.vals[i];
        sa[slot] = (int32_t)p;
        if (!member) {
            if (p < n) rank[p] = slot;
        } else if (o < cap && id <= cap / 2) {   // always with consistent counts
            keys[o] = id;
            vals[o] = p;
            slots[o] = slot;
            if (head) first[id] = slot;
        }
    }
}

// The pool at its start: SA takes its members in any order (ranks are made from all of
// SA), every group its first slot.
__global__ __launch_bounds__(kBlock) void k_pool_start(const uint64_t *__restrict__ keys,
                                                       const uint32_t *__restrict__ vals,
                                                       const uint32_t *__restrict__ slots, uint32_t total, uint32_t n,
                                                       int32_t *__restrict__ sa, uint32_t *__restrict__ first) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= total) return;
    const uint32_t slot = slots[i];
    sa[slot] = (int32_t)min(vals[i], n - 1u);
    if (i == 0 || keys[i] != keys[i - 1]) first[keys[i]] = slot;
}

// A suffix in the pool ranks as its group's first slot.
__global__ __launch_bounds__(kBlock) void k_pool_ranks(const uint64_t *__restrict__ keys,
                                                       const uint32_t *__restrict__ vals,
                                                       const uint32_t *__restrict__ first, uint32_t total, uint32_t n,
                                                       uint32_t *__restrict__ rank) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < total && vals[i] < n) rank[vals[i]] = first[keys[i]];
}

__global__ __launch_bounds__(kBlock) void k_pool_keys(uint64_t *__restrict__ keys, const uint32_t *__restrict__ vals,
                                                      uint32_t total, uint32_t h, uint32_t n, int rank_bits,
                                                      const uint32_t *__restrict__ rank) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= total) return;
    const uint32_t p = vals[i];
    const uint64_t r = p < n && h < n - p ? rank[p + h] + 1u : 0u;   // the end of the text comes first
    keys[i] = (keys[i] << rank_bits) | r;
}

// ------------------------------------------------------------------ driver

struct PrefixHdr {
    uint32_t word[16];
};

lor_status launch_keys(const Joined &x, uint32_t *k, uint32_t *v, OpenBits open, hipStream_t s) {
    LOR_LAUNCH("k_prefix_keys", 9.0 * x.n, s,
               hipLaunchKernelGGL(k_prefix_keys, dim3(div_up(x.n, kKeyTile)), dim3(kBlock), 0, s, x, k, v, open));
    return LOR_OK;
}
lor_status launch_keys(const Tagged &x, uint32_t *k, uint32_t *v, OpenBits open, hipStream_t s) {
    LOR_LAUNCH("k_prefix_keys", 10.0 * x.n, s,
               hipLaunchKernelGGL(k_prefix_keys_tagged, dim3(div_up(x.n, kKeyTile)), dim3(kBlock), 0, s, x, k, v, open));
    return LOR_OK;
}
lor_status launch_keys(const Shared &x, uint32_t *k, uint32_t *, OpenBits open, hipStream_t s) {
    uint32_t top = 1;
    for (int i = 1; i < x.K; ++i) top *= 5u;
    LOR_LAUNCH("k_prefix_keys", 5.0 * x.n, s,
               hipLaunchKernelGGL(k_prefix_keys_shared, dim3(div_up(x.n, kBlock * kShareRun)), dim3(kBlock), 0, s, x,
                                  top, k, open));
    return LOR_OK;
}

lor_status launch_near(const Joined &x, const uint32_t *keys, uint32_t m, int32_t *sa, uint32_t *places,
                       hipStream_t s) {
    const uint32_t slots = x.k * (uint32_t)x.K;
    LOR_LAUNCH("k_merge", 8.0 * x.near, s,
               hipLaunchKernelGGL(k_merge, dim3(div_up(slots, kBlock)), dim3(kBlock), slots * sizeof(uint64_t), s, x,
                                  keys, m, sa, places));
    return LOR_OK;
}
lor_status launch_near(const Tagged &x, const uint32_t *keys, uint32_t m, int32_t *sa, uint32_t *places,
                       hipStream_t s) {
    LOR_LAUNCH("k_merge", 8.0 * x.near, s,
               hipLaunchKernelGGL(k_merge_tagged, dim3(div_up(2ull * x.k * (uint32_t)x.K, kBlock)), dim3(kBlock), 0, s,
                                  x, keys, m, sa, places));
    return LOR_OK;
}
lor_status launch_near(const Shared &, const uint32_t *, uint32_t, int32_t *, uint32_t *, hipStream_t) {
    return LOR_OK;
}

lor_status read_header(uint32_t *hdr, PrefixHdr *h, hipStream_t s) {
    LOR_HIP(hipMemcpyWithStream(h, hdr, sizeof(*h), hipMemcpyDeviceToHost, s));   // waits for the stream
    if (h->word[0]) {
        set_error("input base outside 0..3");
        return LOR_EALPHABET;
    }
    return LOR_OK;
}

// Compares the texts of open runs, up to `deep` symbols; the number still open
// is added to *left.
template <typename X>
lor_status launch_settle(const X &x, const RunList &list, const uint32_t *was, uint32_t *open, int32_t *sa,
                         uint32_t deep, uint32_t *left, uint32_t *hdr, uint32_t budget, hipStream_t s) {
    LOR_LAUNCH("k_settle", 0.125 * list.cap, s,
               hipLaunchKernelGGL(k_settle<X>, dim3(std::min(div_up(list.cap, kSettleTile), kSettleGroups)), dim3(kBlock),
                                  0, s, x, list, was, open, sa, deep, left, hdr, budget));
    return LOR_OK;
}

lor_status copy_words(const uint32_t *a, uint32_t *b, uint32_t count, hipStream_t s) {
    LOR_LAUNCH("k_copy_words", 8.0 * count, s,
               hipLaunchKernelGGL(k_copy_words, dim3(grid_for(count)), dim3(kBlock), 0, s, a, b, count));
    return LOR_OK;
}

// What the sorts of large groups may still cost. A sorted suffix of a round takes
// some 0.13 ns (up to seven passes over 64-bit keys, lookups and scatters), a round's
// launches 70 us; DC3 0.3 to 0.5 ns per suffix of a text with large groups and 1.3 ms
// or more. So half of a DC3 run is spent at most before giving up, or 3.3 ms where
// that is more; mostly a fifth or less, as worth() looks ahead (16M bases with 2,000
// copies of 3,000: 8.0 ms, 6.6 by DC3 alone, 6.6 by doubling to the end).
struct Spend {
    uint64_t left;
    explicit Spend(uint32_t n) : left(std::max<uint64_t>(n + n / 2ull, kLeastSpend)) {}
    bool take(uint32_t members) {
        const uint64_t c = members + kRoundCost;
        if (c > left) return false;
        left -= c;
        return true;
    }
    // Of `members` a round is expected to settle `lost`, and every round twice as many
    // as the one before: a copy's suffixes are told apart where the symbols compared
    // reach its end.
    bool worth(uint64_t members, uint64_t lost) const {
        uint64_t cost = 0;
        for (lost = std::max<uint64_t>(lost, 1); cost <= left; lost *= 2) {
            cost += members + kRoundCost;
            if (lost >= members) return cost <= left;
            members -= lost;
        }
        return false;
    }
};

// Members of large groups in slot order: group number, suffix, slot; the first slot
// of every group; `share` symbols that the members of a group share at least.
struct Pool {
    uint64_t *keys;
    uint32_t *vals, *slots, *first;
    uint32_t total, groups, share;
};

// One round: sorts the pool by the rank `h` symbols on, with buffers as large as
// the pool was first (`cap`). Ranks and *pool are those after the round; `lookups_done`
// runs once all lookups of ranks have been enqueued, before any rank changes.
struct PoolRoom {
    uint64_t *keys;
    uint32_t *vals, *slots, *radix, *tcount, *hcount, *stmp;
    uint32_t cap;
};
template <typename F>
lor_status pool_round(Pool *pool, PoolRoom *room, uint32_t h, uint32_t n, int32_t *sa, uint32_t *rank, uint32_t *hdr,
                      F lookups_done, hipStream_t s) {
    const uint32_t total = pool->total, tiles = div_up(total, kPoolTile);
    const int rank_bits = bits_for(n);
    LOR_LAUNCH("k_pool_keys", 24.0 * total, s,
               hipLaunchKernelGGL(k_pool_keys, dim3(div_up(total, kBlock)), dim3(kBlock), 0, s, pool->keys, pool->vals,
                                  total, h, n, rank_bits, rank));
    LOR_TRY(lookups_done());
    bool alt;
    LOR_TRY(radix_sort<uint64_t>(pool->keys, pool->vals, room->keys, room->vals, total, 0,
                                 rank_bits + bits_for(pool->groups - 1), room->radix, s, &alt));
    if (!alt) {   // the sorted pool is where the next one is not
        std::swap(pool->keys, room->keys);
        std::swap(pool->vals, room->vals);
    }
    const PoolItems sorted{room->keys, room->vals, pool->slots, total};
    LOR_LAUNCH("k_pool_count", 8.0 * total, s,
               hipLaunchKernelGGL(k_pool_count, dim3(tiles), dim3(kBlock), 0, s, sorted, room->tcount, room->hcount));
    LOR_TRY(scan_exclusive(room->tcount, tiles, room->stmp, hdr + kWordTied, s));
    LOR_TRY(scan_exclusive(room->hcount, tiles, room->stmp, hdr + kWordHeads, s));
    LOR_LAUNCH("k_pool_collect", 44.0 * total, s,
               hipLaunchKernelGGL(k_pool_collect, dim3(tiles), dim3(kBlock), 0, s, sorted, room->tcount, room->hcount,
                                  room->cap, n, sa, rank, pool->keys, pool->vals, room->slots, pool->first));
    std::swap(pool->slots, room->slots);
    PrefixHdr w;
    LOR_TRY(read_header(hdr, &w, s));
    if (trace_on())
        fprintf(stderr, "[lor] prefix sort: %u suffixes in %u large groups doubled from %u symbols, %u left\n", total,
                pool->groups, h, w.word[kWordTied]);
    if (w.word[kWordTied] > total || w.word[kWordHeads] > w.word[kWordTied] / 2) {
        set_error("internal: %u suffixes in %u large groups of %u", w.word[kWordTied], w.word[kWordHeads], total);
        return LOR_EINVAL;
    }
    pool->total = w.word[kWordTied];
    pool->groups = w.word[kWordHeads];
    if (pool->total)
        LOR_LAUNCH("k_pool_ranks", 16.0 * pool->total, s,
                   hipLaunchKernelGGL(k_pool_ranks, dim3(div_up(pool->total, kBlock)), dim3(kBlock), 0, s, pool->keys,
                                      pool->vals, pool->first, pool->total, n, rank));
    return LOR_OK;
}

// Settles what is open: `count` suffixes in runs of up to kSmall, compared up to
// `from` symbols so far (0: not yet), and the pool's. *done stays false when the workspace
// does not hold the ranks, the budget is spent or the pool costs too much.
template <typename X>
lor_status settle_runs(const X &x, uint32_t count, uint32_t from, Pool pool, uint32_t *open, int32_t *sa, Arena &ar,
                       uint32_t *hdr, uint32_t budget, Spend &spend, hipStream_t s, bool *done) {
    const uint32_t n = x.n;
    RunList list{nullptr, nullptr, n};
    uint32_t words = div_up(n, 32);
    if (n > kIdentityItems && count > 0) {
        // every run has at least one marked slot for each unmarked one
        list.cap = (uint32_t)std::min<uint64_t>(2ull * count, n);
        const uint32_t groups = div_up(words, kOpenWords), lwords = div_up(list.cap, 32);
        uint32_t *slots = ar.take<uint32_t>(list.cap), *bits = ar.take<uint32_t>(lwords);
        uint32_t *counts = ar.take<uint32_t>(groups), *tmp = ar.take<uint32_t>(kScanTmpWords);
        if (ar.overflow) return LOR_OK;
        LOR_LAUNCH("k_open_count", 4.0 * words, s,
                   hipLaunchKernelGGL(k_open_count, dim3(groups), dim3(kBlock), 0, s, open, words, counts));
        LOR_TRY(scan_exclusive(counts, groups, tmp, hdr + kWordItems, s));
        LOR_TRY(zero_words(bits, lwords, s));
        LOR_LAUNCH("k_open_list", 4.0 * words + 4.0 * list.cap, s,
                   hipLaunchKernelGGL(k_open_list, dim3(groups), dim3(kBlock), 0, s, open, words, counts, list.cap,
                                      slots, bits));
        list.slots = slots;
        list.count = hdr + kWordItems;
        open = bits;
        words = lwords;
    }
    uint32_t *was = ar.take<uint32_t>(words);
    if (ar.overflow) return LOR_OK;
    PrefixHdr w;
    // The ranks of all suffixes (a scatter) and the rounds take about 15 ps per
    // suffix of the text and 80 us; comparing an open suffix to its neighbour
    // through kSettle symbols reads some 60 lines, about 1.5 ns: for few only.
    const uint32_t few = n / 128u + 8192u;
    while (count > 0 && (from == 0 || (from == kDeep && count <= few))) {   // at most two steps
        from = count <= few ? kSettle : kDeep;
        LOR_TRY(copy_words(open, was, words, s));
        LOR_TRY(zero_words(hdr + kWordRound, 1, s));
        LOR_TRY(launch_settle(x, list, was, open, sa, from, hdr + kWordRound, hdr, budget, s));
        LOR_TRY(read_header(hdr, &w, s));
        if (trace_on())
            fprintf(stderr, "[lor] prefix sort: %u open suffixes compared up to %u symbols, %u left%s\n", count, from,
                    w.word[kWordRound], w.word[kWordAbort] ? ", given up" : "");
        if (w.word[kWordAbort]) return LOR_OK;
        count = w.word[kWordRound];
    }
    if (count == 0 && pool.total == 0) {
        *done = true;
        return LOR_OK;
    }
    uint32_t *rank = ar.take<uint32_t>(n);
    const size_t mark = ar.mark();
    if (ar.overflow) return LOR_OK;
    if (n <= kDirectRanks) {
        LOR_LAUNCH("k_ranks", 8.0 * n, s,
                   hipLaunchKernelGGL(k_ranks, dim3(grid_for(n)), dim3(kBlock), 0, s, n, sa,
                                      list.slots ? nullptr : open, rank));
    } else {
        uint32_t *tmp[4], *counts;
        for (int i = 0; i < 4; ++i) tmp[i] = ar.take<uint32_t>(n);
        counts = ar.take<uint32_t>(radix_counts_words(n));
        if (ar.overflow) return LOR_OK;
        LOR_TRY(bucketed_scatter(reinterpret_cast<int32_t *>(rank), n, reinterpret_cast<const uint32_t *>(sa), nullptr,
                                 0, n, tmp, counts, s, true));
    }
    auto run_ranks = [&](const uint32_t *before) -> lor_status {
        LOR_LAUNCH("k_run_ranks", 0.25 * list.cap, s,
                   hipLaunchKernelGGL(k_run_ranks, dim3(grid_for(list.cap)), dim3(kBlock), 0, s, list, open, before, n,
                                      sa, rank));
        return LOR_OK;
    };
    if (list.slots) LOR_TRY(run_ranks(open));
    auto double_runs = [&](uint32_t h, uint32_t *left) -> lor_status {
        LOR_TRY(copy_words(open, was, words, s));
        LOR_LAUNCH("k_double", 0.125 * list.cap, s,
                   hipLaunchKernelGGL(k_double, dim3(std::min(div_up(list.cap, kDoubleTile), kDoubleGroups)),
                                      dim3(kBlock), 0, s, list, was, open, n, h, rank, sa, left));
        return LOR_OK;
    };
    uint64_t h = from;   // what the open runs share
    if (pool.total) {
        ar.release(mark);   // the scatter's buffers
        const uint32_t most = div_up(pool.total, kPoolTile);
        PoolRoom room{};
        room.cap = pool.total;
        room.keys = ar.take<uint64_t>(room.cap);
        room.vals = ar.take<uint32_t>(room.cap);
        room.slots = ar.take<uint32_t>(room.cap);
        room.radix = ar.take<uint32_t>(radix_counts_words(room.cap));
        room.tcount = ar.take<uint32_t>(most);
        room.hcount = ar.take<uint32_t>(most);
        room.stmp = ar.take<uint32_t>(kScanTmpWords);
        if (ar.overflow) return LOR_OK;
        LOR_LAUNCH("k_pool_ranks", 16.0 * pool.total, s,
                   hipLaunchKernelGGL(k_pool_ranks, dim3(div_up(pool.total, kBlock)), dim3(kBlock), 0, s, pool.keys,
                                      pool.vals, pool.first, pool.total, n, rank));
        // The pool's groups share less than the open runs at first; from where they
        // share as much both are doubled together.
        for (uint64_t d = pool.share; pool.total > 0; d *= 2) {
            if (d > 2ull * n) {
                set_error("internal: %u suffixes of %u left unordered", pool.total, n);
                return LOR_EINVAL;
            }
            const uint32_t total = pool.total;
            if (!spend.take(total)) return LOR_OK;
            if (count > 0) d = std::min(d, h);
            const bool both = count > 0 && d == h;
            const uint32_t step = (uint32_t)std::min<uint64_t>(d, n);
            LOR_TRY(zero_words(hdr + kWordRound, 1, s));
            auto runs = [&]() -> lor_status { return both ? double_runs(step, hdr + kWordRound) : LOR_OK; };
            LOR_TRY(pool_round(&pool, &room, step, n, sa, rank, hdr, runs, s));
            if (both) {
                LOR_TRY(run_ranks(was));
                h *= 2;
            }
            if (pool.total && !spend.worth(pool.total, 2ull * (total - pool.total))) return LOR_OK;
        }
        if (count == 0) {
            *done = true;
            return LOR_OK;
        }
    }
    constexpr int kPer = 4;   // rounds between read-backs; a round with nothing open is three short launches
    for (;;) {
        LOR_TRY(zero_words(hdr + kWordRound, kPer, s));
        for (int r = 0; r < kPer; ++r, h *= 2) {
            LOR_TRY(double_runs((uint32_t)std::min<uint64_t>(h, n), hdr + kWordRound + r));
            LOR_TRY(run_ranks(was));
        }
        LOR_TRY(read_header(hdr, &w, s));
        if (trace_on())
            fprintf(stderr, "[lor] prefix sort: doubling up to %llu symbols, open=%u\n", (unsigned long long)h,
                    w.word[kWordRound + kPer - 1]);
        if (w.word[kWordRound + kPer - 1] == 0) break;
        if (h > 2ull * n) {
            set_error("internal: %u suffixes of %u left unordered", w.word[kWordRound + kPer - 1], n);
            return LOR_EINVAL;
        }
    }
    *done = true;
    return LOR_OK;
}

lor_status sum_counts(const uint32_t *tcount, const uint32_t *hcount, const uint32_t *ocount, uint32_t tiles,
                      uint32_t *hdr, hipStream_t s) {
    LOR_LAUNCH("k_resolve_totals", 12.0 * tiles, s,
               hipLaunchKernelGGL(k_resolve_totals, dim3(std::min(div_up(tiles, kBlock), kSumGroups)), dim3(kBlock), 0,
                                  s, tcount, hcount, ocount, tiles, hdr));
    return LOR_OK;
}

// bits: key bits; near: near suffixes (left out of the sort). *done stays
// false when DC3 has to build the array.
template <typename X>
lor_status prefix_sa(X x, int bits, uint32_t near, int32_t *sa, Arena &ar, uint32_t *hdr, hipStream_t s,
                     bool *done) {
    constexpr bool kImplicit = !StopAtSep<X>::value;   // every position is sorted: its value is its index
    *done = false;
    const uint32_t m = x.n - near;
    auto tile_of = [](uint32_t count) { return kBlock * (uint32_t)(count <= kResSmall ? kResItemsSmall : kResItems); };
    const uint32_t tiles = div_up(m ? m : 1, tile_of(m));
    // 32 steps over two texts read about 32 lines, some 0.7 ns of the chip's
    // gather rate; DC3 takes 0.25 to 0.4 ns per suffix. Comparisons cost at most
    // about a third of a DC3 run before they are given up.
    const uint32_t budget = x.n / 8 + 65536u;
    Spend spend(x.n);
    const size_t mark = ar.mark();
    struct Release {
        Arena &a;
        size_t m;
        ~Release() { a.release(m); a.overflow = false; }
    } release{ar, mark};
    const uint32_t owords = div_up(x.n, 32);
    const bool identity = x.n <= kIdentityItems;
    uint32_t *open = ar.take<uint32_t>(owords), *was = identity ? ar.take<uint32_t>(owords) : nullptr;
    if (X::kRepeatBits) x.rep = ar.take<uint32_t>(4 * (size_t)div_up(x.n, 128));   // whole 16-byte steps
    const size_t mark_open = ar.mark();
    const RunList all{nullptr, nullptr, x.n};
    uint32_t *ka = ar.take<uint32_t>(m), *va = ar.take<uint32_t>(m), *places = ar.take<uint32_t>(near + 1);
    // sized for every round: the tiles of a smaller count may be smaller, and more
    const uint32_t most = std::max(tiles, div_up(std::min(m, kResSmall), kBlock * kResItemsSmall)) + 1;
    uint64_t *large = ar.take<uint64_t>((size_t)div_up(m, 64) + 64);
    uint32_t *tcount = ar.take<uint32_t>(most), *hcount = ar.take<uint32_t>(most), *ocount = ar.take<uint32_t>(most);
    uint32_t *stmp = ar.take<uint32_t>(kScanTmpWords);
    const size_t half = ar.mark();
    uint32_t *kb = ar.take<uint32_t>(m), *counts = ar.take<uint32_t>(radix_counts_words(m));
    if (ar.overflow) return LOR_OK;
    uint32_t *vb = reinterpret_cast<uint32_t *>(sa);
    if (m > 0) {
        // the sorted pairs end in (ka, va): sa, the other value buffer, receives the order
        const int step = plan().digit_bits, passes = radix_passes(0, bits);
        uint32_t *ki = passes % 2 ? kb : ka, *ko = passes % 2 ? ka : kb;
        uint32_t *vi = passes % 2 ? vb : va, *vo = passes % 2 ? va : vb;
        LOR_TRY(launch_keys(x, ki, vi, OpenBits{open, was}, s));
        for (int sh = 0; sh < bits; sh += step) {
            const uint32_t *in = kImplicit && sh == 0 ? nullptr : vi;
            LOR_TRY(radix_pass<uint32_t>(ki, in, 0, ko, vo, m, sh, std::min(step, bits - sh), counts, s));
            std::swap(ki, ko);
            std::swap(vi, vo);
        }
    }
    if (near) LOR_TRY(launch_near(x, ka, m, sa, places, s));
    GroupKey gk{0, nullptr};
    if (m > 0) {
        auto *resolve = m <= kResSmall ? k_resolve<X, uint32_t, kResItemsSmall> : k_resolve<X, uint32_t, kResItems>;
        LOR_LAUNCH("k_resolve", 12.0 * m, s,
                   hipLaunchKernelGGL(resolve, dim3(tiles), dim3(kBlock), 0, s, x, gk, ka, va, m, sa,
                                      (const uint32_t *)nullptr, places, near, large, tcount, hcount, ocount, open, was));
        LOR_TRY(sum_counts(tcount, hcount, ocount, tiles, hdr, s));
        if (identity) LOR_TRY(launch_settle(x, all, was, open, sa, kDeep, hdr + kWordRound, hdr, budget, s));
    }
    PrefixHdr h;
    LOR_TRY(read_header(hdr, &h, s));
    if (trace_on())
        fprintf(stderr, "[lor] prefix sort: n=%u near=%u symbols=%d bits=%d large groups=%u with %u suffixes%s\n", x.n,
                near, x.K, bits, h.word[kWordHeads], h.word[kWordTied], h.word[kWordAbort] ? ", given up" : "");
    // Rounds over what is still in large groups: collect it, sort it, resolve it.
    const uint64_t *k64 = nullptr;
    const uint32_t *v64 = nullptr, *slots = nullptr;
    uint32_t cur = m;
    Pool pool{};
    pool.share = (uint32_t)x.K;
    for (int round = 0; h.word[kWordTied] > 0 && !h.word[kWordAbort]; ++round) {
        // Most of the text in large groups (one repeat all through, or of
        // long period): DC3's levels shrink it faster than sorts of all of it.
        if (h.word[kWordTied] > x.n / 2) return LOR_OK;
        // Words with many copies lose few of their members to a round of a few
        // symbols; doubling is for them, whose ranks of all suffixes cost as much as a
        // round over one suffix in 64 of the text.
        if (round == kMaxRounds || (round > 0 && h.word[kWordTied] > std::max(cur / 2, x.n / 64))) {
            pool.total = h.word[kWordTied];
            break;
        }
        if (!spend.take(h.word[kWordTied])) return LOR_OK;
        const uint32_t total = h.word[kWordTied], groups = h.word[kWordHeads];
        if (total > cur || groups > total || groups == 0) {
            set_error("internal: %u suffixes in %u large groups of %u", total, groups, cur);
            return LOR_EINVAL;
        }
        // as many symbols as 56 bits hold beside the group number and the repeat code (40 for a
        // small sort, where a pass costs its launches), at least 5
        const int gb = bits_for(groups - 1);
        const int free_bits = std::max((total <= kResSmall ? 40 : 56) - (int)kCodeBits - gb, 15);
        const GroupKey ng{(uint32_t)std::min(free_bits / 3, 10), round ? ar.take<uint32_t>(groups) : nullptr};
        if (round == 0) ar.release(half);   // kb and the counts are free
        uint64_t *k0 = ar.take<uint64_t>(total), *k1 = ar.take<uint64_t>(total);
        uint32_t *v0 = ar.take<uint32_t>(total), *v1 = ar.take<uint32_t>(total), *ns = ar.take<uint32_t>(total);
        const size_t scratch = ar.mark();
        uint32_t *cnt = ar.take<uint32_t>(radix_counts_words(total));
        if (ar.overflow) return LOR_OK;
        const bool csmall = cur <= kResSmall, tsmall = total <= kResSmall;
        const uint32_t ct = div_up(cur, tile_of(cur)), nt = div_up(total, tile_of(total));
        LOR_TRY(scan_exclusive(tcount, ct, stmp, nullptr, s));
        LOR_TRY(scan_exclusive(hcount, ct, stmp, nullptr, s));
        if (round == 0) {
            auto *collect = csmall ? k_group_collect<uint32_t, kResItemsSmall> : k_group_collect<uint32_t, kResItems>;
            LOR_LAUNCH("k_group_collect", 4.0 * cur + 20.0 * total, s,
                       hipLaunchKernelGGL(collect, dim3(ct), dim3(kBlock), 0, s, gk, x.K, ka, va, cur, large, tcount,
                                          hcount, places, near, slots, total, groups, k0, v0, ns,
                                          (uint32_t *)nullptr));
        } else {
            auto *collect = csmall ? k_group_collect<uint64_t, kResItemsSmall> : k_group_collect<uint64_t, kResItems>;
            LOR_LAUNCH("k_group_collect", 8.0 * cur + 24.0 * total, s,
                       hipLaunchKernelGGL(collect, dim3(ct), dim3(kBlock), 0, s, gk, x.K, k64, v64, cur, large, tcount,
                                          hcount, places, near, slots, total, groups, k0, v0, ns,
                                          const_cast<uint32_t *>(ng.off)));
        }
        gk = ng;
        pool.share += gk.ns;
        LOR_LAUNCH("k_group_keys", 20.0 * total, s,
                   hipLaunchKernelGGL(k_group_keys<X>, dim3(div_up(total, kBlock)), dim3(kBlock), 0, s, x, gk, k0, v0,
                                      total, hdr, budget));
        bool alt;
        LOR_TRY(radix_sort<uint64_t>(k0, v0, k1, v1, total, 0, gb + (int)kCodeBits + 3 * (int)gk.ns, cnt, s, &alt));
        k64 = alt ? k1 : k0;
        v64 = alt ? v1 : v0;
        slots = ns;
        cur = total;
        ar.release(scratch);
        LOR_TRY(zero_words(hdr + kWordTied, 2, s));
        auto *resolve = tsmall ? k_resolve<X, uint64_t, kResItemsSmall> : k_resolve<X, uint64_t, kResItems>;
        LOR_LAUNCH("k_resolve", 20.0 * cur, s,
                   hipLaunchKernelGGL(resolve, dim3(nt), dim3(kBlock), 0, s, x, gk, k64, v64, cur, sa, slots,
                                      (const uint32_t *)nullptr, 0u, large, tcount, hcount, ocount, open, was));
        LOR_TRY(sum_counts(tcount, hcount, ocount, nt, hdr, s));
        if (identity) LOR_TRY(launch_settle(x, all, was, open, sa, kDeep, hdr + kWordRound, hdr, budget, s));
        LOR_TRY(read_header(hdr, &h, s));
        if (trace_on())
            fprintf(stderr, "[lor] prefix sort: round %d, %u suffixes; left: large groups=%u with %u%s\n", round, total,
                    h.word[kWordHeads], h.word[kWordTied], h.word[kWordAbort] ? ", given up" : "");
    }
    if (h.word[kWordAbort]) return LOR_OK;
    if (pool.total) {   // after a round: of its sorted groups, the large ones
        pool.groups = h.word[kWordHeads];
        if (pool.total > cur || pool.groups == 0 || pool.groups > pool.total / 2) {
            set_error("internal: %u suffixes in %u large groups of %u", pool.total, pool.groups, cur);
            return LOR_EINVAL;
        }
        if (!spend.worth(pool.total, (uint64_t)(cur - pool.total) * pool.share / gk.ns)) return LOR_OK;
        // the pool goes where ka and va were, below all that it is collected from
        if (18ull * pool.total + 1024u > 8ull * m) return LOR_OK;
        ar.release(mark_open);
        pool.keys = ar.take<uint64_t>(pool.total);
        pool.vals = ar.take<uint32_t>(pool.total);
        pool.slots = ar.take<uint32_t>(pool.total);
        pool.first = ar.take<uint32_t>(pool.total / 2 + 1);
        if (ar.overflow) return LOR_OK;
        const uint32_t ct = div_up(cur, tile_of(cur));
        LOR_TRY(scan_exclusive(tcount, ct, stmp, nullptr, s));
        LOR_TRY(scan_exclusive(hcount, ct, stmp, nullptr, s));
        auto *collect = cur <= kResSmall ? k_group_collect<uint64_t, kResItemsSmall> : k_group_collect<uint64_t, kResItems>;
        LOR_LAUNCH("k_group_collect", 8.0 * cur + 24.0 * pool.total, s,
                   hipLaunchKernelGGL(collect, dim3(ct), dim3(kBlock), 0, s, gk, x.K, k64, v64, cur, large, tcount,
                                      hcount, places, near, slots, pool.total, pool.groups, pool.keys, pool.vals,
                                      pool.slots, pool.first));
        LOR_LAUNCH("k_pool_start", 20.0 * pool.total, s,
                   hipLaunchKernelGGL(k_pool_start, dim3(div_up(pool.total, kBlock)), dim3(kBlock), 0, s, pool.keys,
                                      pool.vals, pool.slots, pool.total, x.n, sa, pool.first));
        LOR_TRY(zero_words(hdr + kWordTied, 2, s));
        return settle_runs(x, h.word[kWordOpen], 0u, pool, open, sa, ar, hdr, budget, spend, s, done);
    }
    const uint32_t left = h.word[identity ? kWordRound : kWordOpen];
    if (left > 0) {
        ar.release(mark_open);
        return settle_runs(x, left, identity ? kDeep : 0u, pool, open, sa, ar, hdr, budget, spend, s, done);
    }
    *done = true;
    return LOR_OK;
}

// Symbols per key for n suffixes of one text: about one suffix per key on
// random DNA, in whole 8-bit digits.
int symbols_for(uint64_t n) {
    if (n <= 1u << 10) return 4;
    if (n <= 1u << 17) return 8;
    if (n <= 1u << 25) return 12;
    return 16;
}

}  // namespace

lor_status prefix_sa_joined(const uint8_t *text, uint32_t n, const int64_t *offsets, uint32_t k, int32_t *sa,
                            Arena &ar, uint32_t *hdr, hipStream_t s, bool *done) {
    Joined x;
    x.t = text;
    x.n = n;
    x.K = symbols_for(n);
    x.k = k;
    x.near = 0;
    for (uint32_t j = 0; j <= k; ++j) x.start[j] = (int32_t)(offsets[j] + j);
    for (uint32_t j = 0; j < k; ++j) x.near += near_of((uint32_t)(offsets[j + 1] - offsets[j]), x.K);
    return prefix_sa(x, 2 * x.K, x.near, sa, ar, hdr, s, done);
}

lor_status prefix_sa_shared(const uint8_t *text, uint32_t n, int32_t *sa, Arena &ar, uint32_t *hdr, hipStream_t s,
                            bool *done) {
    // 6, 10 or 13 symbols base 5 in 14, 24 or 31 bits
    const Shared x{text, n, n <= 1u << 14 ? 6 : n <= 1u << 22 ? 10 : 13};
    return prefix_sa(x, x.K == 6 ? 14 : x.K == 10 ? 24 : 31, 0, sa, ar, hdr, s, done);
}

lor_status prefix_sa_tagged(const uint16_t *text, uint32_t n, uint32_t pairs, const int32_t *start,
                            const int32_t *alen, const int32_t *h_start, const int32_t *h_alen, int32_t *sa,
                            Arena &ar, uint32_t *hdr, hipStream_t s, bool *done) {
    *done = false;
    uint32_t longest = 0;
    for (uint32_t p = 0; p < pairs; ++p) longest = std::max(longest, (uint32_t)(h_start[p + 1] - h_start[p]));
    const int tag = bits_for(pairs - 1);
    // a symbol more than log4 of the longest pair, then up to whole digits
    const int want = tag + bits_for(longest) + 2;
    const int bits = std::min(32, (want + 7) / 8 * 8);
    const int K = std::min((bits - tag) / 2, kMaxK);
    if ((uint64_t)longest >> (2 * K) > 16) return LOR_OK;   // a huge pair among many: too few symbols fit
    const std::unique_ptr<uint32_t[]> below(new (std::nothrow) uint32_t[pairs]);
    if (!below) return LOR_OK;
    uint32_t near = 0;
    for (uint32_t p = 0; p < pairs; ++p) {
        below[p] = near;
        const uint32_t a = (uint32_t)h_alen[p], b = (uint32_t)(h_start[p + 1] - h_start[p]) - a - 2u;
        near += near_of(a, K) + near_of(b, K);
    }
    const size_t mark = ar.mark();
    uint32_t *d_below = ar.take<uint32_t>(pairs);
    lor_status st = LOR_OK;
    if (!ar.overflow) {
        LOR_HIP(hipMemcpyAsync(d_below, below.get(), pairs * sizeof(uint32_t), hipMemcpyHostToDevice, s));
        const Tagged x{text, n, K, pairs, near, start, alen, d_below, nullptr};
        st = prefix_sa(x, tag + 2 * K, near, sa, ar, hdr, s, done);
        // a finished sort has waited for the stream; others may leave before that, with
        // the copy from `below` still to come
        if (!*done) (void)hipStreamSynchronize(s);
    }
    ar.release(mark);
    ar.overflow = false;
    return st;
}

}  // namespace lor
