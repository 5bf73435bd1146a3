// Longest common substring of every query sequence with one reference, on
// gfx950: the shape of Section V's experiments (a reference group against
// many query sequences), with one suffix array for the whole set.
//
// Text: reference, then every query, each followed by the same separator
// (symbol 5 after the byte + 1 shift). Repeated separators leave the suffix
// order well defined, but an LCP may run across one; a query suffix x is
// therefore credited min(lcp, d(x)), d(x) = its distance to its separator.
// (If lcp(x, y) > d(y) for a reference suffix y, x reads a separator at
// d(y) too, so d(x) = d(y); hence min(lcp, d(x), d(y)) = min(lcp, d(x)).)
//
// For a query suffix x at rank r, the longest match with any reference
// suffix is the larger of its LCP with the nearest reference suffix above
// and below in rank order (the minimum of the LCP array between them). Two
// segmented scans over the ranks give both: forward, the minimum LCP since
// the last reference rank; backward, up to the next one. A query's answer
// is the largest credited match, the smallest query offset among equals
// (a 64-bit atomicMax), and a reference offset at which that
// match occurs (the neighbour that gave it).
#include <algorithm>
#include <climits>
#include <vector>

#include "lor_internal.hpp"

namespace lor {

namespace {

constexpr uint32_t kRqItems = 16;                      // consecutive ranks per thread
constexpr uint32_t kRqTile = kBlock * kRqItems;
constexpr int kRqScanThreads = 1024;                   // one workgroup scans the tile states

// Largest j in [0, count) with start[j] <= x.
__device__ __forceinline__ uint32_t seq_at(const int32_t *__restrict__ start, uint32_t count, uint32_t x) {
    uint32_t lo = 0, hi = count - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if ((uint32_t)start[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Sequence lookups go through buckets of 2^kRqBucketShift positions:
// tab[b] = the sequence holding position min(b << shift, N - 1), b = 0..nb
// with nb = ceil(N / 2^shift). Sequences only grow with the position, so the
// one holding x lies in [tab[x >> shift], tab[(x >> shift) + 1]]: a search
// of a few starts (queries are at least tens of bases) instead of all of
// them.
constexpr uint32_t kRqBucketShift = 6;

__global__ __launch_bounds__(kBlock) void k_rq_buckets(const int32_t *__restrict__ start, uint32_t S, uint32_t N,
                                                       uint32_t nb, int32_t *__restrict__ tab) {
    for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b <= nb; b += gridDim.x * kBlock)
        tab[b] = (int32_t)seq_at(start, S, min((uint64_t)b << kRqBucketShift, (uint64_t)N - 1));
}

// Largest j with start[j] <= x, for x < N.
__device__ __forceinline__ uint32_t seq_fast(const int32_t *__restrict__ start, const int32_t *__restrict__ tab,
                                             uint32_t x) {
    const uint32_t b = x >> kRqBucketShift;
    uint32_t lo = (uint32_t)tab[b], hi = (uint32_t)tab[b + 1];
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if ((uint32_t)start[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// start[j] = joined start of sequence j (0 = reference), start[S] = N. A
// thread writes kRqJoinBytes consecutive positions; when they are all bases
// of one sequence they are the input shifted by the sequence index (aligned
// 8-byte loads, a funnel shift, the base check on whole words), otherwise
// they go position by position.
constexpr uint32_t kRqJoinBytes = 16;

__global__ __launch_bounds__(kBlock) void k_rq_join(const uint8_t *__restrict__ seqs, const int32_t *__restrict__ start,
                                                    const int32_t *__restrict__ tab, uint32_t N, uint32_t total,
                                                    uint8_t *__restrict__ out, uint32_t *__restrict__ err) {
    uint32_t bad = 0;
    const uint32_t stride = gridDim.x * kBlock * kRqJoinBytes;
    for (uint32_t p0 = (blockIdx.x * kBlock + threadIdx.x) * kRqJoinBytes; p0 < N; p0 += stride) {
        uint32_t j = seq_fast(start, tab, p0);
        const uint32_t from = p0 - j;
        if (p0 + kRqJoinBytes < (uint32_t)start[j + 1] && from >= 8u && from + 24u <= total) {
            const uintptr_t addr = reinterpret_cast<uintptr_t>(seqs + from);
            const uint64_t *w = reinterpret_cast<const uint64_t *>(addr & ~(uintptr_t)7);
            const uint32_t sh = (uint32_t)(addr & 7u) * 8u;
            const uint64_t w0 = w[0], w1 = w[1], w2 = w[2];
            const uint64_t lo = sh ? (w0 >> sh) | (w1 << (64u - sh)) : w0;
            const uint64_t hi = sh ? (w1 >> sh) | (w2 << (64u - sh)) : w1;
            bad |= ((lo | hi) & 0xfcfcfcfcfcfcfcfcull) != 0;
            *reinterpret_cast<uint4 *>(out + p0) =   // p0 is a multiple of 16; the text buffer is 16-byte aligned
                make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
            continue;
        }
        for (uint32_t u = 0; u < kRqJoinBytes && p0 + u < N; ++u) {
            const uint32_t p = p0 + u;
            while ((uint32_t)start[j + 1] <= p) ++j;
            uint32_t c;
            if (p + 1 == (uint32_t)start[j + 1]) {
                c = 4u;
            } else {
                c = seqs[p - j];
                bad |= c > 3u;
            }
            out[p] = (uint8_t)c;
        }
    }
    if (__any(bad) && dev::lane_id() == 0) atomicOr(err, 1u);
}

// State of a run of ranks, seen from one end: the reference rank nearest to it
// (-1: none) and the minimum LCP on the way there (over the whole run if none).
// Seen from behind the run, that leaves the reference rank's own LCP out; from
// in front of it, it counts.
struct Near {
    int32_t m, at;
};

__device__ __forceinline__ Near no_near() { return Near{INT_MAX, -1}; }
__device__ __forceinline__ Near comb(const Near &far, const Near &near) {
    return near.at >= 0 ? near : Near{min(far.m, near.m), far.at};
}

struct RankItem {
    int32_t sa, lcp;
    bool ref;
};

// Target sequence: joined positions [tlo, thi) (its separator at thi).
struct Target {
    uint32_t lo, hi, seq;
};

// A thread's kRqItems consecutive ranks, from r0 (a multiple of kRqItems) on.
__device__ __forceinline__ void rank_items(const int32_t *__restrict__ sa, const int32_t *__restrict__ lcp, uint32_t n,
                                           const Target &tg, uint32_t r0, RankItem *it) {
    if (r0 < n && n - r0 >= kRqItems) {
#pragma unroll
        for (uint32_t k = 0; k < kRqItems; k += 4) {
            const int4 a = *reinterpret_cast<const int4 *>(sa + r0 + k);
            const int4 l = *reinterpret_cast<const int4 *>(lcp + r0 + k);
            it[k].sa = a.x, it[k + 1].sa = a.y, it[k + 2].sa = a.z, it[k + 3].sa = a.w;
            it[k].lcp = l.x, it[k + 1].lcp = l.y, it[k + 2].lcp = l.z, it[k + 3].lcp = l.w;
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < kRqItems; ++k) {
            it[k].sa = r0 + k < n ? sa[r0 + k] : -1;
            it[k].lcp = r0 + k < n ? lcp[r0 + k] : 0;   // behind the last rank: no match
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < kRqItems; ++k) it[k].ref = (uint32_t)it[k].sa >= tg.lo && (uint32_t)it[k].sa < tg.hi;
}

__device__ __forceinline__ Near from_behind(const RankItem &it, uint32_t r) {
    return it.ref ? Near{INT_MAX, (int32_t)r} : Near{it.lcp, -1};
}
__device__ __forceinline__ Near from_front(const RankItem &it, uint32_t r) {
    return Near{it.lcp, it.ref ? (int32_t)r : -1};
}

// States of a thread's ranks.
__device__ __forceinline__ void fold(const RankItem *it, uint32_t r0, Near *f, Near *b) {
    *f = *b = no_near();
#pragma unroll
    for (uint32_t k = 0; k < kRqItems; ++k) *f = comb(*f, from_behind(it[k], r0 + k));
#pragma unroll
    for (uint32_t k = kRqItems; k-- > 0;) *b = comb(*b, from_front(it[k], r0 + k));
}

// Exclusive scan of per-thread states across a workgroup of NT threads, in
// thread order or (kBack) from the last thread down: shuffles in the waves, LDS
// between them. s: one entry per wave.
template <int NT, bool kBack>
__device__ __forceinline__ Near block_excl(Near v, Near *s) {
    constexpr uint32_t kWaves = NT / kWave;
    const uint32_t lane = dev::lane_id(), w = threadIdx.x / kWave;
#pragma unroll
    for (uint32_t off = 1; off < (uint32_t)kWave; off <<= 1) {
        const Near o = kBack ? Near{__shfl_down(v.m, off, kWave), __shfl_down(v.at, off, kWave)}
                             : Near{__shfl_up(v.m, off, kWave), __shfl_up(v.at, off, kWave)};
        if (kBack ? lane + off < (uint32_t)kWave : lane >= off) v = comb(o, v);
    }
    if (lane == (kBack ? 0u : (uint32_t)kWave - 1u)) s[w] = v;
    Near x = kBack ? Near{__shfl_down(v.m, 1, kWave), __shfl_down(v.at, 1, kWave)}
                   : Near{__shfl_up(v.m, 1, kWave), __shfl_up(v.at, 1, kWave)};
    if (lane == (kBack ? (uint32_t)kWave - 1u : 0u)) x = no_near();
    __syncthreads();
    Near carry = no_near();
    if (kBack)
        for (uint32_t i = kWaves; i-- > w + 1;) carry = comb(carry, s[i]);
    else
        for (uint32_t i = 0; i < w; ++i) carry = comb(carry, s[i]);
    return comb(carry, x);
}

// Forward and backward states of every tile of kRqTile ranks. Reads the ranks
// once, 16 bytes a load (46M ranks: 558 us with 4-byte loads, each rank twice,
// and LDS scans).
__global__ __launch_bounds__(kBlock) void k_rq_tiles(const int32_t *__restrict__ sa, const int32_t *__restrict__ lcp,
                                                     uint32_t n, Target tg, Near *__restrict__ tf,
                                                     Near *__restrict__ tb) {
    __shared__ Near s_f[kBlock / kWave], s_b[kBlock / kWave];
    const uint32_t r0 = blockIdx.x * kRqTile + threadIdx.x * kRqItems;
    RankItem it[kRqItems];
    rank_items(sa, lcp, n, tg, r0, it);
    Near f, b;
    fold(it, r0, &f, &b);
    const Near fe = block_excl<kBlock, false>(f, s_f), be = block_excl<kBlock, true>(b, s_b);
    if (threadIdx.x == kBlock - 1) tf[blockIdx.x] = comb(fe, f);
    if (threadIdx.x == 0) tb[blockIdx.x] = comb(be, b);
}

// Tile states -> the state of everything before (forward) and after
// (backward) every tile. One workgroup; thread i folds a contiguous run.
__global__ __launch_bounds__(kRqScanThreads) void k_rq_tile_scan(Near *__restrict__ tf, Near *__restrict__ tb,
                                                                 uint32_t tiles) {
    __shared__ Near s_f[kRqScanThreads / kWave], s_b[kRqScanThreads / kWave];
    const uint32_t per = (tiles + kRqScanThreads - 1) / kRqScanThreads;
    const uint32_t t0 = min(tiles, threadIdx.x * per), t1 = min(tiles, t0 + per);
    Near f = no_near(), b = no_near();
#pragma unroll 4
    for (uint32_t t = t0; t < t1; ++t) f = comb(f, tf[t]);
#pragma unroll 4
    for (uint32_t t = t1; t > t0; --t) b = comb(b, tb[t - 1]);
    f = block_excl<kRqScanThreads, false>(f, s_f);
    b = block_excl<kRqScanThreads, true>(b, s_b);
    for (uint32_t t = t0; t < t1; ++t) {
        const Near x = tf[t];
        tf[t] = f;
        f = comb(f, x);
    }
    for (uint32_t t = t1; t > t0; --t) {
        const Near x = tb[t - 1];
        tb[t - 1] = b;
        b = comb(b, x);
    }
}

// Per rank: the credited match of every suffix of another sequence j with the
// target, folded into best[j * stride + base] = max(m << 32 | ~offset), in three
// passes, each of which only looks up (a table, two starts, the best so far:
// random reads, 975 us a pass for 42M query suffixes) what can still matter:
//   kStrong: the ranks whose match is at least `floor` symbols, some more than
//     a random text of the target's size shares with a suffix. Most sequences
//     then have their best, which no shorter match can beat.
//   kWeak: the other ranks of the sequences left (bits of their positions set
//     in `pos`); nothing when there are none.
//   kEmit: the rank that holds a slot's best writes the record: bits of the
//     winning positions are set in `pos`, and no rank below the smallest best
//     (word[1] = its complement) can hold one.
// word[0]: sequences left for kWeak.
enum RqPass { kStrong, kWeak, kEmit };
template <RqPass PASS>
__global__ __launch_bounds__(kBlock) void k_rq_ranks(const int32_t *__restrict__ sa, const int32_t *__restrict__ lcp,
                                                     uint32_t n, Target tg, const int32_t *__restrict__ start,
                                                     const int32_t *__restrict__ tab, uint32_t S,
                                                     const Near *__restrict__ pre, const Near *__restrict__ post,
                                                     int32_t floor, const uint32_t *__restrict__ word,
                                                     const uint32_t *__restrict__ pos, uint32_t stride, int32_t base,
                                                     unsigned long long *__restrict__ best,
                                                     lor_overlap *__restrict__ out) {
    __shared__ Near s_f[kBlock / kWave], s_b[kBlock / kWave];
    if (PASS == kWeak && word[0] == 0) return;
    int32_t least = PASS == kEmit ? (int32_t)~word[1] : PASS == kWeak ? 1 : floor;
    least = max(least, 1);
    const uint32_t r0 = blockIdx.x * kRqTile + threadIdx.x * kRqItems;
    RankItem it[kRqItems];
    rank_items(sa, lcp, n, tg, r0, it);
    Near f, b;
    fold(it, r0, &f, &b);
    f = comb(pre[blockIdx.x], block_excl<kBlock, false>(f, s_f));
    b = comb(post[blockIdx.x], block_excl<kBlock, true>(b, s_b));
    int32_t up[kRqItems], up_at[kRqItems];
#pragma unroll
    for (uint32_t k = 0; k < kRqItems; ++k) {
        f = comb(f, from_behind(it[k], r0 + k));
        up[k] = f.at >= 0 ? f.m : 0;
        up_at[k] = f.at;
    }
#pragma unroll
    for (uint32_t k = kRqItems; k-- > 0;) {
        const int32_t down = b.at >= 0 ? b.m : 0, down_at = b.at;
        b = comb(b, from_front(it[k], r0 + k));
        const uint32_t x = (uint32_t)it[k].sa;
        const int32_t mx = max(up[k], down);
        if (r0 + k >= n || mx < least || (PASS == kWeak && mx >= floor)) continue;
        if (x >= tg.lo && x <= tg.hi) continue;   // target suffix or its separator
        if (x >= n || (PASS != kStrong && !((pos[x >> 5] >> (x & 31u)) & 1u))) continue;
        const uint32_t j = seq_fast(start, tab, x);
        if (j >= S || j == tg.seq) continue;
        const uint32_t d = (uint32_t)start[j + 1] - 1u - x;   // distance to its own separator
        const int32_t m = min(mx, (int32_t)d);
        if (m <= 0) continue;
        const uint32_t off = x - (uint32_t)start[j];
        const unsigned long long key = ((unsigned long long)(uint32_t)m << 32) | (0xffffffffu - off);
        const int64_t slot = (int64_t)j * stride + base;
        if (PASS != kEmit) {
            // best only grows: a stale read can only let a redundant atomic through
            if (key > __hip_atomic_load(&best[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&best[slot], key);
        } else if (best[slot] == key) {
            const int32_t at = up[k] >= down ? up_at[k] : down_at;   // the neighbour that gave m
            lor_overlap rec;
            rec.length = m;
            rec.seq_p = (int32_t)j;
            rec.off_p = off;
            rec.seq_q = (int32_t)tg.seq;
            rec.off_q = (at >= 0 && (uint32_t)at < n) ? sa[at] - (int32_t)tg.lo : -1;
            out[slot] = rec;
        }
    }
}

// Sets the positions of every sequence without a match of `floor` symbols, one
// workgroup per sequence; *left counts them.
__global__ __launch_bounds__(kBlock) void k_rq_left(const int32_t *__restrict__ start, uint32_t S, Target tg,
                                                    int32_t floor, uint32_t stride, int32_t base,
                                                    const unsigned long long *__restrict__ best,
                                                    uint32_t *__restrict__ pos, uint32_t *__restrict__ left) {
    uint32_t mine = 0;
    for (uint32_t j = blockIdx.x; j < S; j += gridDim.x) {
        if (j == tg.seq || (int32_t)(best[(int64_t)j * stride + base] >> 32) >= floor) continue;
        const uint32_t lo = (uint32_t)start[j], hi = (uint32_t)start[j + 1];   // lo < hi: the separator is included
        for (uint32_t w = lo / 32u + threadIdx.x; w <= (hi - 1u) / 32u; w += kBlock) {
            uint32_t v = 0xffffffffu;
            if (w == lo / 32u) v &= 0xffffffffu << (lo & 31u);
            if (w == (hi - 1u) / 32u) v &= 0xffffffffu >> (31u - ((hi - 1u) & 31u));
            atomicOr(&pos[w], v);
        }
        ++mine;
    }
    if (threadIdx.x == 0 && mine) atomicAdd(left, mine);
}

// Sets the position of every slot's best match; *least gets the complement of
// the smallest of their lengths.
__global__ __launch_bounds__(kBlock) void k_rq_winners(const int32_t *__restrict__ start, uint32_t S, Target tg,
                                                       uint32_t stride, int32_t base,
                                                       const unsigned long long *__restrict__ best, uint32_t n,
                                                       uint32_t *__restrict__ pos, uint32_t *__restrict__ least) {
    uint32_t mine = 0;
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < S; j += gridDim.x * kBlock) {
        if (j == tg.seq) continue;
        const unsigned long long k = best[(int64_t)j * stride + base];
        if (k == 0) continue;   // no match
        const uint32_t x = (uint32_t)start[j] + (0xffffffffu - (uint32_t)k);
        if (x < n) atomicOr(&pos[x >> 5], 1u << (x & 31u));
        mine = max(mine, ~(uint32_t)(k >> 32));
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) mine = max(mine, (uint32_t)__shfl_xor((int)mine, off, kWave));
    if (dev::lane_id() == 0 && mine) atomicMax(least, mine);
}

__global__ __launch_bounds__(kBlock) void k_rq_init(uint32_t Q, unsigned long long *__restrict__ best,
                                                    lor_overlap *__restrict__ out) {
    for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < Q; q += gridDim.x * kBlock) {
        best[q] = 0ull;
        lor_overlap rec;
        rec.length = 0;
        rec.seq_p = -1;
        rec.seq_q = -1;
        rec.off_p = -1;
        rec.off_q = -1;
        out[q] = rec;
    }
}

struct RqLayout {
    uint8_t *text;
    int32_t *sa, *lcp, *start, *tab;
    unsigned long long *best;
    Near *tf, *tb;
};

lor_status rq_carve(Arena &ar, uint64_t N, uint32_t S, RqLayout *L) {
    const uint32_t tiles = div_up(N ? N : 1, kRqTile);
    LOR_TAKE(ar, uint8_t, N + 16, L->text);
    LOR_TAKE(ar, int32_t, N, L->sa);
    LOR_TAKE(ar, int32_t, N, L->lcp);
    LOR_TAKE(ar, int32_t, (size_t)S + 1, L->start);
    LOR_TAKE(ar, int32_t, (size_t)div_up(N ? N : 1, 1u << kRqBucketShift) + 1, L->tab);
    LOR_TAKE(ar, unsigned long long, S, L->best);
    LOR_TAKE(ar, Near, tiles, L->tf);
    LOR_TAKE(ar, Near, tiles, L->tb);
    return LOR_OK;
}

// Matches of every other sequence's suffixes with one target sequence:
// tile states, their scan, then the per-rank passes.
lor_status target_scan(const int32_t *sa, const int32_t *lcp, uint32_t n, Target tg, const int32_t *start,
                       const int32_t *tab, uint32_t S, uint32_t stride, int32_t base, Near *tf, Near *tb,
                       unsigned long long *best, lor_overlap *out, Arena &ar, hipStream_t s) {
    const uint32_t tiles = div_up(n, kRqTile), words = div_up(n, 32);
    uint32_t *weak, *won, *word;
    LOR_TAKE(ar, uint32_t, 2 * (size_t)words + 2, weak);
    won = weak + words;
    word = won + words;
    // A suffix's longest match with a random target of L bases is log4 L or a
    // symbol less or more: 3% to 12% of the suffixes reach the rounded log4 L and
    // two more, and of some hundred in a row few have none. (One less: 425 us
    // strong and 212 weak for 42M suffixes of 64k queries, against 342 and 252.)
    int32_t floor = 1;
    for (uint64_t l = 2; 5 * l < 7ull * (tg.hi - tg.lo) && floor < 24; l *= 4) ++floor;   // 7 / 5: root of 2
    floor += floor > 1;
    LOR_TRY(zero_words(weak, 2 * words + 2, s));
    LOR_LAUNCH("k_rq_tiles", 8.0 * n, s,
               hipLaunchKernelGGL(k_rq_tiles, dim3(tiles), dim3(kBlock), 0, s, sa, lcp, n, tg, tf, tb));
    LOR_LAUNCH("k_rq_tile_scan", 32.0 * tiles, s,
               hipLaunchKernelGGL(k_rq_tile_scan, dim3(1), dim3(kRqScanThreads), 0, s, tf, tb, tiles));
    LOR_LAUNCH("k_rq_ranks", 8.0 * n, s,
               hipLaunchKernelGGL(k_rq_ranks<kStrong>, dim3(tiles), dim3(kBlock), 0, s, sa, lcp, n, tg, start, tab, S,
                                  tf, tb, floor, word, weak, stride, base, best, out));
    if (floor > 1) {
        LOR_LAUNCH("k_rq_left", 8.0 * S, s,
                   hipLaunchKernelGGL(k_rq_left, dim3(std::min(S, 8192u)), dim3(kBlock), 0, s, start, S, tg, floor,
                                      stride, base, best, weak, word));
        LOR_LAUNCH("k_rq_ranks", 8.0 * n, s,
                   hipLaunchKernelGGL(k_rq_ranks<kWeak>, dim3(tiles), dim3(kBlock), 0, s, sa, lcp, n, tg, start, tab,
                                      S, tf, tb, floor, word, weak, stride, base, best, out));
    }
    LOR_LAUNCH("k_rq_winners", 12.0 * S, s,
               hipLaunchKernelGGL(k_rq_winners, dim3(grid_for(S)), dim3(kBlock), 0, s, start, S, tg, stride, base, best,
                                  n, won, word + 1));
    LOR_LAUNCH("k_rq_ranks", 8.0 * n, s,
               hipLaunchKernelGGL(k_rq_ranks<kEmit>, dim3(tiles), dim3(kBlock), 0, s, sa, lcp, n, tg, start, tab, S, tf,
                                  tb, floor, word, won, stride, base, best, out));
    return LOR_OK;
}

}  // namespace

size_t refq_workspace(uint64_t total_bases, uint32_t num_queries) {
    const uint32_t S = num_queries + 1;
    const uint64_t N = total_bases + S;
    Arena ar;   // measuring
    ar.top = kHeaderBytes;
    RqLayout L;
    if (rq_carve(ar, N, S, &L) != LOR_OK) return 0;
    size_t phase = dc3_workspace_bound(N);
    phase = phase > lcp_workspace(N) + 4096 ? phase : lcp_workspace(N) + 4096;
    return ar.top + phase + 4096;
}

lor_status refq_overlap(const uint8_t *seqs, const int64_t *offsets, uint32_t Q, lor_overlap *out, void *ws,
                        size_t ws_bytes, hipStream_t s) {
    const uint32_t S = Q + 1;
    std::vector<int32_t> h_start(S + 1);
    uint64_t N = 0;
    for (uint32_t j = 0; j < S; ++j) {
        h_start[j] = (int32_t)N;
        N += (uint64_t)(offsets[j + 1] - offsets[j]) + 1;
    }
    h_start[S] = (int32_t)N;
    const uint32_t ref_len = (uint32_t)(offsets[1] - offsets[0]);

    Arena ar;
    ar.base = static_cast<char *>(ws);
    ar.cap = ws_bytes;
    ar.top = kHeaderBytes;
    uint32_t *hdr = static_cast<uint32_t *>(ws);
    RqLayout L;
    LOR_TRY(rq_carve(ar, N, S, &L));
    const size_t phase = ar.mark();

    LOR_HIP(hipMemcpyAsync(L.start, h_start.data(), (S + 1) * sizeof(int32_t), hipMemcpyHostToDevice, s));
    LOR_TRY(zero_words(hdr, 16, s));
    LOR_LAUNCH("k_rq_init", 40.0 * Q, s,
               hipLaunchKernelGGL(k_rq_init, dim3(grid_for(Q)), dim3(kBlock), 0, s, Q, L.best, out));
    const uint32_t nb = div_up(N, 1u << kRqBucketShift);
    LOR_LAUNCH("k_rq_buckets", 4.0 * (nb + 1), s,
               hipLaunchKernelGGL(k_rq_buckets, dim3(grid_for(nb + 1)), dim3(kBlock), 0, s, L.start, S, (uint32_t)N,
                                  nb, L.tab));
    LOR_LAUNCH("k_rq_join", 2.0 * N, s,
               hipLaunchKernelGGL(k_rq_join, dim3(grid_for(div_up(N, kRqJoinBytes))), dim3(kBlock), 0, s, seqs,
                                  L.start, L.tab, (uint32_t)N, (uint32_t)(N - S), L.text, hdr));
    // symbols byte + 1: bases 1..4, separator 5
    bool done = false;
    LOR_TRY(prefix_sa_shared(L.text, (uint32_t)N, L.sa, ar, hdr, s, &done));
    if (!done) LOR_TRY(dc3_u8(L.text, (uint32_t)N, 5u, L.sa, ar, hdr, s));
    ar.release(phase);
    LOR_TRY(lcp_build(L.text, (uint32_t)N, L.sa, L.lcp, nullptr, ar, s, S));
    ar.release(phase);
    LOR_TRY(target_scan(L.sa, L.lcp, (uint32_t)N, Target{0u, ref_len, 0u}, L.start, L.tab, S, 1u, -1, L.tf, L.tb,
                        L.best, out, ar, s));
    LOR_HIP(hipStreamSynchronize(s));   // the host table must outlive its copy
    return LOR_OK;
}

}  // namespace lor
