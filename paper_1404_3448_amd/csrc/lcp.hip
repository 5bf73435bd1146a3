// LCP array on gfx950 (Section III, Table IV: LCP[r] = lcp of the suffixes
// at ranks r-1 and r; the paper cites Kasai et al. for its construction).
//
// Kasai's method walks the text and needs SA and LCP permuted into text order
// and back, two sorts' worth of passes around one random text read per suffix.
// Neighbouring suffixes of DNA differ within a few dozen symbols, though, so
//   window : every rank reads the first bytes of its own suffix (the one
//            random read per suffix that is left) and takes its predecessor's
//            from the neighbouring lane; LCPs below the window's length are
//            final, and longer ones are marked. Every S-th text position i
//            also notes Phi[i] = SA[rank - 1];
//   plcp   : PLCP[i] = lcp(i, Phi[i]) of those sampled positions only. A
//            sample whose first S symbols agree and whose successor i + S has
//            Phi[i + S] = Phi[i] + S is linked to it: PLCP[i] = PLCP[i + S] + S;
//            the others compare their texts;
//   links  : the end of every chain of links, by scans over 64-sample words and
//            blocks of 64 of them, so a copy of any length is compared only where it ends;
//   finish : a marked rank whose Phi lies on the diagonal of the sample before
//            or behind its position follows from that; others start from
//            Kasai's bound PLCP[i + d] >= PLCP[i] - d at the sample before, so
//            a long repeat costs a rank a few symbols at most.
// LCP is written in rank order throughout. ISA, when wanted, is a scatter of
// its own.
//
// The window kernels are bound by their random reads: 19.3 ms at 2^30 suffixes, 55
// G/s, where random 8-byte reads reach 45 to 51 on tables of 256 MB and more.
// LCP + ISA against the text-order method it replaces: 1,000 symbols 96 -> 36 us,
// 100k 296 -> 37 us, 1M 483 -> 60 us, 16M 1.21 -> 0.53 ms, 256M 14.8 -> 8.6 ms; two
// identical sequences of 2M bases 75 -> 0.11 ms.
#include <algorithm>

#include "lor_internal.hpp"

namespace lor {

namespace {

constexpr uint32_t kMarked = 0x80000000u;
// ISA as plain stores from the window kernel up to here, as a bucketed scatter
// above: random 4-byte stores cost little while ISA stays in the caches, and
// the scatter takes about ten launches. LCP + ISA, plain against bucketed: 1M
// 248 / 279 us, 16M 805 / 849 us, 32M 1589 / 1459 us, 256M 16.7 / 10.4 ms.
constexpr uint32_t kDirectIsa = 1u << 24;

struct __attribute__((packed, aligned(1))) Chunk {
    uint64_t w[1];
};

// Symbols that the window kernel looks at: 24 bytes of a byte text (random DNA
// of 2^30 bases has neighbours that agree on about 15 symbols, practically
// never on 24; 24 bytes straddle a 64-byte line less often than 32), 32 bytes
// of a 16-bit text.
template <typename CH> struct Win {
    static constexpr int words = sizeof(CH) == 1 ? 3 : 4;
    static constexpr uint32_t symbols = 8 * words / sizeof(CH);
};

template <typename CH>
__device__ __forceinline__ void read_window(const CH *__restrict__ t, uint32_t n, uint32_t i, uint64_t *w) {
    constexpr int per = 8 / sizeof(CH);
    if (i < n && n - i >= Win<CH>::symbols) {
#pragma unroll
        for (int c = 0; c < Win<CH>::words; ++c) w[c] = reinterpret_cast<const Chunk *>(t + i)[c].w[0];
        return;
    }
#pragma unroll
    for (int c = 0; c < Win<CH>::words; ++c) {
        uint64_t v = 0;
        for (int d = 0; d < per; ++d) {
            const uint32_t o = c * per + d;
            v |= (uint64_t)((i < n && o < n - i) ? t[i + o] : CH(0)) << (8 * sizeof(CH) * d);
        }
        w[c] = v;
    }
}

constexpr int kLcpItems = 4;

// DIRECT: ISA is stored from here.
template <typename CH, bool DIRECT>
__global__ __launch_bounds__(kBlock) void k_lcp_window(const CH *__restrict__ t, uint32_t n,
                                                       const int32_t *__restrict__ sa, int32_t *__restrict__ lcp,
                                                       uint32_t *__restrict__ phi, int32_t *__restrict__ isa,
                                                       uint32_t shift) {
    constexpr int NW = Win<CH>::words;
    constexpr uint32_t per = 8 / sizeof(CH), WS = Win<CH>::symbols;
    const uint32_t base = blockIdx.x * (kBlock * kLcpItems), lane = threadIdx.x & 63u;
    uint32_t p[kLcpItems], q[kLcpItems];
    uint64_t w[kLcpItems][NW], e[kLcpItems][NW];   // e: lane 0's predecessor
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        const uint32_t r = base + k * kBlock + threadIdx.x;
        p[k] = r < n ? min((uint32_t)sa[r], n - 1u) : 0u;
        q[k] = (lane == 0 && r > 0 && r < n) ? min((uint32_t)sa[r - 1], n - 1u) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) read_window(t, n, p[k], w[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kLcpItems; ++k) read_window(t, n, q[k], e[k]);
    }
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        const uint32_t r = base + k * kBlock + threadIdx.x;
        const uint32_t pj = (uint32_t)__shfl_up((int)p[k], 1, kWave);
        const uint32_t j = lane == 0 ? q[k] : pj;
        uint32_t l = 0;
        bool open = true;
#pragma unroll
        for (int c = 0; c < NW; ++c) {
            const uint64_t up = __shfl_up(w[k][c], 1, kWave);
            const uint64_t x = w[k][c] ^ (lane == 0 ? e[k][c] : up);
            if (open) l += x ? (uint32_t)__builtin_ctzll(x) / (8u * (uint32_t)sizeof(CH)) : per;
            open = open && x == 0;
        }
        if (r >= n) continue;
        const uint32_t i = p[k];
        if (r == 0) {
            lcp[0] = 0;
        } else {
            const uint32_t lim = n - max(i, j);   // a window past the end reads zeros
            lcp[r] = (int32_t)(open && lim > WS ? WS | kMarked : min(l, lim));
        }
        if ((i & ((1u << shift) - 1u)) == 0) phi[i >> shift] = r ? j : 0xffffffffu;
        if constexpr (DIRECT) isa[i] = (int32_t)r;
    }
}

// ---------------------------------------------------------- packed windows
// Large texts are packed to two bits per symbol first, so that a rank's window
// of kPackWin symbols is 8 bytes of a table a quarter (16-bit text: an eighth)
// the size: fewer lines, more of them in the caches. Two bits hold bases only: a
// window that meets anything else, or the end, is flagged, by one bit per
// 2^shift window starts (small enough for the L1 caches), and compares the text itself.
// Packed from 2^21 symbols on, and where sequences (as far as the caller knows)
// are at least kPackSeq long on average. Window and packing, bytes against
// packed: two sequences of 1M symbols 46 / 46 us in all of LCP, 4M 102 / 97, 8M
// 178 / 151, 16M 254 / 139 us, 1G 26.4 / 19.6 ms, 700 pairs with 102M symbols
// 1.27 / 0.85 ms; 65,536 queries of 634 bases, where one window in seven is
// flagged, 0.82 / 0.85 ms. With finer flags, 512 KB to 2 MB of them, that miss the L1
// caches: 16M 173 us, 1G 24.0 ms, as each is one more request to L2 or behind it.
constexpr uint32_t kPackFrom = 1u << 21, kPackSeq = 2048;
constexpr uint32_t kPackWin = 29;   // 32 symbols in 8 bytes less the up to 3 before the first
struct PackedText {
    uint32_t *words;    // symbol p: bits 2 (p % 16) of word p / 16
    uint32_t *flags;
    uint32_t shift;
};

// A base's two bits; 4 and more: no base.
__device__ __forceinline__ uint32_t pack_code(uint8_t c) { return c; }
__device__ __forceinline__ uint32_t pack_code(uint16_t c) { return (c & 7u) - 1u; }

template <typename CH>
__global__ __launch_bounds__(kBlock) void k_lcp_pack(const CH *__restrict__ t, uint32_t n, PackedText pt) {
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x, p = 16u * g;   // the last thread's group holds position n
    if (p > n) return;
    uint32_t v = 0, bad = 0;
    if (n - p >= 16u) {   // p is a multiple of 16, the text 4-byte aligned where this is used
        const uint32_t *w = reinterpret_cast<const uint32_t *>(t + p);
        constexpr uint32_t per = 4 / sizeof(CH);
        uint32_t x[16 / per];
#pragma unroll
        for (uint32_t c = 0; c < 16 / per; ++c) x[c] = w[c];
#pragma unroll
        for (uint32_t c = 0; c < 16; ++c) {
            const uint32_t y = pack_code((CH)(x[c / per] >> (8 * sizeof(CH) * (c % per))));
            v |= (y & 3u) << (2 * c);
            bad |= y >> 2;
        }
    } else {
        for (uint32_t c = 0; c < 16; ++c) {
            const uint32_t y = c < n - p ? pack_code(t[p + c]) : 4u;
            v |= (y & 3u) << (2 * c);
            bad |= y >> 2;
        }
    }
    pt.words[g] = v;
    if (bad) {   // the windows that meet this group start up to kPackWin - 1 before it
        const uint32_t last = min(p + 15u, n - 1u) >> pt.shift;
        for (uint32_t b = (p >= kPackWin ? p - kPackWin + 1u : 0u) >> pt.shift; b <= last; ++b)
            if (!((__hip_atomic_load(&pt.flags[b >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (b & 31u)) & 1u))
                atomicOr(&pt.flags[b >> 5], 1u << (b & 31u));
    }
}

// The kPackWin symbols from i on, and the flag in bit 63.
__device__ __forceinline__ uint64_t packed_window(const PackedText &pt, uint32_t i) {
    const uint64_t v = reinterpret_cast<const Chunk *>(reinterpret_cast<const uint8_t *>(pt.words) + (i >> 2))->w[0];
    const uint32_t b = i >> pt.shift;
    const uint64_t f = (pt.flags[b >> 5] >> (b & 31u)) & 1u;
    return ((v >> (2u * (i & 3u))) & ((1ull << (2u * kPackWin)) - 1ull)) | (f << 63);
}

// In the batched path's 16-bit text the ranks of a pair are its positions, so
// the text at the ranks tells neighbours of different pairs apart.
__device__ __forceinline__ bool same_text(const uint8_t *, uint32_t) { return true; }
__device__ __forceinline__ bool same_text(const uint16_t *t, uint32_t r) { return (t[r] ^ t[r - 1]) < 8u; }

template <typename CH, bool DIRECT>
__global__ __launch_bounds__(kBlock) void k_lcp_packed(const CH *__restrict__ t, uint32_t n, PackedText pt,
                                                       const int32_t *__restrict__ sa, int32_t *__restrict__ lcp,
                                                       uint32_t *__restrict__ phi, int32_t *__restrict__ isa,
                                                       uint32_t shift) {
    const uint32_t base = blockIdx.x * (kBlock * kLcpItems), lane = threadIdx.x & 63u;
    uint32_t p[kLcpItems], q[kLcpItems];
    uint64_t w[kLcpItems], e[kLcpItems];   // e: lane 0's predecessor
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        const uint32_t r = base + k * kBlock + threadIdx.x;
        p[k] = r < n ? min((uint32_t)sa[r], n - 1u) : 0u;
        q[k] = (lane == 0 && r > 0 && r < n) ? min((uint32_t)sa[r - 1], n - 1u) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) w[k] = packed_window(pt, p[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kLcpItems; ++k) e[k] = packed_window(pt, q[k]);
    }
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        const uint32_t r = base + k * kBlock + threadIdx.x;
        const uint32_t pj = (uint32_t)__shfl_up((int)p[k], 1, kWave);
        const uint64_t up = __shfl_up(w[k], 1, kWave);
        const uint32_t i = p[k], j = lane == 0 ? q[k] : pj;
        const uint64_t y = lane == 0 ? e[k] : up, x = (w[k] ^ y) & ~(1ull << 63);
        if (r >= n) continue;
        if (r == 0) {
            lcp[0] = 0;
        } else {
            uint32_t l = x ? (uint32_t)__builtin_ctzll(x) / 2u : kPackWin;
            bool open = x == 0;
            if ((w[k] | y) >> 63) {
                l = dev::extend<CH, 2>(t, n, i, j, 0u, kPackWin);
                open = l >= kPackWin && n - max(i, j) > kPackWin;
            }
            if (!same_text(t, r)) {
                l = 0;
                open = false;
            }
            lcp[r] = (int32_t)(open ? kPackWin | kMarked : l);
        }
        if ((i & ((1u << shift) - 1u)) == 0) phi[i >> shift] = r ? j : 0xffffffffu;
        if constexpr (DIRECT) isa[i] = (int32_t)r;
    }
}

constexpr uint32_t kNoCap = 0xffffffffu;

// PLCP of the unlinked sampled positions, and the links, 64 samples a word.
template <typename CH>
__global__ __launch_bounds__(kBlock) void k_plcp(const CH *__restrict__ t, uint32_t n,
                                                 const uint32_t *__restrict__ phi, uint32_t samples, uint32_t shift,
                                                 uint32_t *__restrict__ plcp, uint64_t *__restrict__ links) {
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x, step = 1u << shift;
    bool linked = false;
    if (s < samples) {
        const uint32_t i = s << shift, j = phi[s];
        const uint32_t next = s + 1 < samples ? phi[s + 1] : kNoCap;
        uint32_t l = 0;
        if (j < n && j != i) {
            l = dev::extend<CH, 4>(t, n, i, j, 0u, step);
            linked = l >= step && next < n && next == j + step;
            if (l >= step && !linked) l = dev::extend<CH, 4>(t, n, i, j, step, kNoCap);
        }
        if (!linked) plcp[s] = l;
    }
    const uint64_t m = __ballot(linked);
    if ((threadIdx.x & 63u) == 0 && s < samples) links[s >> 6] = m;
}

// ends[w] = the first unlinked sample from 64 w to the end of w's block of 64
// words (kNoCap: none there), blocks[c] = the first from block c on. A wave per
// block; one workgroup then completes `blocks` (the last sample is never
// linked, so the last block has one).
__global__ __launch_bounds__(kBlock) void k_plcp_links(const uint64_t *__restrict__ links, uint32_t words,
                                                       uint32_t samples, uint32_t *__restrict__ ends,
                                                       uint32_t *__restrict__ blocks) {
    const uint32_t w = blockIdx.x * kBlock + threadIdx.x, lane = threadIdx.x & 63u;
    uint32_t first = kNoCap;
    if (w < words) {
        const uint32_t left = samples - 64u * w;
        const uint64_t z = ~links[w] & (left >= 64u ? ~0ull : (1ull << left) - 1ull);
        if (z) first = 64u * w + (uint32_t)__builtin_ctzll(z);
    }
#pragma unroll
    for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
        const uint32_t x = (uint32_t)__shfl_down((int)first, o, kWave);
        if (lane + o < (uint32_t)kWave) first = min(first, x);
    }
    if (w < words) {
        ends[w] = first;
        if (lane == 0) blocks[w >> 6] = first;
    }
}

constexpr int kLinkThreads = 1024;
__global__ __launch_bounds__(kLinkThreads) void k_plcp_blocks(uint32_t *__restrict__ blocks, uint32_t count) {
    __shared__ uint32_t s_first[kLinkThreads];
    const uint32_t per = (count + kLinkThreads - 1u) / kLinkThreads;
    const uint32_t b = min(count, threadIdx.x * per), e = min(count, b + per);
    uint32_t first = kNoCap;
    for (uint32_t c = b; c < e; ++c) first = min(first, blocks[c]);
    s_first[threadIdx.x] = first;
    __syncthreads();
    for (uint32_t o = 1; o < (uint32_t)kLinkThreads; o <<= 1) {   // min over this thread's blocks and all later ones
        const uint32_t x = threadIdx.x + o < (uint32_t)kLinkThreads ? s_first[threadIdx.x + o] : kNoCap;
        __syncthreads();
        s_first[threadIdx.x] = min(s_first[threadIdx.x], x);
        __syncthreads();
    }
    uint32_t after = threadIdx.x + 1 < (uint32_t)kLinkThreads ? s_first[threadIdx.x + 1] : kNoCap;
    for (uint32_t c = e; c-- > b;) {
        after = min(after, blocks[c]);
        blocks[c] = after;
    }
}

template <typename CH>
__global__ __launch_bounds__(kBlock) void k_lcp_finish(const CH *__restrict__ t, uint32_t n,
                                                       const int32_t *__restrict__ sa,
                                                       const uint32_t *__restrict__ phi,
                                                       const uint32_t *__restrict__ plcp,
                                                       const uint64_t *__restrict__ links,
                                                       const uint32_t *__restrict__ ends,
                                                       const uint32_t *__restrict__ blocks, uint32_t samples,
                                                       uint32_t shift, int32_t *__restrict__ lcp) {
    const uint32_t base = blockIdx.x * (kBlock * kLcpItems);
    uint32_t v[kLcpItems];
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        const uint32_t r = base + k * kBlock + threadIdx.x;
        v[k] = r < n ? (uint32_t)lcp[r] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kLcpItems; ++k) {
        if (!(v[k] & kMarked)) continue;      // ranks above 0 only
        const uint32_t r = base + k * kBlock + threadIdx.x;
        const uint32_t i = min((uint32_t)sa[r], n - 1u), j = min((uint32_t)sa[r - 1], n - 1u);
        const uint32_t c = i >> shift, d = i & ((1u << shift) - 1u);
        auto sampled = [&](uint32_t q) -> uint32_t {   // PLCP at sample q, through its chain
            const uint64_t z = ~links[q >> 6] >> (q & 63u);
            uint32_t end = q + (uint32_t)__builtin_ctzll(z | (1ull << 63));
            if (!z) {   // then word w + 1 exists: the last sample is not linked
                const uint32_t w = (q >> 6) + 1u;
                end = ends[w];
                if (end == kNoCap) end = blocks[(w >> 6) + 1u];
            }
            end = min(end, samples - 1u);
            return plcp[end] + ((end - q) << shift);
        };
        const uint32_t got = sampled(c), to_next = (1u << shift) - d;
        uint32_t h;
        if (got > d && phi[c] == j - d) {
            h = got - d;                     // same diagonal as the sample before: exact
        } else {
            h = min(max(v[k] & ~kMarked, got > d ? got - d : 0u), n - max(i, j));
            if (h < to_next) h = dev::extend<CH, 4>(t, n, i, j, h, to_next);
            if (h >= to_next) {
                if (c + 1 < samples && phi[c + 1] == j + to_next) h = to_next + sampled(c + 1);   // as the one behind
                else h = dev::extend<CH, 4>(t, n, i, j, h, kNoCap);
            }
        }
        lcp[r] = (int32_t)h;
    }
}

}  // namespace

size_t lcp_workspace(uint64_t n) { return (size_t)n * 28 + radix_counts_words(n) * 4 + 4096; }

template <typename CH>
lor_status lcp_build_t(const CH *text, uint32_t n, const int32_t *sa, int32_t *lcp, int32_t *isa, Arena &ar,
                       hipStream_t s, uint32_t seqs) {
    if (n == 0) return LOR_OK;
    // every 2^shift-th position is sampled: half the plan's steps, 8 to 512
    const uint32_t shift = (uint32_t)bits_for((uint64_t)plan().plcp_steps) - 2u;
    const uint32_t samples = div_up(n, 1u << shift), words = div_up(samples, 64);
    const uint32_t grid = div_up(n, kBlock * kLcpItems);
    uint32_t *phi, *plcp, *ends, *blocks;
    uint64_t *links;
    LOR_TAKE(ar, uint32_t, samples, phi);
    LOR_TAKE(ar, uint32_t, samples, plcp);
    LOR_TAKE(ar, uint64_t, words, links);
    LOR_TAKE(ar, uint32_t, (size_t)words + 1, ends);
    const uint32_t nblocks = div_up(words, 64);
    LOR_TAKE(ar, uint32_t, (size_t)nblocks + 1, blocks);
    const bool direct = isa && n <= kDirectIsa;
    const double bytes = (double)n * (8 + sizeof(CH) + (direct ? 4 : 0));
    const size_t before_pack = ar.mark();
    if (n >= kPackFrom && n / kPackSeq >= seqs && reinterpret_cast<uintptr_t>(text) % 4 == 0) {
        PackedText pt;
        // flags of about 16 KB, which stay in the L1 caches, while the starts that
        // share one with a separator stay below one in 1,024 (one in 128: 700 pairs
        // 811 -> 846 us)
        pt.shift = std::max(bits_for(n) - 17, 4);
        while (pt.shift > 4 && ((uint64_t)std::max(seqs, 32u) << pt.shift) > n / 1024) --pt.shift;
        const uint32_t fwords = div_up(div_up(n, 1u << pt.shift), 32);
        LOR_TAKE(ar, uint32_t, (size_t)n / 16 + 4, pt.words);   // the last window reads up to 8 bytes from n / 4 on
        LOR_TAKE(ar, uint32_t, fwords, pt.flags);
        LOR_TRY(zero_words(pt.flags, fwords, s));
        LOR_LAUNCH("k_lcp_pack", (double)n * (sizeof(CH) + 0.25), s,
                   hipLaunchKernelGGL(k_lcp_pack<CH>, dim3(div_up(n / 16 + 1, kBlock)), dim3(kBlock), 0, s, text, n,
                                      pt));
        auto *kernel = direct ? k_lcp_packed<CH, true> : k_lcp_packed<CH, false>;
        LOR_LAUNCH("k_lcp_packed", bytes, s,
                   hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, s, text, n, pt, sa, lcp, phi, isa, shift));
        ar.release(before_pack);
    } else if (direct)
        LOR_LAUNCH("k_lcp_window", bytes, s,
                   hipLaunchKernelGGL((k_lcp_window<CH, true>), dim3(grid), dim3(kBlock), 0, s, text, n, sa, lcp, phi,
                                      isa, shift));
    else
        LOR_LAUNCH("k_lcp_window", bytes, s,
                   hipLaunchKernelGGL((k_lcp_window<CH, false>), dim3(grid), dim3(kBlock), 0, s, text, n, sa, lcp,
                                      phi, isa, shift));
    LOR_LAUNCH("k_plcp", 8.0 * samples, s,
               hipLaunchKernelGGL(k_plcp<CH>, dim3(div_up(samples, kBlock)), dim3(kBlock), 0, s, text, n, phi,
                                  samples, shift, plcp, links));
    LOR_LAUNCH("k_plcp_links", 12.0 * words, s,
               hipLaunchKernelGGL(k_plcp_links, dim3(div_up(words, kBlock)), dim3(kBlock), 0, s, links, words, samples,
                                  ends, blocks));
    if (nblocks > 1)
        LOR_LAUNCH("k_plcp_blocks", 8.0 * nblocks, s,
                   hipLaunchKernelGGL(k_plcp_blocks, dim3(1), dim3(kLinkThreads), 0, s, blocks, nblocks));
    LOR_LAUNCH("k_lcp_finish", 4.0 * n, s,
               hipLaunchKernelGGL(k_lcp_finish<CH>, dim3(grid), dim3(kBlock), 0, s, text, n, sa, phi, plcp, links, ends,
                                  blocks, samples, shift, lcp));
    if (!isa || direct) return LOR_OK;
    uint32_t *tmp[4], *counts;
    for (int i = 0; i < 4; ++i) LOR_TAKE(ar, uint32_t, n, tmp[i]);
    LOR_TAKE(ar, uint32_t, radix_counts_words(n), counts);
    return bucketed_scatter(isa, n, reinterpret_cast<const uint32_t *>(sa), nullptr, 0, n, tmp, counts, s, true);
}

lor_status lcp_build(const uint8_t *text, uint32_t n, const int32_t *sa, int32_t *lcp, int32_t *isa, Arena &ar,
                     hipStream_t s, uint32_t seqs) {
    return lcp_build_t<uint8_t>(text, n, sa, lcp, isa, ar, s, seqs);
}

lor_status lcp_build_u16(const uint16_t *text, uint32_t n, const int32_t *sa, int32_t *lcp, int32_t *isa, Arena &ar,
                         hipStream_t s, uint32_t seqs) {
    return lcp_build_t<uint16_t>(text, n, sa, lcp, isa, ar, s, seqs);
}

}  // namespace lor
