// Ranked-merge BPE by compatible neighbours: every lane of the chip segments
// its own short chunk of a row, and neighbouring chunks are stitched.
//
// The rule that two tokens may be neighbours, the test for it by undoing their
// merges, and the search over such tokens from the longest down are published:
// van Antwerpen and Neubeck, "So many tokens, so little time: Introducing a
// faster, more flexible byte-pair tokenizer" (GitHub, 2024), and their
// open-source bpe crate. The lanes, the stitch, the joins between waves and the
// walk over repeats are this library's.
//
// Why that is exact. Call two tokens compatible when the merges, applied to
// their concatenated bases, leave exactly those two tokens. A sequence of
// tokens is the segmentation of its text if and only if every adjacent pair
// is compatible:
//  * If all adjacent pairs are compatible, take the first merge over the
//    whole text that would cross a token boundary. Until then every merge
//    stayed inside one token, so the merges inside the two tokens at that
//    boundary came in the order (rank, then leftmost) in which they come when
//    the two are alone, and the crossing merge would come there too: the pair
//    would not be compatible.
//  * In the segmentation of a text no merge crosses a final boundary, so by
//    the same argument each adjacent pair, taken alone, ends as it is.
// Two consequences. A chunk can be segmented by search: walk left to right,
// take a token that is compatible with the one before it, go back when none
// is. (A prefix of the walk is the segmentation of the bases it covers, so a
// position is reached with one predecessor only and a position found to lead
// nowhere never has to be tried again.) And two sequences of compatible
// tokens over overlapping texts that share one token can be joined there:
// left of it the first one, right of it the second; every adjacent pair
// occurs in one of the two. So a lane may stop as soon as its tokens meet
// those that the next lane holds, provided that lane does not give them up
// again: a wave ends when all of its lanes have met or ended at the same
// time. The waves' own sequences are joined at the token across each wave's
// last chunk end. Both waves segment that chunk, the first one's last own lane
// against a lane that ends at its own last base, the second one's first lane
// against one that reads on, so the two may differ: the join stands if both
// hold the same token there and the second wave's first lane has met its
// second one, whose tokens are the ones kept (k_bpe_walk checks it). The
// segmentations of a text from two starting points share a token after a few
// (9 bases in the median, 28 at most over 6,249 cuts of the 4,096-merge
// table's corpus), so a lane reads 64 bases of its own and as many of the
// next chunk's as it takes to meet that lane's segmentation.
//
// N and invalid bytes are barriers: tokens of one base that are compatible
// with everything.
//
// Pipeline (all on the caller's stream):
//  1. k_rowscan_units or k_rowscan (encode.hip, by the number of rows): chunk
//     offsets of the rows, 64 bases per chunk.
//  2. k_bpe_chunks: one lane per chunk; start bits and ids of the tokens.
//  3. k_bpe_walk: chunks that did not meet their neighbour within 127 bases
//     (short tandem repeats), or whose wave ended on other tokens than the
//     next wave holds: one wave per row carries the search on until it meets
//     a later chunk's tokens, a repeat's tokens at once.
//  4. k_bpe_count: exclusive scan of the chunks' token counts.
//  5. k_bpe_put: ids, offsets, specials, pads and mask.
#include <algorithm>
#include <array>
#include <type_traits>
#include <vector>

#include "bpe_pairs.hpp"
#include "common.hpp"
#include "device.hpp"

namespace dnatok {

namespace {

constexpr int kChunk = 64;             // bases a lane owns: the low word of its start mask
constexpr uint32_t kReach = 127;       // bases a lane may read: the bits of the mask
constexpr int kLead = 1;               // lanes of a wave that repeat the chunk before its own
constexpr int kOwn = 64 - kLead - 1;   // chunks a wave owns; its last lane repeats the chunk after them
constexpr int kMaxTokenBases = 64;     // longer tokens: the item path
constexpr int kMaxWavesPerGroup = 8;
constexpr int kMinWavesPerGroup = 2;
constexpr uint32_t kStepCap = 1u << 20;  // never reached: a lane tries at most 64 tokens at each of 127 bases
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));  // (rows start at any byte)
constexpr uint32_t kFailed = 0x80000000u, kTaken = 0x40000000u, kRowBits = 0x3FFFFFFFu;
constexpr size_t kLdsRoom = 160 * 1024;
constexpr int kPutNT = 256;
constexpr int kCountPerThread = 4;
constexpr int64_t kCountUnit = (int64_t)kPutNT * kCountPerThread;

// A token's entry: the three next shorter tokens that begin it (0: none), and
// the bases less one of the token and of the first two.
__host__ __device__ inline uint2 info_entry(uint32_t c1, uint32_t c2, uint32_t c3, uint32_t l0, uint32_t l1,
                                            uint32_t l2) {
    return uint2{c1 | (c2 << 14), c3 | ((l0 - 1) << 14) | ((l1 ? l1 - 1 : 0u) << 20) | ((l2 ? l2 - 1 : 0u) << 26)};
}
__host__ __device__ inline uint32_t info_link(uint2 x) { return x.x & 0x3FFFu; }
__host__ __device__ inline uint32_t info_len(uint2 x) { return ((x.y >> 14) & 63u) + 1u; }

// Whether tokens (x, y) may be neighbours (the published test, see above): undo
// the merges of the two, the later one first (equal ranks: leftmost merged
// first, so the right one is undone first). While a boundary pair stands, it
// must not rank before the merge that ended it.
template <class Rank, class Pair>
__host__ __device__ inline bool boundary_holds(uint32_t x, uint32_t y, uint32_t limit, Rank rank, Pair pair) {
    for (;;) {
        if (rank(x, y) < limit) return false;
        const int32_t rx = x >= 10 ? (int32_t)x - 10 : -1, ry = y >= 10 ? (int32_t)y - 10 : -1;
        if (rx < 0 && ry < 0) return true;
        if (rx > ry) {
            limit = (uint32_t)rx;
            x = pair((uint32_t)rx) >> 16;
        } else {
            limit = (uint32_t)ry + 1u;
            y = pair((uint32_t)ry) & 0xFFFFu;
        }
    }
}

// compat[a * rw + b / 32] bit b % 32: token b may follow token a (b = 0, no
// token: never).
__global__ __launch_bounds__(256) void k_bpe_compat(const uint4 *bucket, const uint32_t *pair, uint32_t nbk,
                                                    uint32_t V, uint32_t rw, uint32_t *compat) {
    const RankTab tab{bucket, pair, nbk};
    const uint64_t n = (uint64_t)V * rw;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
        const uint32_t a = (uint32_t)(i / rw), b0 = (uint32_t)(i % rw) * 32;
        uint32_t w = 0;
        for (uint32_t u = 0; u < 32 && b0 + u < V; ++u)
            w |= (uint32_t)(b0 + u != 0 && boundary_holds(
                                               a, b0 + u, (uint32_t)kNoRank,
                                               [&](uint32_t x, uint32_t y) { return pair_rank(tab, x, y); },
                                               [&](uint32_t r) { return pair[r]; }))
                 << u;
        compat[i] = w;
    }
}

}  // namespace

// Tables of the chunk path: each token's shorter tokens and length; the
// compatible pairs; the automaton that, read from right to left, knows the
// longest token starting at each base (the trie of the reversed tokens,
// completed so that every state has a successor for every base); and the
// trie of the tokens for the walk. Tokens that their own bases do not give
// back (another rank comes first inside them) never occur in a segmentation
// and stay out of all of them. Leaves t.chunked false where a token is too
// long or the automaton's states pass its 16-bit entries.
int build_bpe_chunk_tables(dnatok_vocab *v) {
    BpeTables &t = v->bpe;
    const uint32_t R = (uint32_t)t.n_merges, V = 10 + R;
    const int32_t *m = v->h_merges.data();
    if (v->max_token_bytes > kMaxTokenBases) return DNATOK_OK;
    std::vector<std::pair<uint32_t, uint32_t>> ranks(R);  // (pair, rank), by pair
    auto pair = [&](uint32_t r) { return (uint32_t)m[2 * r] | ((uint32_t)m[2 * r + 1] << 16); };
    for (uint32_t r = 0; r < R; ++r) ranks[r] = {pair(r), r};
    std::sort(ranks.begin(), ranks.end());
    auto rank = [&](uint32_t a, uint32_t b) {
        const uint32_t key = a | (b << 16);
        auto it = std::lower_bound(ranks.begin(), ranks.end(), std::make_pair(key, 0u));
        return it == ranks.end() || it->first != key ? (uint32_t)kNoRank : it->second;
    };
    std::vector<uint8_t> valid(V, 0), text((size_t)V * kMaxTokenBases), len(V, 0);
    auto base = [&](uint32_t id, uint32_t j) -> uint8_t & { return text[(size_t)id * kMaxTokenBases + j]; };
    for (uint32_t b = 0; b < 4; ++b) {
        valid[5 + b] = len[5 + b] = 1;
        base(5 + b, 0) = (uint8_t)b;
    }
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t a = (uint32_t)m[2 * r], b = (uint32_t)m[2 * r + 1], id = 10 + r;
        valid[id] = valid[a] && valid[b] && boundary_holds(a, b, r, rank, pair);
        len[id] = (uint8_t)(len[a] + len[b]);
        std::copy(&base(a, 0), &base(a, 0) + len[a], &base(id, 0));
        std::copy(&base(b, 0), &base(b, 0) + len[b], &base(id, 0) + len[a]);
    }
    struct Node {
        std::array<uint32_t, 4> kid{{0, 0, 0, 0}};
        uint32_t tok = 0;
    };
    auto trie_of = [&](bool reversed) {
        std::vector<Node> trie(1);
        for (uint32_t id = 5; id < V; ++id) {
            if (!valid[id]) continue;
            uint32_t at = 0;
            for (uint32_t j = 0; j < len[id]; ++j) {
                const uint8_t c = base(id, reversed ? len[id] - 1 - j : j);
                if (!trie[at].kid[c]) {
                    trie[at].kid[c] = (uint32_t)trie.size();
                    trie.emplace_back();
                }
                at = trie[at].kid[c];
            }
            trie[at].tok = id;
        }
        return trie;
    };
    const std::vector<Node> fwd = trie_of(false);
    std::vector<Node> rev = trie_of(true);
    if (rev.size() > 0x4000 || fwd.size() > 0xFFFF) return DNATOK_OK;
    std::vector<uint2> info(V, uint2{0, 0});
    info[DNATOK_ID_UNK] = info[9] = info_entry(0, 0, 0, 1, 0, 0);  // barriers
    std::vector<uint32_t> link(V, 0);
    for (uint32_t id = 5; id < V; ++id) {
        uint32_t at = 0;
        for (uint32_t j = 0; valid[id] && j + 1 < len[id]; ++j) {
            at = fwd[at].kid[base(id, j)];
            if (fwd[at].tok) link[id] = fwd[at].tok;
        }
    }
    for (uint32_t id = 5; id < V; ++id) {
        if (!valid[id]) continue;
        const uint32_t c1 = link[id], c2 = link[c1], c3 = link[c2];
        info[id] = info_entry(c1, c2, c3, len[id], len[c1], len[c2]);
    }
    std::vector<uint32_t> kid(4 * fwd.size(), 0);
    for (size_t i = 0; i < fwd.size(); ++i)
        for (int c = 0; c < 4; ++c)
            if (fwd[i].kid[c]) kid[4 * i + c] = fwd[fwd[i].kid[c]].tok | (fwd[i].kid[c] << 16);
    // states breadth first: a state's suffix state is complete before it
    const uint32_t n_states = (uint32_t)rev.size();
    std::vector<uint16_t> next(4 * (size_t)n_states, 0), longest(n_states, 0);
    std::vector<uint32_t> order{0}, suffix(n_states, 0);
    for (size_t i = 0; i < order.size(); ++i) {
        const uint32_t at = order[i];
        longest[at] = (uint16_t)(rev[at].tok ? rev[at].tok : longest[suffix[at]]);
        for (int c = 0; c < 4; ++c) {
            const uint32_t k = rev[at].kid[c], by_suffix = at ? next[4 * (size_t)suffix[at] + c] / 4u : 0u;
            if (k) {
                suffix[k] = by_suffix;
                order.push_back(k);
            }
            next[4 * (size_t)at + c] = (uint16_t)(4 * (k ? k : by_suffix));
        }
    }
    t.rw = (V + 31) / 32;
    t.n_states = n_states;
    // one allocation: automaton, info, trie, pairs (each in whole 16-byte
    // units, the first three for the copy to LDS)
    const void *host[4] = {next.data(), longest.data(), info.data(), kid.data()};
    const size_t size[4] = {next.size() * 2, longest.size() * 2, info.size() * sizeof(uint2), kid.size() * 4};
    size_t at[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < 4; ++i) at[i + 1] = at[i] + (size[i] + 15) / 16 * 16;
    std::vector<uint8_t> all(at[4], 0);
    for (int i = 0; i < 4; ++i) std::copy_n(static_cast<const uint8_t *>(host[i]), size[i], all.begin() + at[i]);
    void *p = nullptr;
    DNATOK_HIP(dev_alloc(&p, at[4] + (size_t)V * t.rw * 4));
    t.d_chunk = static_cast<uint8_t *>(p);
    DNATOK_HIP(hipMemcpy(p, all.data(), at[4], hipMemcpyHostToDevice));
    t.d_longest = reinterpret_cast<const uint16_t *>(t.d_chunk + at[1]);
    t.d_info = reinterpret_cast<const uint2 *>(t.d_chunk + at[2]);
    t.d_kid = reinterpret_cast<const uint32_t *>(t.d_chunk + at[3]);
    t.d_compat = reinterpret_cast<uint32_t *>(t.d_chunk + at[4]);
    const uint64_t words = (uint64_t)V * t.rw;
    hipLaunchKernelGGL(k_bpe_compat, dim3((unsigned)std::min<uint64_t>((words + 255) / 256, 1u << 16)), dim3(256), 0,
                       nullptr, reinterpret_cast<const uint4 *>(t.d_bucket), t.d_pair, t.nbk, V, t.rw, t.d_compat);
    DNATOK_HIP(hipGetLastError());
    t.chunked = true;
    return DNATOK_OK;
}

namespace {

struct ChunkArgs {
    const uint8_t *bytes;
    int64_t nbytes;
    const int64_t *offs;
    int32_t n;
    const int64_t *chunk_off;  // [n + 1] first chunk of each row (every row has one)
    int64_t max_chunks;
    uint64_t *mask;  // [max_chunks] bit x: a token starts at base x of the chunk
    uint64_t *dead;  // [max_chunks] walk: positions that lead nowhere
    uint32_t *row;   // [max_chunks] row of the chunk, kFailed: did not meet the next chunk; kTaken, on a
                     // row's first: a workgroup of the walk has the row
    uint32_t *list;  // [max_chunks] chunks with kFailed, in no order
    uint32_t *edge;  // [tasks][2] token across the start and across the end of a wave's own chunks
    uint64_t *pos;   // [max_chunks + 1] tokens before the chunk (walk: the start bits it replaces)
    uint16_t *sym;   // [nbytes] id of the token that starts at a byte
    uint32_t *count; // entries of list, zero between launches
    const uint16_t *next, *longest;
    const uint2 *info;
    const uint32_t *kid, *compat;
    uint32_t V, rw, n_states;
    uint32_t warm;  // bases of the longest token, less one
};

// Digit of a base (A0 C1 G2 T3), 4: N, 5: any other byte.
__device__ __forceinline__ uint32_t base_class(uint32_t b) {
    const uint32_t f = b | 0x20u, d = ((f >> 1) ^ (f >> 2)) & 3u;
    return f == ((0x74676361u >> (8 * d)) & 0xFFu) ? d : f == 'n' ? 4u : 5u;
}

// 128-bit start mask.
struct Bits {
    uint64_t lo, hi;
};
__device__ __forceinline__ Bits bit_only(uint32_t i) {
    const uint64_t b = 1ull << (i & 63u);
    return i < 64 ? Bits{b, 0ull} : Bits{0ull, b};
}
__device__ __forceinline__ uint32_t highest(Bits b) {
    return b.hi ? 127u - (uint32_t)__builtin_clzll(b.hi) : 63u - (uint32_t)__builtin_clzll(b.lo);
}

constexpr int kDppWaveShl1 = 0x130;
__device__ __forceinline__ uint64_t from_next(uint64_t v) {
    return (uint64_t)dev::dpp_u32<kDppWaveShl1>(0, (uint32_t)v) |
           ((uint64_t)dev::dpp_u32<kDppWaveShl1>(0, (uint32_t)(v >> 32)) << 32);
}
__device__ __forceinline__ uint32_t from_prev(uint32_t v) { return dev::wave_from_prev_u32(v, 0u); }
__device__ __forceinline__ uint64_t from_prev(uint64_t v) {
    return (uint64_t)from_prev((uint32_t)v) | ((uint64_t)from_prev((uint32_t)(v >> 32)) << 32);
}

// LDS: info, then (FAST) the automaton, then each wave's longest tokens:
// entry x * 64 + lane is base x of the lane's chunk, so a wave's lanes write
// neighbouring entries.
__host__ __device__ constexpr uint32_t lds_info(uint32_t V) { return (8u * V + 15u) / 16u * 16u; }
__host__ __device__ constexpr uint32_t lds_next(uint32_t n_states) { return (8u * n_states + 15u) / 16u * 16u; }
__host__ __device__ constexpr uint32_t lds_longest(uint32_t n_states) { return (2u * n_states + 15u) / 16u * 16u; }
constexpr uint32_t kLdsPerWave = 2u * 64u * 64u;

// Copies whole 16-byte units, eight loads in flight per thread.
__device__ __forceinline__ void copy_to_lds(uint8_t *dst, const void *src, uint32_t bytes) {
    const uint4 *g = static_cast<const uint4 *>(src);
    uint4 *d = reinterpret_cast<uint4 *>(dst);
    const uint32_t n = bytes / 16, step = blockDim.x;
    for (uint32_t j0 = threadIdx.x; j0 < n; j0 += 8 * step) {
        uint4 v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = g[min(j0 + u * step, n - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            if (j0 + u * step < n) d[j0 + u * step] = v[u];
    }
}

// One lane per chunk: the longest token at every base, then the search, then
// the stitch. Bound by VALU issue and by the latency of the search's reads
// (an LDS read of the candidates, an L2 read of their pair bits) times the
// steps of a wave's slowest lane, not by bytes: 5.5 MB in and 1 M ids for the
// 1,024-row batch. FAST: the automaton lies in LDS and no token is longer
// than 32 bases; else it is read from L2, and tokens have up to 64.
template <bool FAST>
__global__ __launch_bounds__(64 * kMaxWavesPerGroup) void k_bpe_chunks(ChunkArgs a) {
    extern __shared__ __align__(16) uint8_t dyn[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint32_t at_next = lds_info(a.V), at_longest = at_next + (FAST ? lds_next(a.n_states) : 0u);
    const uint2 *s_info = reinterpret_cast<const uint2 *>(dyn);
    const uint16_t *s_next = reinterpret_cast<const uint16_t *>(dyn + at_next);
    const uint16_t *s_longest = reinterpret_cast<const uint16_t *>(dyn + at_longest);
    uint8_t *own_lds = dyn + at_longest + (FAST ? lds_longest(a.n_states) : 0u) + (size_t)wave * kLdsPerWave;
    uint16_t *best = reinterpret_cast<uint16_t *>(own_lds);
    const int64_t total = min(a.chunk_off[a.n], a.max_chunks);
    const int64_t tasks = (total + kOwn - 1) / kOwn;
    if ((int64_t)blockIdx.x >= tasks) return;  // the whole workgroup
    copy_to_lds(dyn, a.info, lds_info(a.V));
    if constexpr (FAST) {
        copy_to_lds(dyn + at_next, a.next, lds_next(a.n_states));
        copy_to_lds(dyn + at_longest, a.longest, lds_longest(a.n_states));
    }
    __syncthreads();

    for (int64_t task = blockIdx.x + (int64_t)gridDim.x * wave; task < tasks; task += (int64_t)gridDim.x * waves) {
        const int64_t first = task * kOwn - kLead;  // chunk of lane 0
        const int64_t c = first + lane;
        // rows: the first one by search, the others from the chunks at which they start
        const int64_t c_lo = first < 0 ? 0 : first;
        const int64_t r0 =
            dev::wave_lower_bound(0, (int64_t)a.n + 1, [&](int64_t i) { return a.chunk_off[i] > c_lo; }) - 1;
        const int64_t rk = min(r0 + 1 + lane, (int64_t)a.n);
        const int64_t at = a.chunk_off[rk] - first;
        const uint64_t sw = (rk < a.n && at >= 0 && at < 64) ? 1ull << at : 0ull;
        const uint64_t starts = ((uint64_t)dev::wave_or_all_u32((uint32_t)(sw >> 32)) << 32) |
                                dev::wave_or_all_u32((uint32_t)sw);
        const uint64_t upto = starts & (lane == 63 ? ~0ull : (2ull << lane) - 1);
        const int64_t r = min(r0 + __popcll(upto), (int64_t)a.n - 1);
        const bool valid = c >= 0 && c < total;
        const int64_t j = upto ? lane - (63 - __clzll(upto)) : c - a.chunk_off[r0];
        int64_t o0 = a.offs[r], o1 = a.offs[r + 1];
        o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
        o1 = o1 < o0 ? o0 : (o1 > a.nbytes ? a.nbytes : o1);
        const int64_t s = o0 + kChunk * j;
        const int64_t left = valid && s < o1 ? o1 - s : 0;
        // text of the wave, from its first chunk on
        const int lead = first < 0 ? (int)-first : 0;
        const int64_t base = (int64_t)__shfl((long long)s, lead, 64);
        const bool in_text = valid && s >= base && s - base <= 63 * kChunk;  // fails for malformed offsets only
        // the last lane reads its own bases only: what follows is the next wave's
        const uint32_t end = in_text ? (uint32_t)min(left, (int64_t)(lane == 63 ? kChunk : kReach)) : 0u;

        // this lane's text: 64 bases and as many of the next as a token may
        // reach over, read in whole dwords (none past the one with the last
        // byte) and shifted into place; what lies past the row is a barrier
        constexpr int kGroups = FAST ? 6 : 8;  // of 16 bases
        uint32_t code[kGroups], base_bits[kGroups];  // digits (first base on top), and which are bases
        {
            const uintptr_t at = reinterpret_cast<uintptr_t>(a.bytes) + (uint64_t)(end ? s : 0);
            const uint32_t *src = reinterpret_cast<const uint32_t *>(at & ~(uintptr_t)3);
            const uint32_t sh = (uint32_t)at & 3u;
            const int64_t last = (int64_t)((reinterpret_cast<uintptr_t>(a.bytes) + (uint64_t)a.nbytes - 1) >> 2) -
                                 (int64_t)(at >> 2);  // dword of the last byte
            uint32_t w[4 * kGroups + 4];
            if (__ballot(end && last < 4 * kGroups + 3) == 0) {
#pragma unroll
                for (int i = 0; i <= kGroups; ++i) {
                    const u32x4 v = end ? *reinterpret_cast<const u32x4 *>(src + 4 * i) : u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[4 * i + q] = v[q];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4 * kGroups + 4; ++i) w[i] = end ? src[min((int64_t)i, last)] : 0u;
            }
#pragma unroll
            for (int i = 0; i < kGroups; ++i) {
                uint4 v;
                v.x = __builtin_amdgcn_alignbyte(w[4 * i + 1], w[4 * i], sh);
                v.y = __builtin_amdgcn_alignbyte(w[4 * i + 2], w[4 * i + 1], sh);
                v.z = __builtin_amdgcn_alignbyte(w[4 * i + 3], w[4 * i + 2], sh);
                v.w = __builtin_amdgcn_alignbyte(w[4 * i + 4], w[4 * i + 3], sh);
                dev::classify16(v, code[i], base_bits[i]);
                const uint32_t in_row = (uint32_t)min(max(left - 16 * i, (int64_t)0), (int64_t)16);
                base_bits[i] &= ~(0xFFFFFFFFu >> in_row);
            }
        }
        // the longest token at each base, right to left: one table step a base
        // (a trie walk from each base took eight). FAST: the two halves of
        // the chunk side by side, each after the bases that a token may reach
        // over, so two chains of reads are under way.
        {
            auto wide = [](uint32_t x, uint32_t y) { return ((uint64_t)x << 32) | y; };
            auto bits32 = [&](int g) { return (base_bits[g] & 0xFFFF0000u) | (base_bits[g + 1] >> 16); };
            auto step = [&](uint32_t st, uint32_t digit) -> uint32_t {
                return FAST ? s_next[st + digit] : a.next[st + digit];
            };
            auto put = [&](int x, uint32_t st) { best[x * 64 + lane] = FAST ? s_longest[st >> 2] : a.longest[st >> 2]; };
            if constexpr (FAST) {
                uint32_t st0 = 0, st1 = 0;
                const uint64_t c0 = wide(code[2], code[3]), c1 = wide(code[4], code[5]);
                const uint32_t b0 = bits32(2), b1 = bits32(4);
                for (int x = (int)a.warm - 1; x >= 0; --x) {
                    st0 = step(st0, (uint32_t)(c0 >> (62 - 2 * x)) & 3u);
                    st1 = step(st1, (uint32_t)(c1 >> (62 - 2 * x)) & 3u);
                    st0 = (b0 >> (31 - x)) & 1u ? st0 : 0u;
                    st1 = (b1 >> (31 - x)) & 1u ? st1 : 0u;
                }
#pragma unroll
                for (int x = 31; x >= 0; --x) {
                    const int g = x >> 4, at = 15 - (x & 15);
                    st0 = step(st0, (code[g] >> (2 * at)) & 3u);
                    st1 = step(st1, (code[g + 2] >> (2 * at)) & 3u);
                    st0 = (base_bits[g] >> (16 + at)) & 1u ? st0 : 0u;
                    st1 = (base_bits[g + 2] >> (16 + at)) & 1u ? st1 : 0u;
                    put(x, st0);
                    put(32 + x, st1);
                }
            } else {
                uint32_t st = 0;
                const uint64_t c0 = wide(code[4], code[5]), c1 = wide(code[6], code[7]);
                const uint32_t b0 = bits32(4), b1 = bits32(6);
                for (int x = (int)a.warm - 1; x >= 0; --x) {
                    const int y = x & 31;
                    st = step(st, (uint32_t)((x < 32 ? c0 : c1) >> (62 - 2 * y)) & 3u);
                    st = ((x < 32 ? b0 : b1) >> (31 - y)) & 1u ? st : 0u;
                }
#pragma unroll
                for (int x = 63; x >= 0; --x) {
                    const int g = x >> 4, at = 15 - (x & 15);
                    st = step(st, (code[g] >> (2 * at)) & 3u);
                    st = (base_bits[g] >> (16 + at)) & 1u ? st : 0u;
                    put(x, st);
                }
            }
            // barriers in the row
            uint64_t bar = ~(wide(bits32(0), bits32(2)));
            if (left < 64) bar &= left > 0 ? ~0ull << (uint32_t)(64 - left) : 0ull;
            for (; bar; bar &= ~(1ull << (63 - __builtin_clzll(bar)))) {
                const int x = __builtin_clzll(bar);
                best[x * 64 + lane] =
                    (uint16_t)((a.bytes[s + x] | 0x20u) == 'n' ? 9u : (uint32_t)DNATOK_ID_UNK);
            }
        }
        wave_sync();
        auto best_at = [&](uint32_t x) -> uint32_t { return best[(x & 63u) * 64 + lane + (x >> 6)]; };

        // the search: frontier p, the token before it, the next one to try
        // (three at a time: it and the next shorter two). The last four
        // tokens before `prev` sit in `stack`; deeper ones are found again
        // from the text and the start bits.
        const bool next_same = lane < 63 && valid && c + 1 < total && !((starts >> (lane + 1)) & 1u);
        const bool prev_same = lane > 0 && valid && j > 0;
        uint32_t p = 0, prev = 0, cand = best[lane];
        uint64_t stack = 0;
        Bits own{1, 0};
        // positions a token may end at: up to `end`, less those that lead nowhere
        Bits open{~0ull, ~0ull};
        if (end < 64) open = Bits{(2ull << end) - 1, 0};
        else if (end < 127) open.hi = (2ull << (end - 64)) - 1;
        bool need = false;
        uint32_t meet = 0;  // where this lane's tokens met the next lane's, from that lane's start
        for (uint32_t step = 0; step < kStepCap; ++step) {
            if ((step & 3u) == 0) {
                const uint64_t next = from_next(own.lo);
                // ends of tokens that both have: a common start, nothing of
                // either up to the next start, and that one common too (the
                // add carries each common start up to the next start)
                const uint64_t both = own.hi & next, any = own.hi | next;
                const uint64_t hit = next_same ? ((both << 1) + ~any) & both : 0ull;
                meet = hit ? (uint32_t)__builtin_ctzll(hit) : 0u;
                // tokens up to the row's end need no other lane's: met there
                if (next_same && p == end && left == (int64_t)end) meet = end - kChunk;
                need = valid && p != end && (lane == 63 ? prev_same : meet == 0);
                if (!__ballot(need)) break;
            }
            if (need) {
                const uint2 x = s_info[cand];
                const uint32_t c1 = x.x & 0x3FFFu, c2 = (x.x >> 14) & 0x3FFFu;
                const uint32_t l0 = (x.y >> 14) & 63u, l1 = (x.y >> 20) & 63u, l2 = x.y >> 26;
                auto pair_bits = [&](uint32_t c) {
                    const uint32_t word = __umul24(prev, a.rw) + (c >> 5);
                    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(a.compat) + 4u * word) >>
                           (c & 31u);
                };
                const uint32_t w0 = pair_bits(cand), w1 = pair_bits(c1), w2 = pair_bits(c2);
                // bit i: position p + 1 + i is open
                const uint32_t sh = (p + 1) & 63u;
                const bool up = p >= 63;
                using Ahead = std::conditional_t<FAST, uint32_t, uint64_t>;
                const Ahead ahead =
                    (Ahead)(((up ? open.hi : open.lo) >> sh) | (((up ? 0ull : open.hi) << 1) << (63u - sh)));
                const uint32_t k0 = w0 & (uint32_t)(ahead >> l0) & 1u;
                const uint32_t k1 = w1 & (uint32_t)(ahead >> l1) & 1u;
                const uint32_t k2 = w2 & (uint32_t)(ahead >> l2) & 1u;
                if (k0 | k1 | k2) {
                    stack = (stack << 16) | prev;
                    prev = k0 ? cand : k1 ? c1 : c2;
                    p += 1 + (k0 ? l0 : k1 ? l1 : l2);
                    cand = best_at(p);
                    const Bits one = bit_only(p);
                    own.lo |= one.lo;
                    own.hi |= one.hi;
                    need = p != end;
                } else {
                    cand = x.y & 0x3FFFu;
                    if (cand == 0) {
                        // nothing fits after p: give the token before it up
                        const Bits one = bit_only(p);
                        open.lo &= ~one.lo;
                        open.hi &= ~one.hi;
                        own.lo &= ~one.lo;
                        own.hi &= ~one.hi;
                        cand = prev;  // ends at the closed position: the next shorter ones follow
                        prev = (uint32_t)stack & 0xFFFFu;
                        stack >>= 16;
                        if (p == 0) {
                            // no segmentation: never, every base is a token
                            dev::raise_error(a.count - HDR_BPE_FAILED, DNATOK_DERR_INTERNAL);
                            own.lo = 1;
                            need = false;
                            p = end;
                        } else {
                            p = highest(own);
                            if (p && !prev) {
                                const Bits here = bit_only(p);
                                const uint32_t p2 = highest(Bits{own.lo & ~here.lo, own.hi & ~here.hi});
                                prev = best_at(p2);
                                uint2 y = s_info[prev];
                                while (prev && info_len(y) != p - p2) {
                                    prev = info_link(y);
                                    y = s_info[prev];
                                }
                            }
                        }
                    }
                }
            }
        }

        // the stitch: the lane's own bits count from where the previous lane
        // met it, that lane's below
        const uint32_t met_at = from_prev(meet);  // by all lanes: a lane's move reads active lanes only
        const uint32_t from = prev_same ? met_at : 0u;
        const uint64_t below = (1ull << from) - 1;
        const uint64_t prev_hi = from_prev(own.hi);
        const Bits t{(own.lo & ~below) | (prev_hi & below), own.hi};
        // the token across a chunk end, for k_bpe_walk to compare. Lane 0 has
        // one only if its tokens go on in lane 1's: lane 1 keeps tokens that
        // start at its own chunk edge otherwise.
        if (lane == kLead - 1 || lane == 62) {
            const uint32_t side = lane == 62 ? 1u : 0u;
            uint32_t token = 0;
            if (next_same)
                token = t.lo && t.hi && (side || meet) ? 0x10000u | ((63u - (uint32_t)__builtin_clzll(t.lo)) << 8) |
                                                             (uint32_t)__builtin_ctzll(t.hi)
                                                       : 0x20000u + side;
            a.edge[2 * task + side] = token;
        }
        if (lane >= kLead && lane < 63 && valid) {
            const bool failed = next_same && !meet;
            const uint64_t m = left >= kChunk ? t.lo : t.lo & ((1ull << (uint32_t)left) - 1);
            a.mask[c] = m;
            a.row[c] = (uint32_t)r | (failed ? kFailed : 0u);
            if (failed) a.list[atomicAdd(a.count, 1u)] = (uint32_t)c;
            uint64_t rest = t.lo;
            for (uint64_t y = m; y;) {
                const uint32_t at0 = (uint32_t)__builtin_ctzll(y);
                y &= y - 1;
                rest &= ~(1ull << at0);
                const uint32_t at1 =
                    rest ? (uint32_t)__builtin_ctzll(rest) : t.hi ? 64u + (uint32_t)__builtin_ctzll(t.hi) : 128u;
                const uint32_t want = at1 - at0 - 1;
                uint32_t tok = best[at0 * 64 + lane];
                for (uint2 x = s_info[tok]; tok && ((x.y >> 14) & 63u) > want; x = s_info[tok])
                    tok = ((x.y >> 20) & 63u) == want ? x.x & 0x3FFFu
                          : (x.y >> 26) == want       ? (x.x >> 14) & 0x3FFFu
                                                      : x.y & 0x3FFFu;
                a.sym[s + at0] = (uint16_t)tok;
            }
        }
        wave_sync();
    }
}

// Carries the segmentation on, row by row, from each chunk that did not meet
// its neighbour: the same search with the row's own start bits as its stack,
// until it shares a token with the bits that the later chunks left (up to the
// next chunk that failed), or to the row's end. That happens in short tandem
// repeats, inside which segmentations from two starting points meet only where
// their distance is a multiple of the bases that the repeated tokens cover, so
// one may have to go on to the repeat's end. One wave per row: the longest
// tokens of 64 positions at a time, a token and the next two shorter ones tried
// together, and, where the tokens taken repeat and the text goes on repeating,
// the tokens of all repetitions written at once. Bound by the latency of the
// reads of a step. Whole encodes with the 4,096-merge table, in us, by merge
// rounds instead of chunks / by a walk of the same stretches that reads one
// token at a time and knows no cycles / now: CAG repeated to 20,000 bases 980 /
// 4,210 / 101, to 10^6 12,900 / 209,000 / 1,980; 1,024 rows of 500 to 20,000
// random bases with a repeat of 40 to 250 every 2,000 1,420 / 2,370 / 760.
constexpr int kRing = 64;        // tokens remembered, to find a cycle of up to half of them
constexpr int kCycle = 1024;     // bases of the longest cycle
constexpr int kCycleEvery = 8;   // tokens between two looks for one
constexpr int kCycleMin = 96;    // bases that are worth writing at once
__global__ __launch_bounds__(64) void k_bpe_walk(ChunkArgs a) {
    __shared__ uint16_t s_tok[kRing], s_cycle[kCycle];
    __shared__ int32_t s_at[kRing];
    const int64_t entries = *a.count;
    const int lane = threadIdx.x;
    const int64_t total = min(a.chunk_off[a.n], a.max_chunks), tasks = (total + kOwn - 1) / kOwn;
    const uint32_t longest_token = a.warm + 1;
    // whether chunk c (c < total) does not go on in chunk c + 1
    auto fails = [&](int64_t c) -> bool {
        if (a.row[c] & kFailed) return true;
        const int64_t t = c / kOwn;
        return c == t * kOwn + kOwn - 1 && t + 1 < tasks && a.edge[2 * t + 1] != a.edge[2 * (t + 1)];
    };
    auto walk_row = [&](int64_t r) {
        const int64_t cb = a.chunk_off[r], ce = min(a.chunk_off[r + 1], a.max_chunks);
        int64_t o0 = a.offs[r], o1 = a.offs[r + 1];
        o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
        o1 = o1 < o0 ? o0 : (o1 > a.nbytes ? a.nbytes : o1);
        // rows that overlap (malformed offsets) can have more chunks than there
        // are; the last row then ends with the last chunk
        const int64_t nch = ce - cb, L = min(o1 - o0, nch * (int64_t)kChunk);
        uint64_t *mask = a.mask + cb, *dead = a.dead + cb;
        uint64_t *old = a.pos + cb;
        const uint8_t *text = a.bytes + o0;
        uint16_t *sym = a.sym + o0;
        // Words of start bits and closed positions change by atomic operations
        // of one lane, which no step waits for, and are read past the L1.
        auto change = [&](uint64_t *words, int64_t p, bool set) {
            unsigned long long *w = reinterpret_cast<unsigned long long *>(words + (p >> 6));
            if (lane == 0) {
                if (set) atomicOr(w, 1ull << (p & 63));
                else atomicAnd(w, ~(1ull << (p & 63)));
            }
        };
        auto last_start = [&](int64_t p) -> int64_t {  // greatest start below p (p > 0)
            int64_t k = (p - 1) >> 6;
            uint64_t m = dev::ld_relaxed(mask + k) & (~0ull >> (63 - ((p - 1) & 63)));
            while (!m) m = dev::ld_relaxed(mask + --k);
            return (k << 6) + 63 - __builtin_clzll(m);
        };
        // the first chunk from k on that fails
        auto next_failed = [&](int64_t k) -> int64_t {
            for (; k < nch; k += 64) {
                const uint64_t hit = __ballot(k + lane < nch && fails(cb + k + lane));
                if (hit) return k + __builtin_ctzll(hit);
            }
            return nch;
        };
        // longest token at each of 64 positions, one per lane, and its entry
        int64_t window = -64;
        uint32_t best = 0;
        uint2 best_info{0, 0};
        auto look = [&](int64_t p) {
            if (p >= window && p < window + 64) return;
            window = p;
            best = 0;
            if (p + lane < L) {
                const uint32_t c0 = base_class(text[p + lane]);
                if (c0 > 3) {
                    best = c0 == 4 ? 9u : (uint32_t)DNATOK_ID_UNK;
                } else {
                    uint32_t node = 0, c = c0;
                    for (int64_t x = p + lane; x < L && c < 4;) {
                        ++x;
                        const uint32_t ahead = x < L ? base_class(text[x]) : 5u;  // asked for beside the node
                        const uint32_t h = a.kid[4 * node + c];
                        best = (h & 0xFFFFu) ? h & 0xFFFFu : best;
                        node = h >> 16;
                        c = node ? ahead : 5u;
                    }
                }
            }
            best_info = a.info[best];
        };
        int64_t f = next_failed(0);
        while (f < nch) {
            int64_t p = last_start((f + 1) << 6);
            const int64_t first = p;
            uint32_t prev = p ? sym[last_start(p)] : 0u;
            int64_t top = f, low = p >> 6;  // chunks entered; chunks whose closed positions are set up
            for (int64_t k = low; k <= top; ++k) dead[k] = 0;
            bool any_dead = false;
            auto enter = [&](int64_t to) {
                for (; top < to; ++top) {
                    const uint64_t m = dev::ld_relaxed(mask + top + 1);
                    if (lane == 0) {
                        old[top + 1] = m;
                        mask[top + 1] = 0;
                        dead[top + 1] = 0;
                    }
                }
            };
            // tokens taken; how many of the last ones the rings hold; those
            // taken until the next look for a cycle
            uint32_t taken = 0, kept = 0, until = kCycleEvery;
            int64_t resume = nch, held_at = -1;
            uint64_t held = 0;  // old[held_at]
            bool fresh = true;  // the longest token at p is tried first, else `cand`
            uint32_t cand = 0;
            uint2 x{0, 0};
            for (;;) {
                if (fresh) {
                    look(p);
                    const uint32_t at = (uint32_t)(p - window);
                    cand = dev::wave_read_u32(best, at);
                    x = uint2{dev::wave_read_u32(best_info.x, at), dev::wave_read_u32(best_info.y, at)};
                    fresh = false;
                } else if (cand) {
                    x = a.info[cand];
                }
                if (cand == 0) {
                    // nothing fits at p: give the token before it up
                    if (p == 0) {  // never, every base is a token
                        dev::raise_error(a.count - HDR_BPE_FAILED, DNATOK_DERR_INTERNAL);
                        return;
                    }
                    change(dead, p, true);
                    change(mask, p, false);
                    any_dead = true;
                    p = last_start(p);
                    for (; low > (p >> 6); --low)
                        if (lane == 0) dead[low - 1] = 0;
                    // its end is closed now, so a shorter one follows; a token
                    // that a chunk's own search took may have ended at the
                    // chunk's last base, so longer ones are tried too
                    fresh = kept == 0;
                    cand = prev;
                    if (kept) {
                        --kept;
                        --taken;
                    }
                    prev = kept ? s_tok[(taken - 1) % kRing] : p ? sym[last_start(p)] : 0u;
                    continue;
                }
                // it and the next two shorter ones, one per lane
                const uint32_t mine =
                    lane == 0 ? cand : lane == 1 ? x.x & 0x3FFFu : lane == 2 ? (x.x >> 14) & 0x3FFFu : 0u;
                const int64_t to = p + 1 + (lane == 0 ? (x.y >> 14) & 63u : lane == 1 ? (x.y >> 20) & 63u : x.y >> 26);
                bool fits = false;
                if (mine && to <= L) {
                    const uint32_t follow = a.compat[prev * a.rw + (mine >> 5)] >> (mine & 31u);
                    const bool closed =
                        any_dead && to < L && (to >> 6) <= top && ((dev::ld_relaxed(dead + (to >> 6)) >> (to & 63)) & 1ull);
                    fits = (follow & 1u) && !closed;
                }
                const uint64_t which = __ballot(fits);
                if (!which) {
                    cand = x.y & 0x3FFFu;
                    continue;
                }
                const uint32_t lane_of = (uint32_t)__builtin_ctzll(which);
                cand = dev::wave_read_u32(mine, lane_of);
                const int64_t q = p + dev::wave_read_u32((uint32_t)(to - p), lane_of);
                if (lane == 0) sym[p] = (uint16_t)cand;
                if (q == L) {
                    enter(nch - 1);
                    break;
                }
                enter(q >> 6);
                change(mask, q, true);
                // met: the bits it replaces hold this token too, in chunks that met
                if ((p >> 6) > f) {
                    const int64_t kp = p >> 6, kq = q >> 6;
                    if (held_at != kp) {
                        held_at = kp;
                        held = old[kp];
                    }
                    uint64_t m = held;
                    bool met = (m >> (p & 63)) & 1u;
                    m &= ~((2ull << (p & 63)) - 1);
                    int64_t k = kp;
                    for (; met && k < kq && !m; m = old[++k]) met = !fails(cb + k);
                    met = met && k == kq && m && __builtin_ctzll(m) == (int)(q & 63);
                    if (met) {
                        const uint64_t lower = (1ull << (q & 63)) - 1, m0 = dev::ld_relaxed(mask + kq);
                        if (lane == 0) {
                            mask[kq] = (m0 & lower) | (old[kq] & ~lower);
                            for (int64_t i = kq + 1; i <= top; ++i) mask[i] = old[i];
                        }
                        resume = kq;
                        break;
                    }
                }
                if (lane == 0) {
                    s_tok[taken % kRing] = (uint16_t)cand;
                    s_at[taken % kRing] = (int32_t)(p - first);
                }
                ++taken;
                kept = min(kept + 1, (uint32_t)kRing);
                prev = cand;
                p = q;
                fresh = true;
                wave_sync();
                if (--until) continue;
                until = kCycleEvery;
                // lane i: whether the last i + 1 tokens are those before them once more
                const uint32_t j = (uint32_t)lane + 1;
                bool again = 2 * j <= kept;
                for (uint32_t i = 1; again && i <= j; ++i)
                    again = s_tok[(taken - i) % kRing] == s_tok[(taken - i - j) % kRing];
                const uint64_t cycles = __ballot(again);
                if (!cycles) continue;
                const uint32_t tokens = (uint32_t)__builtin_ctzll(cycles) + 1u;
                const int64_t begin = first + s_at[(taken - tokens) % kRing], bases = p - begin;
                if (bases > kCycle) continue;
                // where the text stops repeating: 16 bases per lane
                int64_t end = p;
                for (;;) {
                    const int64_t at = end + 16 * lane;
                    int same = 0;
                    if (at + 16 <= L) {
                        uint64_t u[2], v[2];
                        __builtin_memcpy(u, text + at, 16);
                        __builtin_memcpy(v, text + at - bases, 16);
                        const uint64_t d0 = (u[0] ^ v[0]) & ~0x2020202020202020ull;
                        const uint64_t d1 = (u[1] ^ v[1]) & ~0x2020202020202020ull;
                        same = d0 ? __builtin_ctzll(d0) / 8 : d1 ? 8 + __builtin_ctzll(d1) / 8 : 16;
                    } else {
                        while (at + same < L && ((text[at + same] ^ text[at + same - bases]) & ~0x20u) == 0) ++same;
                    }
                    const uint64_t ends = __ballot(same < 16);
                    if (ends) {
                        const uint32_t l = (uint32_t)__builtin_ctzll(ends);
                        end += 16 * l + dev::wave_read_u32((uint32_t)same, l);
                        break;
                    }
                    end += 16 * 64;
                }
                // Every pair of the cycle has been found to fit, so the tokens
                // of its repetitions are the row's as far as the text repeats;
                // the last bases are left to the search.
                const int64_t room = end - 2 * (int64_t)longest_token - p;
                const int64_t past = p + (room > 0 ? room / bases * bases : 0);
                if (past - p < kCycleMin) continue;
                for (int64_t o = lane; o < bases; o += 64) s_cycle[o] = 0;
                wave_sync();
                if ((uint32_t)lane < tokens) {
                    const uint32_t i = (taken - tokens + (uint32_t)lane) % kRing;
                    s_cycle[first + s_at[i] - begin] = s_tok[i];
                }
                wave_sync();
                for (int64_t k = (p >> 6) + lane; k <= past >> 6; k += 64) {
                    const int64_t x0 = max(k * 64, p), x1 = min(k * 64 + 63, past);
                    const uint64_t m = dev::ld_relaxed(mask + k);
                    uint64_t w = 0;
                    uint32_t o = (uint32_t)((x0 - p) % bases);
                    for (int64_t y = x0; y <= x1; ++y) {
                        const uint16_t token = s_cycle[o];
                        if (token) {
                            w |= 1ull << (y & 63);
                            if (y < past) sym[y] = token;
                        }
                        o = o + 1 == (uint32_t)bases ? 0u : o + 1;
                    }
                    if (k > top) {
                        old[k] = m;
                        dead[k] = 0;
                    } else {
                        w |= m;
                    }
                    mask[k] = w;
                }
                __threadfence();
                top = max(top, past >> 6);
                p = past;
                kept = 0;
            }
            f = next_failed(resume);
        }
    };
    // Rows with a chunk that fails. A wave looks at 64 such chunks and takes
    // one row of theirs at a time, so that others find the rest.
    const int64_t items = entries + max(tasks - 1, (int64_t)0);
    const uint32_t turn = blockIdx.x % 64;
    for (int64_t i0 = 0; i0 < items; i0 += (int64_t)gridDim.x * 64) {
        const int64_t i = i0 + (int64_t)lane * gridDim.x + blockIdx.x;
        int64_t c = -1, first = 0;
        if (i < entries) {
            c = a.list[i];
        } else if (i < items) {
            const int64_t k = (i - entries) * kOwn + kOwn - 1;
            if (!(a.row[k] & kFailed) && fails(k)) c = k;
        }
        uint32_t row = 0;
        if (c >= 0) {
            row = a.row[c] & kRowBits;
            first = a.chunk_off[row];
        }
        for (;;) {
            const uint64_t open = __ballot(c >= 0 && !(dev::ld_relaxed32(a.row + first) & kTaken));
            if (!open) break;
            const uint64_t turned = turn ? (open >> turn) | (open << (64 - turn)) : open;
            const uint32_t pick = ((uint32_t)__builtin_ctzll(turned) + turn) % 64;
            const uint32_t was = (uint32_t)lane == pick ? atomicOr(a.row + first, kTaken) : 0u;
            const uint32_t mine = dev::wave_read_u32(row, pick);
            if (!(dev::wave_read_u32(was, pick) & kTaken)) walk_row(mine);
        }
    }
}

struct CountArgs {
    const uint64_t *mask;
    const int64_t *total_at;  // chunk_off[n]
    int64_t *pos;
    int64_t max_chunks;
    int64_t nunits;
    dev::TileQueue q;
};

// Exclusive scan of the chunks' token counts, units of 1,024 chunks.
__global__ __launch_bounds__(kPutNT) void k_bpe_count(CountArgs a) {
    __shared__ int64_t s_tmp[kPutNT / dev::kWave + 1];
    __shared__ int64_t s_unit, s_excl;
    const int tid = threadIdx.x;
    const uint32_t parity = dev::ld_relaxed32(a.q.hdr + 2);
    uint64_t *st = parity ? a.q.status1 : a.q.status0;
    uint64_t *st_other = parity ? a.q.status0 : a.q.status1;
    const int64_t total = min(*a.total_at, a.max_chunks);
    const int64_t units = max((total + kCountUnit - 1) / kCountUnit, (int64_t)1);
    for (;;) {
        if (tid == 0) s_unit = (int64_t)atomicAdd(a.q.hdr + 0, 1u);
        __syncthreads();
        const int64_t u = s_unit;
        __syncthreads();
        if (u >= a.nunits) break;
        for (int64_t j = u + (int64_t)tid * a.nunits; j < a.q.clear_n; j += (int64_t)kPutNT * a.nunits)
            st_other[j] = 0;
        if (u >= units) continue;  // beyond the chunks present: nothing to chain
        const int64_t i0 = u * kCountUnit + (int64_t)tid * kCountPerThread;
        uint32_t v[kCountPerThread];
        int64_t mine = 0;
#pragma unroll
        for (int j = 0; j < kCountPerThread; ++j) {
            const uint64_t x = total > 0 ? a.mask[i0 + j < total ? i0 + j : total - 1] : 0ull;
            v[j] = i0 + j < total ? (uint32_t)__popcll(x) : 0u;
            mine += v[j];
        }
        int64_t utot;
        const int64_t pre = dev::block_excl_scan<kPutNT>(mine, s_tmp, &utot);
        if (tid < dev::kWave) {
            if (tid == 0) dev::publish_aggregate(st, u, utot);
            const int64_t ex = dev::wave_lookback(st, u, utot, a.q.hdr);
            if (tid == 0) s_excl = ex;
        }
        __syncthreads();
        int64_t run = s_excl + pre;
#pragma unroll
        for (int j = 0; j < kCountPerThread; ++j) {
            if (i0 + j < total) a.pos[i0 + j] = run;
            run += v[j];
        }
        if (u == units - 1 && tid == 0) a.pos[total] = s_excl + utot;
        __syncthreads();
    }
    if (tid == 0) dev::finish_block(a.q.hdr);
}

struct PutArgs {
    const int64_t *offs;
    int64_t nbytes;
    int32_t n;
    const int64_t *chunk_off;
    int64_t max_chunks;
    const uint64_t *mask;
    const uint32_t *row;
    const int64_t *pos;
    const uint16_t *sym;
    int32_t *ids;
    int64_t cap;
    int64_t *out_offs;
    int8_t *mask_out;
    int32_t cls, padded, left;
    int32_t pad_id, cls_id, sep_id;
    int64_t W;
    int64_t base;
    uint32_t *hdr;
};

// Ids of every chunk, four threads each (a thread's tokens are a chain of
// reads and stores; one thread per chunk took 12.1 us on the 1,024-row batch,
// four 7.0), then the rows' offsets, specials and pads. The list of failed
// chunks is emptied for the next launch.
__global__ __launch_bounds__(kPutNT) void k_bpe_put(PutArgs a) {
    const int tid = threadIdx.x;
    const int64_t gid = (int64_t)blockIdx.x * kPutNT + tid, threads = (int64_t)gridDim.x * kPutNT;
    uint32_t err = 0;
    auto first_chunk = [&](int64_t i) { return min(a.chunk_off[i], a.max_chunks); };
    const int64_t total = first_chunk(a.n);
    if (gid == 0) {
        dev::st_relaxed32(a.hdr + HDR_BPE_FAILED, 0u);
        if (a.n == 0) a.out_offs[0] = a.base;
    }
    for (int64_t g = gid; g < 4 * total; g += threads) {
        const int64_t c = g >> 2;
        const uint64_t all = a.mask[c];
        const uint32_t from = 16 * (uint32_t)(g & 3);
        uint64_t m = all & (0xFFFFull << from);
        const int64_t before = __popcll(all & ((1ull << from) - 1));
        const int64_t i = a.row[c] & kRowBits;
        const int64_t cb = a.chunk_off[i];
        int64_t o0 = a.offs[i];
        o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
        const uint16_t *src = a.sym + o0 + kChunk * (c - cb);
        if (!a.padded) {
            int64_t d = a.pos[c] + before + 2 * a.cls * i + a.cls;
            for (; m; m &= m - 1, ++d) {
                if (d < a.cap) a.ids[d] = src[__builtin_ctzll(m)];
                else err |= DNATOK_DERR_CAPACITY;
            }
        } else {
            const int64_t r0 = a.pos[first_chunk(i)], len = a.pos[first_chunk(i + 1)] - r0 + 2 * a.cls;
            if (len > a.W) continue;
            int64_t d = i * a.W + (a.left ? a.W - len : 0) + a.cls + (a.pos[c] + before - r0);
            for (; m; m &= m - 1, ++d) {
                a.ids[d] = src[__builtin_ctzll(m)];
                a.mask_out[d] = 1;
            }
        }
    }
    if (!a.padded) {
        for (int64_t i = gid; i < a.n; i += threads) {
            const int64_t d0 = a.pos[first_chunk(i)] + 2 * a.cls * i;
            const int64_t d1 = a.pos[first_chunk(i + 1)] + 2 * a.cls * (i + 1);
            a.out_offs[i] = a.base + d0;
            if (i == a.n - 1) a.out_offs[a.n] = a.base + d1;
            if (a.cls) {
                if (d0 < a.cap) a.ids[d0] = a.cls_id;
                if (d1 - 1 < a.cap) a.ids[d1 - 1] = a.sep_id;
                else err |= DNATOK_DERR_CAPACITY;
            }
        }
    } else {
        for (int64_t i = blockIdx.x; i < a.n; i += gridDim.x) {
            const int64_t p0 = a.pos[first_chunk(i)], p1 = a.pos[first_chunk(i + 1)];
            const int64_t len = p1 - p0 + 2 * a.cls;
            if (tid == 0) {
                a.out_offs[i] = a.base + p0 + 2 * a.cls * i;
                if (i == a.n - 1) a.out_offs[a.n] = a.base + p1 + 2 * a.cls * a.n;
            }
            if (len > a.W) {
                err |= DNATOK_DERR_ROW_WIDTH;
                continue;
            }
            const int64_t lead = a.left ? a.W - len : 0;
            int32_t *row = a.ids + i * a.W;
            int8_t *mrow = a.mask_out + i * a.W;
            if (a.cls && tid == 0) {
                row[lead] = a.cls_id;
                mrow[lead] = 1;
                row[lead + len - 1] = a.sep_id;
                mrow[lead + len - 1] = 1;
            }
            const int64_t from = a.left ? 0 : len;  // the row's W - len pads
            for (int64_t x = tid; x < a.W - len; x += kPutNT) {
                row[from + x] = a.pad_id;
                mrow[from + x] = 0;
            }
        }
    }
    if (err) dev::raise_error(a.hdr, err);
}

// Scratch of one call, laid out inside the bytes that the item path needs.
struct ChunkScratch {
    int64_t max_chunks, sym, bits, words, edge, pos, off, total;
};
ChunkScratch chunk_scratch(int64_t nbytes, int32_t n) {
    auto al = [](int64_t x) { return (x + 255) / 256 * 256; };
    ChunkScratch b;
    b.max_chunks = nbytes / kChunk + (int64_t)n + 1;
    b.sym = al(2 * (nbytes + 1));
    b.bits = al(8 * b.max_chunks);
    b.words = al(4 * b.max_chunks);
    b.edge = al(8 * (b.max_chunks / kOwn + 1));
    b.pos = al(8 * (b.max_chunks + 1));
    b.off = al(8 * ((int64_t)n + 1));
    b.total = b.sym + 2 * b.bits + 2 * b.words + b.edge + b.pos + b.off;
    return b;
}
// Waves of a workgroup that fit beside its tables; *automaton: the FAST
// kernel, unless a token is too long for it or it would leave room for fewer
// than four waves.
int chunk_waves(const dnatok_vocab *v, bool *automaton, uint32_t *tables) {
    const BpeTables &t = v->bpe;
    const uint32_t info = lds_info(10u + (uint32_t)t.n_merges), both = lds_next(t.n_states) + lds_longest(t.n_states);
    *automaton = v->max_token_bytes <= 32 && info + both + 4 * kLdsPerWave <= kLdsRoom;
    *tables = info + (*automaton ? both : 0u);
    return (int)std::min<size_t>(kMaxWavesPerGroup, (kLdsRoom - *tables) / kLdsPerWave);
}

}  // namespace

int64_t bpe_chunk_tiles(int64_t nbytes, int32_t n) {
    return (chunk_scratch(nbytes, n).max_chunks + kCountUnit - 1) / kCountUnit;
}

int launch_bpe_chunks(const dnatok_vocab *v, const uint8_t *d_bytes, int64_t nbytes, const int64_t *d_offsets,
                      int32_t n, int32_t *d_ids, int64_t cap, int64_t *d_out_offsets, int8_t *d_mask,
                      const dnatok_encode_opts &o, Workspace *ws, hipStream_t stream, bool *used) {
    const BpeTables &bt = v->bpe;
    *used = false;
    // The item path instead: a token of more than 64 bases (the walk reads 64
    // at a time), a table of more states than the automaton's entries hold, a
    // batch whose chunk indices pass 30 bits, or scratch that holds the item
    // path's arrays but not these.
    const ChunkScratch cs = chunk_scratch(nbytes, n);
    if (!bt.chunked || cs.max_chunks >= (int64_t)1 << 30 || cs.total > ws->scratch_bytes) return DNATOK_OK;
    bool automaton = false;
    uint32_t tables = 0;
    const int most = chunk_waves(v, &automaton, &tables);
    const int64_t units = bpe_chunk_tiles(nbytes, n);
    if (units > ws->cap) return DNATOK_OK;
    *used = true;
    uint8_t *sp = ws->d_scratch;
    auto take = [&](int64_t bytes) {
        uint8_t *p = sp;
        sp += bytes;
        return p;
    };
    ChunkArgs a;
    a.bytes = d_bytes;
    a.nbytes = nbytes;
    a.offs = d_offsets;
    a.n = n;
    int64_t *chunk_off = reinterpret_cast<int64_t *>(take(cs.off));
    a.chunk_off = chunk_off;
    a.max_chunks = cs.max_chunks;
    a.pos = reinterpret_cast<uint64_t *>(take(cs.pos));
    a.mask = reinterpret_cast<uint64_t *>(take(cs.bits));
    a.dead = reinterpret_cast<uint64_t *>(take(cs.bits));
    a.row = reinterpret_cast<uint32_t *>(take(cs.words));
    a.list = reinterpret_cast<uint32_t *>(take(cs.words));
    a.edge = reinterpret_cast<uint32_t *>(take(cs.edge));
    a.sym = reinterpret_cast<uint16_t *>(take(cs.sym));
    a.count = ws->d_hdr + HDR_BPE_FAILED;
    a.next = reinterpret_cast<const uint16_t *>(bt.d_chunk);
    a.longest = bt.d_longest;
    a.info = bt.d_info;
    a.kid = bt.d_kid;
    a.compat = bt.d_compat;
    a.V = 10u + (uint32_t)bt.n_merges;
    a.rw = bt.rw;
    a.n_states = bt.n_states;
    a.warm = (uint32_t)v->max_token_bytes - 1;
    const int cus = device_cu_count();
    int rc = launch_rowscan(d_offsets, n, nbytes, chunk_off, kChunk, 0, stream, true);
    if (rc) return rc;

    // one workgroup per CU (the tables fill a third of its LDS), the tasks
    // spread over all of them before a workgroup gets a second wave; at least
    // two waves, which share the copy of the tables
    const int64_t tasks = std::max<int64_t>(1, (cs.max_chunks + kOwn - 1) / kOwn);
    const int64_t groups = std::min<int64_t>(tasks, cus);
    const int waves = (int)std::min<int64_t>(most, std::max<int64_t>(kMinWavesPerGroup, (tasks + groups - 1) / groups));
    const uint32_t lds = tables + (uint32_t)waves * kLdsPerWave;
    auto *chunks = automaton ? k_bpe_chunks<true> : k_bpe_chunks<false>;
    DNATOK_HIP(hipFuncSetAttribute((const void *)chunks, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(chunks, dim3((unsigned)groups), dim3(64 * waves), lds, stream, a);
    DNATOK_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_bpe_walk, dim3((unsigned)std::min<int64_t>(n > 0 ? n : 1, 8 * (int64_t)cus)), dim3(64), 0, stream, a);
    DNATOK_HIP(hipGetLastError());

    CountArgs ca;
    ca.mask = a.mask;
    ca.total_at = chunk_off + n;
    ca.pos = reinterpret_cast<int64_t *>(a.pos);
    ca.max_chunks = cs.max_chunks;
    ca.nunits = units;
    ca.q.hdr = ws->d_hdr;
    ca.q.status0 = ws->d_status;
    ca.q.status1 = ws->d_status + ws->cap;
    if (units > ws->high_water) ws->high_water = units;
    ca.q.clear_n = ws->high_water;
    hipLaunchKernelGGL(k_bpe_count, dim3((unsigned)std::min<int64_t>(units, (int64_t)cus * 4)), dim3(kPutNT), 0,
                       stream, ca);
    DNATOK_HIP(hipGetLastError());

    PutArgs e;
    e.offs = d_offsets;
    e.nbytes = nbytes;
    e.n = n;
    e.chunk_off = chunk_off;
    e.max_chunks = cs.max_chunks;
    e.mask = a.mask;
    e.row = a.row;
    e.pos = reinterpret_cast<const int64_t *>(a.pos);
    e.sym = a.sym;
    e.ids = d_ids;
    e.cap = cap;
    e.out_offs = d_out_offsets;
    e.mask_out = d_mask;
    e.cls = o.add_cls_sep ? 1 : 0;
    e.padded = o.layout == DNATOK_PADDED ? 1 : 0;
    e.left = o.pad_side == DNATOK_PAD_LEFT ? 1 : 0;
    e.pad_id = v->pad_id;
    e.cls_id = v->cls_id;
    e.sep_id = v->sep_id;
    e.W = e.padded ? o.pad_to : 0;
    e.base = o.offset_base;
    e.hdr = ws->d_hdr;
    const int64_t work = std::max<int64_t>((4 * cs.max_chunks + kPutNT - 1) / kPutNT, e.padded ? n : 1);
    hipLaunchKernelGGL(k_bpe_put, dim3((unsigned)std::min<int64_t>(work, (int64_t)cus * 8)), dim3(kPutNT), 0, stream,
                       e);
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

}  // namespace dnatok
