// Decode: ids -> uppercase bases (the inverse table the paper lists as
// future work, Discussion, "Decode Operations": the same LUT principle run
// backwards). Not on the hot path.
//
// Tiles of token positions, each tile's output bytes contiguous, one
// workgroup per tile: it reads its ids once, sums its output bytes, takes its
// output position from the tiles before it, stages its bytes in LDS and
// writes them with 16-byte stores. Tiles follow the workgroup index: a
// workgroup starts only after every lower-indexed one on its XCD, and the
// XCDs take workgroups in index order, so the tile with the lowest index
// still running never waits and every wait ends (with no ticket counter: one
// device-wide counter serializes at about 12 ns per ticket, which at
// thousands of tiles outweighs the decode).
//
// Single-nucleotide and k-mer ids are K bytes or none each (k_decode_fixed),
// BPE ids tokens of any length (k_decode_bpe); both take one launch.
#include "common.hpp"
#include "device.hpp"

namespace dnatok {

namespace {

constexpr int NT = 256;
constexpr int kMaxStage = 32768;  // most bytes of a BPE tile's output staged in LDS
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t ids4 __attribute__((ext_vector_type(4), aligned(4)));

struct DecodeArgs {
    const int32_t *ids;
    int64_t n_ids;
    const int64_t *offs;
    int32_t n;
    uint8_t *out;
    int64_t cap;
    int64_t *out_offs;
    int32_t vocab;
    const int32_t *tok_len;
    const int64_t *tok_off;
    const uint8_t *tok_chars;
    int64_t ntiles;
    int32_t stage;       // bytes the LDS stage holds (a tile with more output writes its tokens directly)
    uint32_t *err_hdr;
    double rows_per_id;
    uint32_t codes;      // 4^k
};

__device__ __forceinline__ bool is_silent(int32_t id) {
    return id == DNATOK_ID_PAD || id == DNATOK_ID_CLS || id == DNATOK_ID_SEP || id == DNATOK_ID_MASK;
}

// Output bytes of one BPE id.
__device__ __forceinline__ int32_t width_of(const DecodeArgs &a, int32_t id) {
    if (is_silent(id)) return 0;
    return id >= 10 && id < a.vocab ? a.tok_len[id] : 1;
}

// The letter of 2-bit code c (0..3: A, C, G, T) from one packed word: a
// table in memory would cost a dependent load per base.
__device__ __forceinline__ uint8_t base_letter(uint32_t c) { return (uint8_t)(0x54474341u >> (8 * (c & 3))); }

// The letter of a single-nucleotide id (N and unknown ids: 'N').
__device__ __forceinline__ uint8_t single_letter(int32_t id) {
    return (id >= 5 && id <= 8) ? base_letter((uint32_t)(id - 5)) : (uint8_t)'N';
}

__device__ __forceinline__ void write_token(const DecodeArgs &a, int32_t id, int64_t pos, uint32_t &err) {
    if (is_silent(id)) return;
    if (id >= 10 && id < a.vocab) {
        const int64_t L = a.tok_len[id], o = a.tok_off[id];
#pragma unroll 1
        for (int64_t j = 0; j < L; ++j) {
            if (pos + j < a.cap) a.out[pos + j] = a.tok_chars[o + j];
            else err |= DNATOK_DERR_CAPACITY;
        }
        return;
    }
    if (pos < a.cap) a.out[pos] = single_letter(id);
    else err |= DNATOK_DERR_CAPACITY;
}

// The staged output of a tile (agg bytes from stage byte 0) to out + base:
// output byte base + b is stage byte b, for b below the capacity (past it:
// the flag); the output's 16-byte units from out + base - ph on, each read
// from the stage as 5 dwords realigned by ph.
__device__ __forceinline__ void store_stage(const DecodeArgs &a, const uint8_t *s_out, int64_t base, int64_t agg,
                                            uint32_t &err) {
    const int tid = threadIdx.x;
    const int64_t room = a.cap - base;
    const int64_t lim = room <= 0 ? 0 : (room < agg ? room : agg);
    if (lim < agg) err |= DNATOK_DERR_CAPACITY;
    const int32_t ph = (int32_t)((reinterpret_cast<uintptr_t>(a.out) + (uintptr_t)base) & 15);
    uint8_t *ob = a.out + base - ph;
    const uint32_t *s32 = reinterpret_cast<const uint32_t *>(s_out);
    const int32_t bytes = (int32_t)lim, nu = lim > 0 ? (ph + bytes + 15) / 16 : 0;  // lim < 2^16
    for (int32_t u = tid; u < nu; u += NT) {
        const int32_t lo = 16 * u - ph, hi = lo + 16;  // the unit's stage bytes
        if (lo >= 0 && hi <= bytes) {
            const uint32_t w0 = (uint32_t)lo >> 2, r = (uint32_t)lo & 3;
            uint32_t w[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) w[q] = s32[w0 + q];
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = __builtin_amdgcn_alignbyte(w[q + 1], w[q], r);
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(ob + 16 * u));
        } else {
            for (int32_t b = (lo > 0 ? lo : 0); b < hi && b < bytes; ++b) ob[ph + b] = s_out[b];
        }
    }
}

// State of the scan over tiles: per tile its output bytes, per
// group of 64 tiles and per super of 64 groups their sum, each word complete
// when bit 63 is set. The last tile of a group adds its group up as soon as
// the group's tiles have published, so a group hangs on no look-back, and the
// position of any tile is the sum of the supers, groups and tiles before it
// within its own super and group: two or three loads of one wave, whereas in
// a chain of inclusive prefixes a position takes a round trip per 64 tiles
// (2,000 resident tiles: 8 to 10 us). Words are stored, never added to:
// 4,096 atomic adds on counters in a few lines took 200 us.
// The words are held twice. A launch works on the half that head[0] names
// and clears what the launch before it (head[1 + half]: its tiles) left in
// the other; its last tile, which has seen every tile publish and so every
// tile's read of head[0], then changes the half.
struct ScanState {
    uint64_t *head;  // half, tiles left in half 0, in half 1
    uint64_t *half[2];
    int64_t tiles, groups;  // capacity: tile words, then group words, then super words
};
constexpr int64_t kHeadWords = 16;
inline int64_t scan_groups(int64_t tiles) { return (tiles + 63) / 64; }
inline int64_t half_words(int64_t tiles) { return tiles + scan_groups(tiles) + scan_groups(scan_groups(tiles)); }
inline int64_t scan_words(int64_t tiles) { return kHeadWords + 2 * half_words(tiles); }
inline ScanState scan_state(uint64_t *w, int64_t tiles) {
    return ScanState{w, {w + kHeadWords, w + kHeadWords + half_words(tiles)}, tiles, scan_groups(tiles)};
}
constexpr uint64_t kComplete = 1ull << 63;

// Sum of the complete words p[i] for i in [lo, hi), waited for by one wave.
// A word that stays incomplete for kLookbackMaxPolls polls raises
// DNATOK_DERR_INTERNAL and counts what it has: every launch drains.
__device__ __forceinline__ int64_t sum_complete(const uint64_t *p, int64_t lo, int64_t hi, uint32_t *hdr) {
    const int lane = threadIdx.x & (dev::kWave - 1);
    int64_t sum = 0;
    for (int64_t j = lo; j < hi; j += dev::kWave) {
        const bool live = j + lane < hi;
        uint64_t w = live ? dev::ld_relaxed(p + j + lane) : kComplete;
        uint32_t polls = 0;
        while (__ballot(!(w & kComplete))) {
            if (++polls >= dev::kLookbackMaxPolls) {
                if (lane == 0) dev::raise_error(hdr, DNATOK_DERR_INTERNAL);
                break;
            }
            __builtin_amdgcn_s_sleep(4);
            if (!(w & kComplete)) w = dev::ld_relaxed(p + j + lane);
        }
        sum += live ? (int64_t)(w & (kComplete - 1)) : 0;
    }
    return dev::wave_sum(sum);
}

// Row r's offsets, checked: a tile looks at kCheckRows rows (whatever their
// place), further workgroups at kCheckBlock of those left.
constexpr int kCheckRows = dev::kWave, kCheckBlock = 8 * NT;
__device__ __forceinline__ uint32_t check_rows(const DecodeArgs &a, int64_t r) {
    if (r >= a.n) return 0;
    const int64_t o0 = a.offs[r], o1 = a.offs[r + 1];
    return o0 < 0 || o1 < o0 || o1 > a.n_ids ? DNATOK_DERR_OFFSETS : 0;
}

// The rows past those that tiles check.
__device__ __forceinline__ void check_rest(const DecodeArgs &a, int64_t block) {
    const int64_t r0 = a.ntiles * kCheckRows + block * kCheckBlock;
    uint32_t err = 0;
    for (int64_t r = r0 + threadIdx.x; r < r0 + kCheckBlock; r += NT) err |= check_rows(a, r);
    if (err) dev::raise_error(a.err_hdr, err);
}

// The half of the state that this launch works on, and what is left to clear
// in the other.
struct ScanView {
    uint64_t half;
    int64_t left;
    uint64_t *tile, *group, *super, *other;
};
__device__ __forceinline__ ScanView scan_view(const ScanState &st) {
    ScanView v;
    v.half = dev::ld_relaxed(st.head) & 1u;
    v.left = (int64_t)dev::ld_relaxed(st.head + 2 - v.half);
    v.tile = v.half ? st.half[1] : st.half[0];
    v.other = v.half ? st.half[0] : st.half[1];
    v.group = v.tile + st.tiles;
    v.super = v.group + st.groups;
    return v;
}
// Publishes tile t's bytes (one thread of the first wave) and clears a share
// of the other half (all threads).
__device__ __forceinline__ void publish_tile(const ScanState &st, const ScanView &v, int64_t t, int64_t ntiles,
                                             int64_t agg) {
    if (threadIdx.x == 0) dev::st_relaxed(v.tile + t, kComplete | (uint64_t)agg);
    for (int64_t i = t * NT + threadIdx.x; i < v.left; i += ntiles * NT) {
        dev::st_relaxed(v.other + i, 0);
        if (i % 64 == 0) dev::st_relaxed(v.other + st.tiles + i / 64, 0);
        if (i % 4096 == 0) dev::st_relaxed(v.other + st.tiles + st.groups + i / 4096, 0);
    }
}
// Bytes before tile t, by one wave. Nearest words first: the older ones are
// then there already.
__device__ __forceinline__ int64_t tile_position(const ScanView &v, int64_t t, int64_t agg, uint32_t *hdr) {
    const int64_t g = t / 64, sp = g / 64;
    const bool one = (threadIdx.x & (dev::kWave - 1)) == 0;
    int64_t sum = sum_complete(v.tile, g * 64, t, hdr);
    if (t % 64 == 63 && one) dev::st_relaxed(v.group + g, kComplete | (uint64_t)(sum + agg));
    sum += sum_complete(v.group, sp * 64, g, hdr);
    if (t % 4096 == 4095 && one) dev::st_relaxed(v.super + sp, kComplete | (uint64_t)(sum + agg));
    return sum + sum_complete(v.super, 0, sp, hdr);
}
// The last tile ends the offsets and hands the other half to the next launch
// (one thread).
__device__ __forceinline__ void finish_tiles(const DecodeArgs &a, const ScanState &st, const ScanView &v,
                                             int64_t total) {
    a.out_offs[a.n] = total;
    dev::st_relaxed(st.head + 1 + v.half, (uint64_t)a.ntiles);
    dev::st_relaxed(st.head, v.half ^ 1u);
}

// The rows around a tile: the offsets of 64 from g0 on (asked for early by
// one wave, g0 being where the tile would start if rows were equally long),
// and the first row that starts in the tile.
struct TileRows {
    int64_t po[dev::kWave];
    int64_t g0, ia;
};
__device__ __forceinline__ int64_t probe_rows(const DecodeArgs &a, int64_t P0, int64_t *g0) {
    int64_t g = (int64_t)((double)P0 * a.rows_per_id) - dev::kWave / 2;
    if (g + dev::kWave > a.n) g = a.n - dev::kWave;
    if (g < 0) g = 0;
    *g0 = g;
    return a.offs[min(g + (int64_t)(threadIdx.x & (dev::kWave - 1)), (int64_t)a.n)];
}
__device__ __forceinline__ void find_rows(const DecodeArgs &a, int64_t P0, int64_t g0, int64_t po, TileRows &rows) {
    const int lane = threadIdx.x & (dev::kWave - 1);
    const int64_t n = a.n;
    auto pred = [&](int64_t r) { return a.offs[r] >= P0; };
    const uint64_t hit = __ballot(g0 + lane < n ? po >= P0 : true);
    int64_t ia;
    if ((hit & 1ull) && g0 > 0) ia = dev::wave_lower_bound(0, g0, pred);
    else if (hit == 0) ia = dev::wave_lower_bound(g0 + dev::kWave, n, pred);
    else ia = g0 + __builtin_ctzll(hit);
    rows.po[lane] = po;
    if (lane == 0) {
        rows.ia = min(ia, n);
        rows.g0 = g0;
    }
}
// Output offsets of the rows that start in [P0, P0 + tt) (the last tile: from
// P0 on); bytes_at(rel): the tile's bytes before its position rel.
template <class F>
__device__ __forceinline__ void put_rows(const DecodeArgs &a, const TileRows &rows, int64_t P0, int64_t tt, bool last,
                                         int64_t base, F bytes_at) {
    const int64_t w0 = rows.g0, end = last ? INT64_MAX : P0 + tt;
    auto offset = [&](int64_t i) { return i >= w0 && i - w0 < dev::kWave ? rows.po[i - w0] : a.offs[i]; };
    int64_t i = rows.ia + threadIdx.x, o = i < a.n ? offset(i) : INT64_MAX;
    // a tile of more rows than threads (empty rows, rows of a few ids): the next
    // row's place asked for ahead, equal places looked up once (100,000 empty
    // rows 152 us without, 86 so)
    int64_t seen = -1, at = 0;
    while (o < end && i < a.n) {
        const int64_t next = i + NT < a.n ? offset(i + NT) : INT64_MAX;
        if (o != seen) at = base + bytes_at((int32_t)min(max(o - P0, (int64_t)0), tt));
        seen = o;
        a.out_offs[i] = at;
        i += NT;
        o = next;
    }
}

// The K letters of known k-mer code v, first letter in the low byte of w[0];
// bytes past the K-th are zero. known false: K letters N.
template <int K>
__device__ __forceinline__ void letters(uint32_t v, bool known, uint32_t (&w)[(K + 3) / 4]) {
#pragma unroll
    for (int i = 0; i < (K + 3) / 4; ++i) {
        constexpr int kLast = K % 4 ? K % 4 : 4;
        const int have = i == (K + 3) / 4 - 1 ? kLast : 4, at = 2 * (K - 4 * i - 4);  // digits below the word's
        uint32_t f = (at >= 0 ? v >> (at > 0 ? at : 0) : v << (at < 0 ? -at : 0)) & 0xFFu;
        f = (f | (f << 12)) & 0x000F000Fu;
        f = (f | (f << 6)) & 0x03030303u;  // digit j in byte j
        const uint32_t x = __builtin_bswap32(__builtin_amdgcn_perm(0u, 0x54474341u, f));
        const uint32_t mask = have == 4 ? 0xFFFFFFFFu : (1u << (8 * have)) - 1u;
        w[i] = (known ? x : 0x4E4E4E4Eu) & mask;
    }
}

// Single-nucleotide and k-mer ids. A wave takes U slices of 256 consecutive
// ids, four per lane. A slice without a silent id (PAD, CLS, SEP, MASK) is
// 256 K contiguous bytes, K dwords per lane at constant shifts; the others
// place each id by the ballots of the non-silent ones below it. The kernel is
// bound by the VALU beside its traffic (an instruction per id takes 0.85 us
// for 33.6M ids): four ids in a vector, their letters from byte permutes,
// 5 instructions per single-nucleotide id instead of the 35 that one id per
// lane and load took. 4,096 rows of 8,192 bases: single-nucleotide ids 65 ->
// 42 us (168 MB), 6-mers 25 -> 18 us (56 MB), in one launch instead of two.
template <int K, int U>
__global__ __launch_bounds__(NT) void k_decode_fixed(DecodeArgs a, ScanState st) {
    constexpr int NW = NT / dev::kWave;
    constexpr int WT = 256 * U, FT = NW * WT;  // ids of a wave, of the tile
    constexpr int NWORD = (K + 3) / 4;
    extern __shared__ __align__(16) uint8_t s_out[];
    __shared__ uint32_t s_wave[NW];        // non-silent ids of a wave
    __shared__ uint32_t s_pre[NW * U];     // non-silent ids of the wave before a slice
    __shared__ uint64_t s_silent[NW * U][4];
    __shared__ TileRows s_rows;
    __shared__ int64_t s_base;
    const int tid = threadIdx.x, lane = tid & (dev::kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    const int64_t t = blockIdx.x;
    const int64_t P0 = t * FT;
    const int64_t n = a.n;
    uint32_t err = 0;
    if (t >= a.ntiles) {
        check_rest(a, t - a.ntiles);
        return;
    }

    ids4 id[U];
    const int64_t p0 = P0 + w * WT + 4 * lane;
    if (P0 + FT <= a.n_ids) {
#pragma unroll
        for (int s = 0; s < U; ++s) id[s] = __builtin_nontemporal_load(reinterpret_cast<const ids4 *>(a.ids + p0 + 256 * s));
    } else {
#pragma unroll
        for (int s = 0; s < U; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t p = p0 + 256 * s + q;
                id[s][q] = p < a.n_ids ? a.ids[p] : DNATOK_ID_PAD;
            }
    }
    const int64_t first = n > 0 ? a.offs[0] : 0, last = n > 0 ? a.offs[n] : 0;
    const ScanView v = scan_view(st);
    int64_t g0 = 0, po = 0;
    if (w == NW - 1) {
        err |= check_rows(a, t * kCheckRows + lane);
        po = probe_rows(a, P0, &g0);
    }
    if (P0 < first || P0 + FT > last) {  // ids outside the rows decode to nothing
#pragma unroll
        for (int s = 0; s < U; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t p = p0 + 256 * s + q;
                if (p < first || p >= last) id[s][q] = DNATOK_ID_PAD;
            }
    }
    uint32_t mine = 0, pre[U];
    bool gaps[U];
#pragma unroll
    for (int s = 0; s < U; ++s) {
        const uint32_t lowest = min(min((uint32_t)id[s][0], (uint32_t)id[s][1]), min((uint32_t)id[s][2], (uint32_t)id[s][3]));
        gaps[s] = __ballot(lowest < 5u) != 0;  // (an UNK is not silent, but rare)
        pre[s] = mine;
        uint64_t m[4] = {0, 0, 0, 0};
        mine += 256;
        if (gaps[s]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                m[q] = __ballot(is_silent(id[s][q]));
                mine -= (uint32_t)__popcll(m[q]);
            }
        }
        if (lane == 0) {
            s_pre[w * U + s] = pre[s];
#pragma unroll
            for (int q = 0; q < 4; ++q) s_silent[w * U + s][q] = m[q];
        }
    }
    if (lane == 0) s_wave[w] = mine;
    __syncthreads();
    uint32_t before = 0, total = 0;  // of the waves before this one, of the tile
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        before += i < w ? s_wave[i] : 0;
        total += s_wave[i];
    }
    const int64_t agg = (int64_t)K * total;
    publish_tile(st, v, t, a.ntiles, agg);
    if (w == NW - 1) find_rows(a, P0, g0, po, s_rows);
    // the bytes to LDS
#pragma unroll
    for (int s = 0; s < U; ++s) {
        uint8_t *p = s_out + (uint32_t)K * (before + pre[s]);
        if (!gaps[s]) {
            uint32_t out[K];
            if constexpr (K == 1) {
                uint32_t sel = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) sel |= min((uint32_t)id[s][q] - 5u, 4u) << (8 * q);
                out[0] = __builtin_amdgcn_perm(0x4E4E4E4Eu, 0x54474341u, sel);
            } else {
#pragma unroll
                for (int i = 0; i < K; ++i) out[i] = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t x[NWORD];
                    const uint32_t v = (uint32_t)id[s][q] - 5u;
                    letters<K>(v, v < a.codes, x);
#pragma unroll
                    for (int i = 0; i < NWORD; ++i) {
                        const int at = q * K + 4 * i, sh = 8 * (at % 4);
                        const int bytes = i == NWORD - 1 ? K - 4 * i : 4;
                        out[at / 4] |= x[i] << sh;
                        if (sh / 8 + bytes > 4) out[at / 4 + 1] |= x[i] >> (32 - sh);
                    }
                }
            }
            __builtin_memcpy(p + 4 * K * lane, out, 4 * K);
        } else {
            uint32_t below = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t m = ~s_silent[w * U + s][q];
                below += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            }
            p += (uint32_t)K * below;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (is_silent(id[s][q])) continue;
                uint32_t x[NWORD];
                const uint32_t v = (uint32_t)id[s][q] - 5u;
                letters<K>(v, v < a.codes, x);
                __builtin_memcpy(p, x, K);
                p += K;
            }
        }
    }
    if (w == 0) {
        const int64_t sum = tile_position(v, t, agg, a.err_hdr);
        if (lane == 0) s_base = sum;
    }
    __syncthreads();
    const int64_t base = s_base;
    store_stage(a, s_out, base, agg, err);
    // rows starting in the tile: K bytes per non-silent id before their first position
    put_rows(a, s_rows, P0, FT, t == a.ntiles - 1, base, [&](int32_t rel) {
        uint32_t c = total;
        if (rel < FT) {
            const int sl = rel / 256, l = (rel % 256) / 4, q0 = rel % 4;
            c = s_pre[sl] + (uint32_t)(rel % 256);
            for (int i = 0; i < sl / U; ++i) c += s_wave[i];
            for (int q = 0; q < 4; ++q) {
                const uint64_t m = s_silent[sl][q];
                c -= (uint32_t)__popcll(m & ((1ull << l) - 1ull));
                if (q < q0) c -= (uint32_t)(m >> l) & 1u;
            }
        }
        return (int64_t)K * c;
    });
    if (err) dev::raise_error(a.err_hdr, err);
    if (t == a.ntiles - 1 && tid == 0) finish_tiles(a, st, v, base + agg);
}

// The first L (up to 16) bytes of v to p.
__device__ __forceinline__ void put_bytes(uint8_t *p, const u32x4 &v, int32_t L) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int32_t r = L - 4 * w;
        const uint32_t x = v[w];
        if (r >= 4) {
            __builtin_memcpy(p + 4 * w, &x, 4);
        } else if (r > 0) {
            if (r >= 2) __builtin_memcpy(p + 4 * w, &x, 2);
            if (r & 1) p[4 * w + r - 1] = (uint8_t)(x >> (8 * (r - 1)));
        }
    }
}

// BPE ids, TPT consecutive ones per thread: their lengths and the first 16
// bases of each are asked for together (three dependent loads a tile, whatever
// its tokens; a loop of byte loads per token took 0.5 us a byte), then staged.
// A tile whose output exceeds the stage writes its tokens to the output one by
// one. Bound by that chain of loads and the wait for the position: 968,000
// ids (5.5 MB of bases) 30.6 -> 14.8 us, 174,000 28.5 -> 9.7, 184 18.7 -> 7.4;
// a row pass, a chain of prefixes and the byte loops before.
template <int TPT>
__global__ __launch_bounds__(NT) void k_decode_bpe(DecodeArgs a, ScanState st) {
    constexpr int FT = NT * TPT;
    extern __shared__ __align__(16) uint8_t s_out[];
    __shared__ int64_t s_tpre[NT + 1];  // in-tile bytes before each thread's first position (and the total)
    __shared__ int64_t s_tmp[NT / dev::kWave + 1];
    __shared__ TileRows s_rows;
    __shared__ int64_t s_base;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    const int64_t t = blockIdx.x;
    const int64_t P0 = t * FT, p0 = P0 + tid * TPT;
    const int64_t n = a.n;
    uint32_t err = 0;
    if (t >= a.ntiles) {
        check_rest(a, t - a.ntiles);
        return;
    }
    int32_t id[TPT];
    if (P0 + FT <= a.n_ids) {
#pragma unroll
        for (int j = 0; j < TPT; j += 4) {
            const ids4 x = *reinterpret_cast<const ids4 *>(a.ids + p0 + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) id[j + q] = x[q];
        }
    } else {
#pragma unroll
        for (int j = 0; j < TPT; ++j) id[j] = p0 + j < a.n_ids ? a.ids[p0 + j] : DNATOK_ID_PAD;
    }
    const int64_t first = n > 0 ? a.offs[0] : 0, last = n > 0 ? a.offs[n] : 0;
    const ScanView v = scan_view(st);
    int64_t g0 = 0, po = 0;
    if (w == NT / dev::kWave - 1) {
        err |= check_rows(a, t * kCheckRows + (tid & (dev::kWave - 1)));
        po = probe_rows(a, P0, &g0);
    }
    auto merged = [&](int32_t x) { return x >= 10 && x < a.vocab; };
    int32_t len[TPT];
    int64_t off[TPT];
#pragma unroll
    for (int j = 0; j < TPT; ++j) {
        if (p0 + j < first || p0 + j >= last) id[j] = DNATOK_ID_PAD;  // ids outside the rows decode to nothing
        len[j] = is_silent(id[j]) ? 0 : 1;
        off[j] = 0;
        if (merged(id[j])) {
            len[j] = a.tok_len[id[j]];
            off[j] = a.tok_off[id[j]];
        }
    }
    int64_t mine = 0;
#pragma unroll
    for (int j = 0; j < TPT; ++j) mine += len[j];
    int64_t agg;
    const int64_t pre = dev::block_excl_scan<NT>(mine, s_tmp, &agg);
    publish_tile(st, v, t, a.ntiles, agg);
    if (w == NT / dev::kWave - 1) find_rows(a, P0, g0, po, s_rows);
    s_tpre[tid] = pre;
    if (tid == NT - 1) s_tpre[NT] = pre + mine;
    const bool staged = agg <= a.stage;
    if (staged) {
        uint32_t pos = (uint32_t)pre;  // the stage holds at most 32 KiB
#pragma unroll
        for (int j0 = 0; j0 < TPT; j0 += 4) {
            u32x4 x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = u32x4{single_letter(id[j0 + j]), 0, 0, 0};
                if (merged(id[j0 + j])) __builtin_memcpy(&x[j], a.tok_chars + off[j0 + j], 16);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t L = len[j0 + j];
                put_bytes(s_out + pos, x[j], min(L, 16));
                for (int32_t b = 16; b < L; b += 16) {
                    u32x4 y;
                    __builtin_memcpy(&y, a.tok_chars + off[j0 + j] + b, 16);
                    put_bytes(s_out + pos + b, y, min(L - b, 16));
                }
                pos += (uint32_t)L;
            }
        }
    }
    if (w == 0) {
        const int64_t sum = tile_position(v, t, agg, a.err_hdr);
        if (tid == 0) s_base = sum;
    }
    __syncthreads();
    const int64_t base = s_base;
    if (staged) {
        store_stage(a, s_out, base, agg, err);
    } else {
        int64_t pos = base + pre;
#pragma unroll
        for (int j = 0; j < TPT; ++j) {
            write_token(a, id[j], pos, err);
            pos += len[j];
        }
    }
    // a row's bytes before its first position: the owning thread's prefix and
    // its ids before that position (read again from the cache)
    put_rows(a, s_rows, P0, FT, t == a.ntiles - 1, base, [&](int32_t rel) {
        const int th = rel / TPT;
        int64_t sum = s_tpre[th];
        for (int64_t q = P0 + (int64_t)th * TPT; q < P0 + rel; ++q) {
            const bool live = q >= first && q < last && q < a.n_ids;
            sum += width_of(a, live ? a.ids[q] : DNATOK_ID_PAD);
        }
        return sum;
    });
    if (err) dev::raise_error(a.err_hdr, err);
    if (t == a.ntiles - 1 && tid == 0) finish_tiles(a, st, v, base + agg);
}

static_assert(kDecodeWords == kHeadWords + 2 * (kDecodeTiles + kDecodeTiles / 64 + kDecodeTiles / 4096), "the workspace's words");

__global__ void k_clear_words(uint64_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Tiles of tt ids: their count, the scan's state and the launch's grid.
int plan_tiles(DecodeArgs &a, int64_t tt, Workspace *ws, hipStream_t stream, ScanState *st, dim3 *grid) {
    a.ntiles = a.n_ids / tt + 1;
    if (a.ntiles >= (1ll << 31)) return set_error(DNATOK_EINVAL, "too many ids for one decode");
    a.rows_per_id = a.n_ids > 0 ? (double)a.n / (double)a.n_ids : 0.0;
    if (a.ntiles <= kDecodeTiles) {
        int rc = ensure_decode(ws);
        if (rc) return rc;
    }
    *st = scan_state(ws->d_decode, kDecodeTiles);
    if (!ws->d_decode || a.ntiles > kDecodeTiles) {
        const int64_t nw = scan_words(a.ntiles);
        int rc = ensure_scratch(ws, 8 * nw);
        if (rc) return rc;
        *st = scan_state(reinterpret_cast<uint64_t *>(ws->d_scratch), a.ntiles);
        hipLaunchKernelGGL(k_clear_words, dim3((unsigned)std::min<int64_t>((nw + 255) / 256, 1024)), dim3(256), 0, stream,
                           st->head, nw);
        DNATOK_HIP(hipGetLastError());
    }
    const int64_t unchecked = std::max<int64_t>(0, a.n - a.ntiles * kCheckRows);
    *grid = dim3((unsigned)(a.ntiles + (unchecked + kCheckBlock - 1) / kCheckBlock));
    return DNATOK_OK;
}

template <int K>
int launch_fixed(DecodeArgs a, Workspace *ws, hipStream_t stream) {
    // Ids per tile: 1,024 times U. Tiles that do not all fit the card at once
    // wait for a second set of prefixes, 6 us; large tiles leave fewer waves.
    // So the smallest U with at most 7 tiles per CU (single letters 5), up to
    // what a stage of 48 KiB holds. Measured, in us at U = 2 / 4 / 8 / 16:
    // 6.7M 5-mers 24.7 / 18.2 / 23.9 / -, 10M single letters - / 21.9 / 17.4 /
    // 20.4, 3M 11.1 / 10.1 / 10.0 / -, 33.6M 61 / 56 / 43.1 / 40.5.
    constexpr int UMAX = K == 1 ? 16 : K <= 6 ? 8 : K <= 12 ? 4 : 2;
    static_assert(1024 * UMAX * K <= 49152, "three tiles' stages fit a CU");
    int U = 1;
    while (U < UMAX && a.n_ids > 1024 * (int64_t)U * (K == 1 ? 5 : 7) * device_cu_count()) U <<= 1;
    a.codes = 1u << (2 * K);
    ScanState st;
    dim3 grid;
    int rc = plan_tiles(a, 1024 * U, ws, stream, &st, &grid);
    if (rc) return rc;
    const dim3 block(NT);
    const size_t dyn = (size_t)1024 * U * K + 16;  // a unit's realigning reads go up to 3 bytes past the data
    switch (U) {
    case 1: hipLaunchKernelGGL((k_decode_fixed<K, 1>), grid, block, dyn, stream, a, st); break;
    case 2: hipLaunchKernelGGL((k_decode_fixed<K, 2>), grid, block, dyn, stream, a, st); break;
    case 4: if constexpr (UMAX >= 4) hipLaunchKernelGGL((k_decode_fixed<K, 4>), grid, block, dyn, stream, a, st); break;
    case 8: if constexpr (UMAX >= 8) hipLaunchKernelGGL((k_decode_fixed<K, 8>), grid, block, dyn, stream, a, st); break;
    default: if constexpr (UMAX >= 16) hipLaunchKernelGGL((k_decode_fixed<K, 16>), grid, block, dyn, stream, a, st); break;
    }
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

}  // namespace

int launch_decode(const dnatok_vocab *v, const int32_t *d_ids, int64_t n_ids, const int64_t *d_offsets, int32_t n,
                  uint8_t *d_out, int64_t out_capacity, int64_t *d_out_offsets, hipStream_t stream) {
    DecodeArgs a = {};
    a.ids = d_ids;
    a.n_ids = n_ids;
    a.offs = d_offsets;
    a.n = n;
    a.out = d_out;
    a.cap = out_capacity;
    a.out_offs = d_out_offsets;
    a.vocab = v->vocab_size;
    a.tok_len = v->bpe.d_tok_len;
    a.tok_off = v->bpe.d_tok_off;
    a.tok_chars = v->bpe.d_tok_chars;
    Workspace *ws = nullptr;
    int rc = get_workspace(stream, 1, &ws);
    if (rc) return rc;
    a.err_hdr = ws->d_hdr;
    if (v->kind != DNATOK_BPE) {
        switch (v->kind == DNATOK_KMER ? v->k : 1) {
        case 1: return launch_fixed<1>(a, ws, stream);
        case 2: return launch_fixed<2>(a, ws, stream);
        case 3: return launch_fixed<3>(a, ws, stream);
        case 4: return launch_fixed<4>(a, ws, stream);
        case 5: return launch_fixed<5>(a, ws, stream);
        case 6: return launch_fixed<6>(a, ws, stream);
        case 7: return launch_fixed<7>(a, ws, stream);
        case 8: return launch_fixed<8>(a, ws, stream);
        case 9: return launch_fixed<9>(a, ws, stream);
        case 10: return launch_fixed<10>(a, ws, stream);
        case 11: return launch_fixed<11>(a, ws, stream);
        case 12: return launch_fixed<12>(a, ws, stream);
        case 13: return launch_fixed<13>(a, ws, stream);
        case 14: return launch_fixed<14>(a, ws, stream);
        default: return launch_fixed<15>(a, ws, stream);
        }
    }
    // the stage holds a tile's output at the vocabulary's widest token. Tiles
    // of 1,024 ids while all of them fit the card at once, else of 4,096.
    const bool small = n_ids <= 1024 * 7 * (int64_t)device_cu_count();
    const int64_t tt = small ? 1024 : 4096;
    a.stage = (int32_t)std::min<int64_t>(tt * std::max<int64_t>(v->max_token_bytes, 1), kMaxStage);
    ScanState st;
    dim3 grid;
    rc = plan_tiles(a, tt, ws, stream, &st, &grid);
    if (rc) return rc;
    const size_t dyn = (size_t)a.stage + 16;  // a unit's realigning reads go up to 3 bytes past the data
    if (small) hipLaunchKernelGGL(k_decode_bpe<4>, grid, dim3(NT), dyn, stream, a, st);
    else hipLaunchKernelGGL(k_decode_bpe<16>, grid, dim3(NT), dyn, stream, a, st);
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

}  // namespace dnatok
