// Byte -> identifier encode by wave tiles (SINGLE, LUT256, KMER; PACKED and
// PADDED; reverse complement and overlapping windows; several k-mer
// vocabularies in one pass).
//
// Paper: Design, "Encoding paths", bytes path (a device-resident 256-entry
// LUT applied to staged ASCII) and the bytes branch of the EmbedFromStrings
// algorithm (MapKmer for k-mer vocabularies, left padding to token_len);
// Discussion (reverse complementation as the augmentation to run on the
// GPU); Introduction (overlapping k-mers of stride 1, L - k + 1 tokens).
//
// The concatenated input is cut into tiles of U KiB from its 16-byte-aligned
// base, and every tile belongs to one wavefront: it reads the tile's bytes
// (16 bytes a lane, U times) and the rows' offsets together, stages the bytes
// in its own LDS, and writes every output cell it owns. No barrier and no
// other wave is involved, so the fixed chain of a tile is three loads long
// (row probe and bytes, the rows' offsets, a table) and up to eight waves per
// SIMD hide each other's. A workgroup-wide tile or row band has the same
// chain with four to six barriers in it, 10 to 15 us per workgroup whatever
// its work, measured.
//
// Ownership. A token belongs to the tile that holds its first byte in the
// input; the cells before the first token (pads on the left, CLS) and after
// the last one (SEP, pads on the right) to the tiles that hold the row's
// first and last byte (reverse complement: last and first). A tile therefore
// owns one contiguous run of cells per row it touches. Its wave takes the
// first 64 of those rows; further waves, one per 64 rows of the batch, look
// whether their rows come later than that in some tile (empty rows and rows
// of a few bases) and write them from a stage of their own: one wave going
// through a tile of 20,000 empty rows took 650 us, this way 20.
//
// Writing. Per vocabulary each lane works out one row's run.
// Long runs are written row by row: the run's facts are uniform across the
// wave, and a 16-byte group of four full frames costs one 32-base window
// read. Short runs (reads) are written all together: every lane takes one
// 16-byte group and looks its row up in LDS.
#include <type_traits>

#include "common.hpp"
#include "device.hpp"
#include "rowscan.hpp"

namespace dnatok {

namespace {

constexpr int NTR = 256;               // threads: four independent waves
constexpr int kRowWaves = NTR / 64;
constexpr int kRowVocabs = 8;
constexpr int32_t kSelfScanRows = 2 * NTR;  // PACKED, one vocabulary: each workgroup scans the rows itself
// Pads of a row belong to the tile of its last byte (on the left: first), and
// one wave writes about 4,400 cells a microsecond. Above this row width, or
// when most of the matrix is pads, waves of their own write them, up to
// kPadCells cells each: 64 rows of 50 bases padded to 10^6 take 52 us, written by
// their tiles 4,774; 300 of 100 padded to 30,000 11 and 89. Narrow rows
// keep them: they share most 16-byte groups with tokens.
constexpr int64_t kPadsApartWidth = 1024;
constexpr int32_t kPadCells = 32768;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

struct RowsVocab {
    int32_t k;
    uint32_t kinv;
    int32_t al;  // element misalignment of ids within 16 bytes
    int32_t pad_id, cls_id, sep_id;
    int32_t *ids;
    int8_t *mask;
    int64_t cap;
    int64_t *out_offs;
    int64_t W;
    int64_t base;
    // pads_apart: this vocabulary's first unit; rows of a unit, or (1) the
    // parts of a row
    int32_t pad_first, pad_rows, pad_parts;
};

struct RowsArgs {
    const uint8_t *abase;  // input base aligned down to 16 bytes
    int64_t shift;         // d_bytes - abase
    int64_t nbytes;
    const int64_t *offs;
    int32_t n;
    int32_t nv;
    int32_t cls, padded, left;
    int32_t overlap, revcomp;
    int64_t ntiles;
    // workgroups before the tiles: row scans (nv * scan_units of them), pads,
    // rows past the first 64 of a tile, then idle
    int32_t pads, lead;
    int32_t scan_units;
    int32_t self_scan;  // PACKED: each workgroup scans the row lengths itself
    uint32_t wave_lds;  // dynamic LDS bytes of a wave
    int32_t wide;       // PADDED: a row width past 28 bits
    int32_t pads_apart; // PADDED: the pads are written by workgroups before the tiles
    int32_t pad_units;  // of all vocabularies
    int32_t pad_cells;  // cells of a unit
    double rows_per_byte;
    const int32_t *lut;
    uint32_t *err_hdr;
    RowsVocab vo[kRowVocabs];
};

// A row's run of cells in a tile, cells counted from the run's first.
struct Run {
    int64_t dlo;        // element of cell 0
    int32_t ncell;      // cells
    int32_t f0, f1;     // full frames
    int32_t tail;       // the short final frame (UNK), -1: none
    int32_t ccls, csep; // CLS and SEP, -1: none
    uint32_t idx;       // staged byte (mod 2^32) of cell 0's token
    // long runs: groups before the first of four full frames, such groups;
    // the first group of four pads, such groups
    int32_t before, nfast, pad0, npad;
};
// Average 16-byte groups of a run from which runs are written row by row. A
// row costs about 100 instructions however few groups it has, a group written
// among those of all rows about 6 (350 for 64 of them); both measured alike
// at 20 groups a run.
constexpr uint32_t kLongRun = 20;

// Digits of the k-mer at staged byte idx (win64[m] holds the digits of
// 16-base chunks m and m + 1, first base on top, val32[m] their validity):
// -1 if a byte is not A/C/G/T.
__device__ __forceinline__ int32_t one_kmer(const uint64_t *win64, const uint32_t *val32, uint32_t idx, int32_t k) {
    const uint32_t w = idx >> 4, o = idx & 15u;
    const uint32_t digits = (uint32_t)(win64[w] >> (64 - 2 * (o + (uint32_t)k))) & ((1u << (2 * k)) - 1u);
    const uint32_t km = (1u << k) - 1u;
    return ((val32[w] >> (32 - o - (uint32_t)k)) & km) == km ? (int32_t)digits : -1;
}

// The k 2-bit digits of v in reverse order, complemented.
__device__ __forceinline__ uint32_t rc_digits(uint32_t v, int32_t k) {
    uint32_t r = __builtin_bitreverse32(v);
    r = ((r >> 1) & 0x55555555u) | ((r & 0x55555555u) << 1);
    return (r >> (32 - 2 * k)) ^ ((1u << (2 * k)) - 1u);
}

// Four ids from the 32 staged bases from byte idx0 on: id q is the k-mer at
// base p0 + q * dp of that window (all inside it).
__device__ __forceinline__ i32x4 four_kmers(const uint64_t *win64, const uint32_t *val32, uint32_t idx0, int32_t k,
                                            int32_t p0, int32_t dp, bool rc) {
    const uint32_t w = idx0 >> 4, o = idx0 & 15u;
    const uint64_t w0 = win64[w], w1 = win64[w + 1];
    const uint32_t v0 = val32[w], v1 = val32[w + 1];
    const uint64_t X = (w0 << (2 * o)) | (((uint64_t)(uint32_t)w1 << (2 * o)) >> 32);
    const uint32_t nV = ~(uint32_t)((((uint64_t)v0 << 32) | (uint64_t)(v1 << 16)) << o >> 32);
    const uint32_t dm = (1u << (2 * k)) - 1u, km = (1u << k) - 1u;
    i32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int32_t p = p0 + q * dp;
        const uint32_t fv = (uint32_t)(X >> (64 - 2 * (p + k))) & dm;
        const bool bad = ((nV >> (32 - p - k)) & km) != 0;
        r[q] = bad ? DNATOK_ID_UNK : 5 + (int32_t)(rc ? rc_digits(fv, k) : fv);
    }
    return r;
}

__device__ __forceinline__ uint32_t complement_of(uint32_t b) {
    switch (b) {
    case 'A': return 'T';
    case 'T': return 'A';
    case 'C': return 'G';
    case 'G': return 'C';
    case 'a': return 't';
    case 't': return 'a';
    case 'c': return 'g';
    case 'g': return 'c';
    default: return b;
    }
}

__device__ __forceinline__ int32_t uni(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ int64_t uni64(int64_t v, int lane) {
    return (int64_t)(((uint64_t)(uint32_t)uni((int32_t)(v >> 32), lane) << 32) | (uint32_t)uni((int32_t)v, lane));
}

// LDS of a tile's staged bytes, and of a wave's 64 runs with their first
// groups.
template <bool KMER>
__host__ __device__ constexpr uint32_t stage_bytes(uint32_t chunks) {
    return KMER ? ((chunks + 2u) * 12u + 15u) / 16u * 16u : (chunks + 2u) * 16u;
}
constexpr uint32_t kRunBytes = 64 * sizeof(Run) + 64 * 4;

// One wave's share of the pads: pad_rows rows of a vocabulary, or pad_cells
// cells of one.
template <bool KMER>
__device__ __forceinline__ void write_pads(const RowsArgs &a, int unit, int lane) {
    int vi = 0;
    while (vi + 1 < a.nv && unit >= a.vo[vi + 1].pad_first) ++vi;
    const RowsVocab &o = a.vo[vi];
    unit -= o.pad_first;
    const int64_t r0 = o.pad_parts > 1 ? unit / o.pad_parts : (int64_t)unit * o.pad_rows;
    const int64_t part0 = o.pad_parts > 1 ? (int64_t)(unit % o.pad_parts) * a.pad_cells : 0;
    const int64_t part1 = o.pad_parts > 1 ? min(part0 + a.pad_cells, o.W) : o.W;
    const RowLen rl{a.offs, a.nbytes, a.n, KMER ? o.k : 1, o.kinv, KMER ? 1 : 0, a.overlap, a.cls, o.W};
    int64_t first = 0, cells = 0;
    if (lane < o.pad_rows && r0 + lane < a.n) {
        uint32_t over = 0;  // (the row scan raises it)
        const int64_t len = rl.len(r0 + lane, over);
        const int64_t p0 = max(a.left ? 0 : len, part0), p1 = min(a.left ? o.W - len : o.W, part1);
        if (len <= o.W && p1 > p0) {
            first = (r0 + lane) * o.W + p0;
            cells = p1 - p0;
        }
    }
    const i32x4 y{o.pad_id, o.pad_id, o.pad_id, o.pad_id};
    for (uint64_t w = __ballot(cells > 0); w; w &= w - 1) {
        const int l = __builtin_ctzll(w);
        const int64_t e = uni64(first, l);
        const int32_t nc = uni((int32_t)cells, l), m = (int32_t)((uint32_t)(e + o.al) & 3u);
        int32_t *ids = o.ids + (e - m);
        int8_t *mask = o.mask + (e - m);
        const bool mask4 = (reinterpret_cast<uintptr_t>(mask) & 3) == 0;
        for (int32_t g = lane; g * 4 < m + nc; g += dev::kWave) {
            if (4 * g >= m && 4 * g + 4 <= m + nc) {
                __builtin_nontemporal_store(y, reinterpret_cast<i32x4 *>(ids) + g);
                if (mask4) {
                    *reinterpret_cast<uint32_t *>(mask + 4 * g) = 0u;
                    continue;
                }
            }
#pragma unroll
            for (int32_t c = 4 * g; c < 4 * g + 4; ++c) {
                if (c >= m && c < m + nc) {
                    ids[c] = o.pad_id;
                    mask[c] = 0;
                }
            }
        }
    }
}

// What a launch writes: one vocabulary forward in frames; one vocabulary
// reverse complemented or in overlapping windows; several vocabularies; as the
// second, a tile's waves all staging it and writing a quarter of its groups each.
enum RowsMode { ROWS_PLAIN = 0, ROWS_VARIANT = 1, ROWS_MULTI = 2, ROWS_SHARED = 3 };

// ROWS_MULTI: a tile of four times the bytes belongs to the workgroup, whose
// waves stage a quarter each and, after one barrier, write one vocabulary
// each (a wave writing four vocabularies of its own tile in turn took 24.5 us
// on 142 rows of 8.6 to 16 kbases for k = 2..5, this 11.7).
template <bool KMER, int U, bool PADDED, RowsMode MODE>
__global__ __launch_bounds__(NTR) void k_rows(RowsArgs a) {
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ int64_t s_tmp[kRowWaves + 1];
    __shared__ int32_t s_lut[KMER ? 1 : 256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = (int)blockIdx.x - (PADDED ? a.nv * a.scan_units : 0);
    if (PADDED && b < 0) {
        const int vi = (int)blockIdx.x / a.scan_units, unit = (int)blockIdx.x - vi * a.scan_units;
        const RowsVocab &o = a.vo[vi];
        rowscan_independent(RowLen{a.offs, a.nbytes, a.n, KMER ? o.k : 1, o.kinv, KMER ? 1 : 0, a.overlap, a.cls, o.W},
                            o.out_offs, o.base, unit, s_tmp, a.err_hdr);
        return;
    }
    if (PADDED && b < a.pads) {
        const int unit = b * kRowWaves + wave;
        if (unit < a.pad_units) write_pads<KMER>(a, unit, lane);
        return;
    }
    constexpr bool MULTI = MODE == ROWS_MULTI, PLAIN = MODE == ROWS_PLAIN;
    const bool extra = (int)blockIdx.x < a.lead;
    int64_t tile = extra ? (PADDED ? b - a.pads : b) : (int64_t)blockIdx.x - a.lead;
    constexpr bool shared = MODE == ROWS_SHARED, VARIANT = MODE == ROWS_VARIANT || shared;
    if (!MULTI && !shared) tile = tile * kRowWaves + wave;
    const bool rc = VARIANT && a.revcomp != 0, overlap = VARIANT && a.overlap != 0;
    constexpr int64_t T = 1024 * U * (MULTI ? kRowWaves : 1);
    constexpr uint32_t nch = (uint32_t)(T / 16);
    uint8_t *lds = MULTI ? dyn : dyn + (size_t)wave * a.wave_lds;
    // this wave's vocabularies are v0, v0 + vstep, ...; of each it writes the
    // groups l0, l0 + lstep, ... (two vocabularies: two waves each)
    const int share = MULTI && a.nv == 2 ? 2 : 1;
    const int v0 = MULTI ? wave / share : 0, vstep = MULTI ? kRowWaves / share : 1;
    const int32_t nv = MULTI ? a.nv : 1;
    const int32_t l0 = lane + (MULTI ? 64 * (wave % share) : shared ? 64 * wave : 0);
    const int32_t lstep = shared ? 64 * kRowWaves : 64 * share;
    const uint32_t m0 = MULTI ? (uint32_t)wave * 64u * U : 0u;  // first chunk this wave stages
    uint64_t *win64 = reinterpret_cast<uint64_t *>(lds);
    uint32_t *val32 = reinterpret_cast<uint32_t *>(win64 + nch + 2);
    uint8_t *raw = lds;
    Run *runs = reinterpret_cast<Run *>(
        MULTI ? dyn + stage_bytes<KMER>(nch) + (size_t)wave * kRunBytes : lds + stage_bytes<KMER>(nch));
    uint32_t *first_group = reinterpret_cast<uint32_t *>(runs + 64);
    int64_t *s_prefix = reinterpret_cast<int64_t *>(dyn + (size_t)kRowWaves * a.wave_lds);  // self_scan
    const int64_t n = a.n;
    int64_t i = 0, o0 = 0, o1 = 0;  // a row per lane
    bool live = tile < a.ntiles, mine = false;
    int64_t before0 = 0, before1 = 0;
    if (extra) {
        // the 64 rows from 64 * (tile + 1) on, if the tile that the first of
        // them starts in has 64 rows before them
        i = 64 * (tile + 1) + lane;
        live = 64 * (tile + 1) < n;
        tile = 0;
        if (live) {
            o0 = a.offs[min(i, n)];
            o1 = a.offs[min(i + 1, n)];
            before0 = a.offs[min(i, n) - 64];
            before1 = a.offs[min(i, n) - 63];
            tile = min((min(max(uni64(o0, 0), (int64_t)0), a.nbytes) + a.shift) / T, a.ntiles - 1);
        }
    }
    const int64_t q0 = tile * T;               // tile in abase bytes
    const int64_t P0 = q0 - a.shift;           // in input bytes
    const int64_t P1 = tile >= a.ntiles - 1 ? INT64_MAX : P0 + T;
    // a row's last byte (or, empty, its place) lies at P0 or beyond
    auto reaches = [&](int64_t r0, int64_t r1) { return (r1 > r0 ? r1 - 1 : r0) >= P0; };
    if (extra) {
        mine = live && i < n && o0 < P1 && reaches(before0, before1);
        live = __ballot(mine) != 0;
    }

    // everything that can be asked for at once: the tile's bytes, 64 rows'
    // offsets around the row the tile would start in if rows were equally
    // long, the byte table
    uint4 v[U], halo = make_uint4(0, 0, 0, 0);
    const bool whole = q0 >= a.shift && q0 + T + 16 <= a.shift + a.nbytes;
    if (live && whole) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(a.abase + q0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u32x4 x = __builtin_nontemporal_load(src + m0 + u * 64 + lane);
            v[u] = make_uint4(x[0], x[1], x[2], x[3]);
        }
        const u32x4 x = src[nch];
        halo = make_uint4(x[0], x[1], x[2], x[3]);
    } else if (live) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = dev::load16(a.abase, q0 + 16 * (int64_t)(m0 + u * 64 + lane), a.shift, a.shift + a.nbytes);
        halo = dev::load16(a.abase, q0 + T, a.shift, a.shift + a.nbytes);
    }
    int64_t g0 = (int64_t)((double)(P0 > 0 ? P0 : 0) * a.rows_per_byte) - 32;
    if (g0 + 64 > n) g0 = n - 64;
    if (g0 < 0) g0 = 0;
    int64_t po0 = 0, po1 = 0;
    if (n > 0 && !extra) {
        po0 = a.offs[min(g0 + lane, n)];
        po1 = a.offs[min(g0 + lane + 1, n)];
    }
    if constexpr (!KMER) {
        s_lut[tid] = a.lut[a.revcomp ? complement_of((uint32_t)tid) : (uint32_t)tid];
    }
    uint32_t err = 0;
    if (PLAIN && !PADDED && a.self_scan) {
        // two rows per thread; the first workgroup also writes the offsets
        const RowLen rl{a.offs, a.nbytes, a.n, KMER ? a.vo[0].k : 1, a.vo[0].kinv, KMER ? 1 : 0, 0, a.cls, INT64_MAX};
        const bool first = (int)blockIdx.x == a.lead;
        uint32_t e2 = 0;
        const int64_t l0 = 2 * tid < n ? rl.len(2 * (int64_t)tid, e2) : 0;
        const int64_t l1 = 2 * tid + 1 < n ? rl.len(2 * (int64_t)tid + 1, e2) : 0;
        int64_t total;
        const int64_t run = dev::block_excl_scan<NTR>(l0 + l1, s_tmp, &total);
        if (2 * tid < n) s_prefix[2 * tid] = run;
        if (2 * tid + 1 < n) s_prefix[2 * tid + 1] = run + l0;
        if (first) {
            if (2 * tid < n) a.vo[0].out_offs[2 * tid] = a.vo[0].base + run;
            if (2 * tid + 1 < n) a.vo[0].out_offs[2 * tid + 1] = a.vo[0].base + run + l0;
            if (tid == 0) a.vo[0].out_offs[n] = a.vo[0].base + total;
            err |= e2;
        }
    }
    if (!KMER || (PLAIN && !PADDED && a.self_scan)) __syncthreads();
    if (!live) {
        if (err) dev::raise_error(a.err_hdr, err);
        return;
    }

    // stage the tile and the 16 bytes after it
    auto stage = [&](uint32_t m, uint4 x) {
        if constexpr (KMER) {
            uint32_t c, vb;
            dev::classify16(x, c, vb);
            uint32_t *w32 = reinterpret_cast<uint32_t *>(win64);
            uint16_t *v16 = reinterpret_cast<uint16_t *>(val32);
            w32[2 * m + 1] = c;
            v16[2 * m + 1] = (uint16_t)(vb >> 16);
            if (m > 0) {
                w32[2 * m - 2] = c;
                v16[2 * m - 2] = (uint16_t)(vb >> 16);
            }
        } else {
            reinterpret_cast<uint4 *>(raw)[m] = x;
        }
    };
    if (!extra) {
        // 64 rows from the first that reaches into the tile
        int64_t ia;
        auto pred = [&](int64_t r) { return reaches(a.offs[r], a.offs[r + 1]); };
        const uint64_t hit = __ballot(g0 + lane < n ? reaches(po0, po1) : true);
        if ((hit & 1ull) && g0 > 0) ia = dev::wave_lower_bound(0, g0, pred);
        else if (hit == 0) ia = dev::wave_lower_bound(g0 + 64, n, pred);
        else ia = g0 + __builtin_ctzll(hit);
        if (ia > n) ia = n;
        i = ia + lane;
        if (ia >= g0 && uni64(po0, 63) >= P1) {
            // all of the tile's rows were probed
            const int src = (int)(ia - g0) + lane;
            o0 = __shfl((long long)po0, src & 63, 64);
            o1 = __shfl((long long)po1, src & 63, 64);
            mine = src < 64 && i < n && o0 < P1;
        } else {
            o0 = a.offs[min(i, n)];
            o1 = a.offs[min(i + 1, n)];
            mine = i < n && o0 < P1;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) stage(m0 + (uint32_t)(u * 64 + lane), v[u]);
    if (lane == 0 && (!MULTI || wave == 0)) stage(nch, halo);
    if (MULTI) __syncthreads();
    else dev::wave_sync();

    if (__ballot(mine) != 0) {
        o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
        o1 = o1 < o0 ? o0 : (o1 > a.nbytes ? a.nbytes : o1);
        const int64_t L = o1 - o0;
        // 32-bit arithmetic unless a row is longer than it holds
        const bool small = __ballot(mine && L >= (1 << 28)) == 0 && !a.wide;
        for (int vi = v0; vi < nv; vi += vstep) {
            const RowsVocab &o = a.vo[vi];
            const int32_t k = KMER ? o.k : 1;
            const int32_t st = (KMER && !overlap) ? k : 1;        // bytes between tokens
            const uint32_t inv = (KMER && !overlap) ? o.kinv : 0xFFFFFFFFu;
            const int32_t step = rc ? -st : st;
            int64_t out1 = 0;  // PACKED: the row's first token
            if (!PADDED && mine) out1 = PLAIN && a.self_scan ? s_prefix[i] : o.out_offs[i] - o.base;
            Run run{};  // no cells: nothing of it is written
            auto facts = [&](auto zero) {
                using I = decltype(zero);  // int32_t or int64_t
                auto quot = [&](I x, int32_t d, uint32_t dinv) -> I {  // x >= 0
                    if constexpr (sizeof(I) == 4) {
                        uint32_t q = __umulhi((uint32_t)x, dinv);
                        if ((uint32_t)x - q * (uint32_t)d >= (uint32_t)d) ++q;
                        return (I)q;
                    } else {
                        return (I)div_k(x, d, dinv);
                    }
                };
                const I len_b = (I)L, start = (I)max(o0 - P0, -(int64_t)L);  // row start from the tile's
                const I tile_end = P1 == INT64_MAX ? (I)(len_b + (I)T) : (I)T;
                const I place = start + (len_b > 0 ? len_b - 1 : 0);        // the row's last byte
                const bool has_first = start >= 0 && (P1 == INT64_MAX || start < tile_end);
                const bool has_last = place >= 0 && (P1 == INT64_MAX || place < tile_end);
                const I b0 = max(-start, (I)0);                             // the row's bytes in the tile
                const I b1 = P1 == INT64_MAX ? len_b : min((I)(tile_end - start), len_b);
                I nb = len_b;
                if (KMER) nb = overlap ? (len_b >= k ? len_b - k + 1 : (len_b > 0 ? 1 : 0)) : quot(len_b + k - 1, k, o.kinv);
                const I len = nb + 2 * a.cls, width = PADDED ? (I)o.W : len;
                // full frames (all tokens but a short final one)
                const bool tail = KMER && (overlap ? (len_b > 0 && len_b < k) : nb * k != len_b);
                const I nf = nb - (tail ? 1 : 0);
                const I lead = PADDED && a.left ? width - len : 0, bA = lead + a.cls;
                // tokens whose first byte lies in the tile
                I j0, j1;
                if (!rc) {
                    j0 = min(quot(b0 + st - 1, st, inv), nb);
                    j1 = min(quot(max(b1, (I)0) + st - 1, st, inv), nb);
                } else {
                    const I x0 = len_b - k - b1, x1 = len_b - k - b0;
                    j0 = x0 >= 0 ? min((I)(quot(x0, st, inv) + 1), nf) : 0;
                    j1 = x1 >= 0 ? min((I)(quot(x1, st, inv) + 1), nf) : 0;
                }
                const bool head = rc ? has_last : has_first, foot = rc ? has_first : has_last;
                I clo = head ? 0 : bA + j0, chi = foot ? width : bA + max(j1, j0);
                if (PADDED && a.pads_apart) {
                    if (head) clo = lead;
                    if (foot) chi = lead + len;
                }
                if (mine && !(PADDED && len > width) && chi > clo) {
                    const I nc = chi - clo;
                    auto within = [&](I x) { return (int32_t)(x < 0 ? 0 : (x > nc ? nc : x)); };
                    auto cell_or_none = [&](I x) { return x >= 0 && x < nc ? (int32_t)x : -1; };
                    run.ncell = (int32_t)nc;
                    run.f0 = within(bA - clo);
                    run.f1 = within(bA + nf - clo);
                    run.tail = tail ? cell_or_none(bA + nb - 1 - clo) : -1;
                    run.ccls = a.cls ? cell_or_none(lead - clo) : -1;
                    run.csep = a.cls ? cell_or_none(lead + len - 1 - clo) : -1;
                    const I j = clo - bA;  // token at cell 0
                    run.idx = (uint32_t)(o0 - P0) + (uint32_t)(rc ? len_b - k - j * st : j * st);
                    run.dlo = (PADDED ? i * o.W : out1) + clo;
                }
            };
            if (small) facts((int32_t)0);
            else facts((int64_t)0);
            const int32_t al = o.al;
            const bool mask4 = ((reinterpret_cast<uintptr_t>(o.mask) - (uintptr_t)al) & 3) == 0;
            const bool window = !KMER || 3 * st + k <= 32;
            // four cells from c0 on (c0 may lie before the run): ids and mask bytes of those inside
            auto put_group = [&](const Run &r, int32_t c0) {
                int32_t id[4];
                uint32_t mk = 0;
                bool in[4], all_in = true;
                int32_t *dst = o.ids + (r.dlo + c0);
                const int64_t room = PADDED ? INT64_MAX : o.cap - r.dlo;
                if (window && c0 >= r.f0 && c0 + 4 <= r.f1 && c0 + 4 <= room) {
                    i32x4 y;
                    if constexpr (KMER) {
                        const uint32_t at = r.idx + (uint32_t)((rc ? c0 + 3 : c0) * step);
                        y = four_kmers(win64, val32, at, k, rc ? 3 * st : 0, step, rc);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) y[q] = s_lut[raw[r.idx + (uint32_t)((c0 + q) * step)]];
                    }
                    __builtin_nontemporal_store(y, reinterpret_cast<i32x4 *>(dst));
                    if (PADDED) {
                        int8_t *md = o.mask + (r.dlo + c0);
                        if (mask4) *reinterpret_cast<uint32_t *>(md) = 0x01010101u;
                        else
                            for (int q = 0; q < 4; ++q) md[q] = 1;
                    }
                    return;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int32_t c = c0 + q;
                    in[q] = c >= 0 && c < r.ncell;
                    if (in[q] && c >= room) {
                        in[q] = false;
                        err |= DNATOK_DERR_CAPACITY;
                    }
                    all_in = all_in && in[q];
                    int32_t x = o.pad_id;
                    uint32_t m = 1;
                    if (in[q] && c >= r.f0 && c < r.f1) {
                        const uint32_t at = r.idx + (uint32_t)(c * step);
                        if constexpr (KMER) {
                            const int32_t d = one_kmer(win64, val32, at, k);
                            x = d < 0 ? DNATOK_ID_UNK : 5 + (rc ? (int32_t)rc_digits((uint32_t)d, k) : d);
                        } else {
                            x = s_lut[raw[at]];
                        }
                    } else if (c == r.tail) {
                        x = DNATOK_ID_UNK;
                    } else if (c == r.ccls) {
                        x = o.cls_id;
                    } else if (c == r.csep) {
                        x = o.sep_id;
                    } else {
                        m = 0;
                    }
                    id[q] = x;
                    mk |= m << (8 * q);
                }
                if (all_in) {
                    __builtin_nontemporal_store(i32x4{id[0], id[1], id[2], id[3]}, reinterpret_cast<i32x4 *>(dst));
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (in[q]) dst[q] = id[q];
                }
                if (PADDED) {
                    int8_t *md = o.mask + (r.dlo + c0);
                    if (all_in && mask4) {
                        *reinterpret_cast<uint32_t *>(md) = mk;
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (in[q]) md[q] = (int8_t)((mk >> (8 * q)) & 1u);
                    }
                }
            };
            const uint64_t with = __ballot(run.ncell > 0);
            if (with == 0) continue;
            // aligned groups of four that the run touches
            const int32_t m = run.ncell > 0 ? (int32_t)((uint32_t)(run.dlo + al) & 3u) : 0;
            const int32_t ngroups = run.ncell > 0 ? (m + run.ncell + 3) >> 2 : 0;
            const uint32_t nrows = (uint32_t)__popcll(with);
            const uint32_t all = dev::wave_read_u32(dev::wave_incl_sum_u32((uint32_t)ngroups), 63);
            run.before = run.nfast = run.pad0 = run.npad = 0;
            if (all >= (shared ? kRowWaves : 1) * kLongRun * nrows) {
                // groups of four full frames, and of four pads
                const int32_t fhi = PADDED ? run.f1 : (int32_t)min((int64_t)run.f1, max(o.cap - run.dlo, (int64_t)0));
                const int32_t cA = run.f0 + ((4 - ((m + run.f0) & 3)) & 3);
                run.nfast = run.ncell > 0 && window && fhi > cA ? (fhi - cA) >> 2 : 0;
                run.before = run.nfast > 0 ? (m + cA) >> 2 : 0;
                if (PADDED) {
                    const bool frames = run.f1 > run.f0;
                    if (a.left) {
                        const uint32_t f = min(min((uint32_t)run.ccls, (uint32_t)run.csep),
                                               min((uint32_t)run.tail, frames ? (uint32_t)run.f0 : ~0u));
                        run.pad0 = (m + 3) >> 2;
                        run.npad = ((m + (int32_t)min(f, (uint32_t)run.ncell)) >> 2) - run.pad0;
                    } else {
                        const int32_t e = max(max(run.ccls, run.csep), max(run.tail, frames ? run.f1 - 1 : -1)) + 1;
                        run.pad0 = (m + e + 3) >> 2;
                        run.npad = ((m + run.ncell) >> 2) - run.pad0;
                    }
                    run.npad = run.ncell > 0 ? max(run.npad, 0) : 0;
                }
                const uint64_t wide_runs = __ballot(run.nfast + run.npad > 0);
                for (uint64_t w = wide_runs; w; w &= w - 1) {
                    const int l = __builtin_ctzll(w);
                    const int64_t e0 = uni64(run.dlo, l) - uni(m, l);  // element of group 0
                    const int32_t nfast = uni(run.nfast, l), first = uni(run.before, l), npad = uni(run.npad, l);
                    const int32_t c0 = 4 * first - uni(m, l);          // cell of the first fast group
                    const uint32_t idx = (uint32_t)uni((int32_t)run.idx, l);
                    i32x4 *ids4 = reinterpret_cast<i32x4 *>(o.ids + e0) + first;
                    int8_t *mask0 = o.mask + e0 + 4 * first;
                    auto fast = [&](auto four) {
                        for (int32_t t = l0; t < nfast; t += lstep) {
                            const i32x4 y = four(t);
                            __builtin_nontemporal_store(y, ids4 + t);
                            if (PADDED) {
                                // through the cache: a wave's mask words fill lines only together
                                if (mask4) *reinterpret_cast<uint32_t *>(mask0 + 4 * t) = 0x01010101u;
                                else
                                    for (int q = 0; q < 4; ++q) mask0[4 * t + q] = 1;
                            }
                        }
                    };
                    if constexpr (KMER) {
                        // k = 3..6 fixed at compile time: constant shifts and masks
                        auto plain = [&](auto kc) {
                            constexpr int K = decltype(kc)::value;
                            fast([&](int32_t t) {
                                return four_kmers(win64, val32, idx + (uint32_t)((c0 + 4 * t) * K), K, 0, K, false);
                            });
                        };
                        if (rc || overlap || k < 3 || k > 6) {
                            fast([&](int32_t t) {
                                const int32_t c = c0 + 4 * t;
                                return four_kmers(win64, val32, idx + (uint32_t)((rc ? c + 3 : c) * step), k,
                                                  rc ? 3 * st : 0, step, rc);
                            });
                        } else if (k == 3) {
                            plain(std::integral_constant<int, 3>{});
                        } else if (k == 4) {
                            plain(std::integral_constant<int, 4>{});
                        } else if (k == 5) {
                            plain(std::integral_constant<int, 5>{});
                        } else {
                            plain(std::integral_constant<int, 6>{});
                        }
                    } else {
                        const uint32_t *raw32 = reinterpret_cast<const uint32_t *>(raw);
                        fast([&](int32_t t) {
                            const int32_t c = c0 + 4 * t;
                            const uint32_t at = idx + (uint32_t)((rc ? c + 3 : c) * step);
                            const uint32_t b = __builtin_amdgcn_alignbyte(raw32[(at >> 2) + 1], raw32[at >> 2], at & 3u);
                            i32x4 y;
#pragma unroll
                            for (int q = 0; q < 4; ++q) y[q] = s_lut[(b >> (8 * (rc ? 3 - q : q))) & 0xFFu];
                            return y;
                        });
                    }
                    if (PADDED && npad > 0) {
                        const int32_t pad0 = uni(run.pad0, l);
                        const i32x4 y{o.pad_id, o.pad_id, o.pad_id, o.pad_id};
                        i32x4 *p4 = reinterpret_cast<i32x4 *>(o.ids + e0) + pad0;
                        int8_t *md = o.mask + e0 + 4 * pad0;
                        for (int32_t t = l0; t < npad; t += lstep) {
                            __builtin_nontemporal_store(y, p4 + t);
                            if (mask4) *reinterpret_cast<uint32_t *>(md + 4 * t) = 0u;
                            else
                                for (int q = 0; q < 4; ++q) md[4 * t + q] = 0;
                        }
                    }
                }
            }
            // the groups left (edges; all groups of short runs), whatever their row
            const uint32_t rest = (uint32_t)(ngroups - run.nfast - run.npad);
            const uint32_t upto = dev::wave_incl_sum_u32(rest);
            const uint32_t total = dev::wave_read_u32(upto, 63);
            runs[lane] = run;
            first_group[lane] = upto - rest;
            dev::wave_sync();
            for (uint32_t t = (uint32_t)l0; t < total; t += lstep) {
                uint32_t r = 0;  // the last row whose first group is at t or before
                if (nrows <= 4) {
                    for (uint64_t w = with; w; w &= w - 1) {
                        const int l = __builtin_ctzll(w);
                        r = (uint32_t)uni((int32_t)(upto - rest), l) <= t ? (uint32_t)l : r;
                    }
                } else {
#pragma unroll
                    for (uint32_t d = 32; d > 0; d >>= 1)
                        if (first_group[r + d] <= t) r += d;
                }
                const Run x = runs[r];
                // in the row's order: left pads lie before the frames, right ones after
                int32_t g = (int32_t)(t - first_group[r]);
                if (PADDED && x.npad > 0 && a.left && g >= x.pad0) g += x.npad;
                if (x.nfast > 0 && g >= x.before) g += x.nfast;
                if (PADDED && x.npad > 0 && !a.left && g >= x.pad0) g += x.npad;
                put_group(x, 4 * g - (int32_t)((uint32_t)(x.dlo + al) & 3u));
            }
            dev::wave_sync();
        }
    }
    if (err) dev::raise_error(a.err_hdr, err);
}

template <bool KMER, int U>
int launch_one(RowsArgs a, hipStream_t stream) {
    const bool multi = a.nv > 1, plain = !multi && !a.revcomp && !a.overlap;
    const int64_t T = 1024 * U * (multi ? kRowWaves : 1);
    a.ntiles = std::max<int64_t>(1, (a.nbytes + a.shift + T - 1) / T);
    const uint32_t stage = stage_bytes<KMER>((uint32_t)(T / 16));
    a.wave_lds = stage + kRunBytes;
    const size_t dyn = (multi ? stage + (size_t)kRowWaves * kRunBytes : (size_t)kRowWaves * a.wave_lds) +
                       (a.self_scan ? 8 * (size_t)kSelfScanRows : 0);
    const int32_t extra = a.n > 0 ? (a.n - 1) / 64 : 0;
    // A variant's cell takes some 20 instructions more than a plain one, and a
    // small batch leaves most of the chip idle: 1,000 rows of 50 to 100 bases
    // PADDED as overlapping 6-mers take 15.1 us with a wave per tile, 7.3 with
    // four. Past two tiles a CU, or with more 64-row steps than tiles, the
    // staging done four times costs more (10^6 bases 7.7 and 8.2 us).
    const bool shared = !multi && !plain && U == 1 && extra <= a.ntiles && a.ntiles <= 2 * (int64_t)device_cu_count();
    const int per_group = multi || shared ? 1 : kRowWaves;  // tiles
    constexpr RowsMode SHARED = U == 1 ? ROWS_SHARED : ROWS_VARIANT;
    auto *kernel = a.padded ? (plain    ? k_rows<KMER, U, true, ROWS_PLAIN>
                               : multi  ? k_rows<true, U, true, ROWS_MULTI>
                               : shared ? k_rows<KMER, U, true, SHARED>
                                        : k_rows<KMER, U, true, ROWS_VARIANT>)
                            : (plain    ? k_rows<KMER, U, false, ROWS_PLAIN>
                               : multi  ? k_rows<true, U, false, ROWS_MULTI>
                               : shared ? k_rows<KMER, U, false, SHARED>
                                        : k_rows<KMER, U, false, ROWS_VARIANT>);
    a.pads = (a.pad_units + kRowWaves - 1) / kRowWaves;
    a.lead = a.nv * a.scan_units + a.pads + (extra + per_group - 1) / per_group;
    a.lead = (a.lead + 7) / 8 * 8;  // keeps tile workgroup b on XCD b % 8
    const int64_t grid = a.lead + (a.ntiles + per_group - 1) / per_group;
    if (dyn > 64 * 1024)
        DNATOK_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn));
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NTR), dyn, stream, a);
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

template <bool KMER>
int launch_u(const RowsArgs &a, int U, hipStream_t stream) {
    switch (U) {
    case 1: return launch_one<KMER, 1>(a, stream);
    case 2: return launch_one<KMER, 2>(a, stream);
    case 4: return launch_one<KMER, 4>(a, stream);
    default: return launch_one<KMER, 8>(a, stream);
    }
}

}  // namespace

int launch_encode_rows(const dnatok_vocab *const *vs, int nv, const uint8_t *d_bytes, int64_t nbytes,
                       const int64_t *d_offsets, int32_t n, int32_t *const *d_ids, const int64_t *caps,
                       int64_t *const *d_out_offsets, int8_t *const *d_masks, const dnatok_encode_opts *os,
                       int64_t tile_bytes, hipStream_t stream) {
    const dnatok_vocab *v = vs[0];
    const dnatok_encode_opts &o = os[0];
    const bool kmer = v->kind == DNATOK_KMER;
    RowsArgs a = {};
    const uintptr_t addr = reinterpret_cast<uintptr_t>(d_bytes);
    a.shift = (int64_t)(addr & 15);
    a.abase = d_bytes ? d_bytes - a.shift : nullptr;
    a.nbytes = nbytes;
    a.offs = d_offsets;
    a.n = n;
    a.nv = nv;
    a.cls = o.add_cls_sep ? 1 : 0;
    a.padded = o.layout == DNATOK_PADDED ? 1 : 0;
    a.left = o.pad_side == DNATOK_PAD_LEFT ? 1 : 0;
    a.overlap = kmer && (o.variant & DNATOK_VARIANT_OVERLAP) ? 1 : 0;
    a.revcomp = o.variant & DNATOK_VARIANT_REVCOMP ? 1 : 0;
    a.rows_per_byte = nbytes > 0 ? (double)n / (double)nbytes : 0.0;
    a.lut = v->d_lut;
    Workspace *ws = nullptr;
    int rc = get_workspace(stream, 1, &ws);
    if (rc) return rc;
    a.err_hdr = ws->d_hdr;
    // (the variants' kernel takes the scan from its own launch)
    a.self_scan = !a.padded && nv == 1 && !a.revcomp && !a.overlap && n <= kSelfScanRows ? 1 : 0;
    const bool fused = a.padded && n <= kFusedScanRows;
    a.scan_units = fused ? (int32_t)rowscan_units(n) : 0;
    double cells = 0;
    for (int vi = 0; vi < nv; ++vi) {
        const int64_t W = a.padded ? os[vi].pad_to : 0, st = kmer && !a.overlap ? vs[vi]->k : 1;
        if (W > kPadsApartWidth || (double)W * n * (double)st > 8.0 * ((double)nbytes + 3.0 * n)) a.pads_apart = 1;
        cells += (double)W * n;
    }
    a.pad_cells = kPadCells / 8;  // larger while every CU has two units
    while (a.pad_cells < kPadCells && cells / (2 * a.pad_cells) >= 2.0 * device_cu_count()) a.pad_cells *= 2;
    for (int vi = 0; vi < nv; ++vi) {
        RowsVocab &x = a.vo[vi];
        x.k = kmer ? vs[vi]->k : 1;
        x.kinv = 0xFFFFFFFFu / (uint32_t)x.k;
        x.al = (int32_t)((reinterpret_cast<uintptr_t>(d_ids[vi]) >> 2) & 3);
        x.pad_id = vs[vi]->pad_id;
        x.cls_id = vs[vi]->cls_id;
        x.sep_id = vs[vi]->sep_id;
        x.ids = d_ids[vi];
        x.mask = d_masks[vi];
        x.cap = caps[vi];
        x.out_offs = d_out_offsets[vi];
        x.W = a.padded ? os[vi].pad_to : 0;
        if (x.W >= (1 << 28)) a.wide = 1;
        x.pad_first = a.pad_units;
        if (a.pads_apart) {
            x.pad_parts = (int32_t)std::max<int64_t>(1, (x.W + a.pad_cells - 1) / a.pad_cells);
            x.pad_rows = (int32_t)std::min<int64_t>(64, std::max<int64_t>(1, a.pad_cells / x.W));
            a.pad_units += x.pad_parts > 1 ? (int32_t)((int64_t)n * x.pad_parts) : (n + x.pad_rows - 1) / x.pad_rows;
        }
        x.base = os[vi].offset_base;
        if (!fused && !a.self_scan) {
            RowScanSpec sp;
            sp.offs = d_offsets;
            sp.n = n;
            sp.nbytes = nbytes;
            sp.out = d_out_offsets[vi];
            sp.k = x.k;
            sp.kmer = kmer ? 1 : 0;
            sp.overlap = a.overlap;
            sp.cls = a.cls;
            sp.padded = a.padded;
            sp.W = x.W;
            sp.base = x.base;
            rc = launch_rowscan_spec(sp, stream);
            if (rc) return rc;
        }
    }
    int U = 1;
    while (U < 8 && 1024 * (int64_t)(2 * U) * kRowWaves <= tile_bytes) U <<= 1;
    return kmer ? launch_u<true>(a, U, stream) : launch_u<false>(a, U, stream);
}

}  // namespace dnatok
