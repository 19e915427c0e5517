// Output-parallel cell kernel: the embedding lookup, fused with the encode
// (every variant) or applied to given identifiers.
//
// Paper: Design (the embedder embed_tokens maps B x T identifiers to
// B x T x D activations; the bytes branch of the EmbedFromStrings algorithm
// maps bytes to identifiers on the device, left-pads them to token_len and
// hands them to embed_tokens); Discussion, "Integration with Data
// Augmentation" (reverse complement as a character-level map suited to the
// GPU); Introduction (overlapping k-mers of stride 1, L - k + 1 tokens).
//
// MI355X-first decomposition. The output dominates the traffic: an embedding
// row of D values per token (256 bytes for D = 128 in bf16, against about one
// input byte). Work is therefore cut by output cells rather than input tiles:
//  * A block takes a tile of about 32 KiB of output (4 to 1,024 consecutive
//    cells; cells = tokens plus pads), a thread CPT consecutive cells: one, or
//    four of small rows, whose ids go out as one 16-byte store and their mask
//    bytes as one word. Every XCD takes one contiguous part of the tiles. A
//    thread finds the row of its first cell (PADDED: cell / W with a 32-bit
//    reciprocal; PACKED: its wave looks its first cell's row up, first among
//    those around the place it would have were all rows equally long, reads that
//    row and the 63 after it, one per lane, and a thread finds its own among
//    them) and steps to the next row only at a row end. It places
//    every cell first (pad, CLS, SEP or body token, and the bytes a body
//    token reads), then issues all of its reads at once: a k-mer reads the
//    three (k <= 8) or five dwords that hold it and classifies them with
//    the same 16-byte classifier the encode uses; reverse complement
//    reverses and complements the digits in registers (the bytes are never
//    rewritten), and for table kinds it reads a table already mapped
//    through the complement.
//  * The tile's table rows go to LDS and the block copies
//    them out in UB-byte units (UB = 16 whenever the row size and
//    pointers allow): lane l of a wave moves unit l, so a wave writes 1 KiB
//    of contiguous output per instruction. Several units are loaded before
//    any is stored. Table rows are read through L2 (a 4101 x 256-byte table
//    is 1 MiB, resident there); the output is the only HBM stream.
// The store pattern bounds it: the same stores without the lookup take 101 of
// 103 us when 256 KiB belong to a block in grid order. 4,096 rows of 512
// bases, 256-byte table rows (541 MB): 103 -> 86 us, a fill of it 78; 300 rows
// of 3,000 bases as 6-mers: 18.7 -> 10.5; 1,000 of 50 to 100: 19.4 -> 6.0;
// PACKED, 100,000 of 20 to 150: 105 -> 89.
// Bounds: every output index is below the capacity the caller gave; bad
// offsets are clamped exactly as the row scan clamps them, so cell positions
// and the written offsets agree.
#include "common.hpp"
#include "device.hpp"
#include "rowscan.hpp"

namespace dnatok {

namespace {

constexpr int NT = 256;
static_assert(NT == kScanNT, "the fused row scan runs with the cell kernel's block size");
constexpr int64_t kMaxGrid = 1 << 20;        // workgroups of cells
constexpr int kWalkersPerCu = 20;            // of them, where they take tiles in turn
constexpr int kMaxCells = NT * 4;            // cells of a tile
constexpr int kTileBytes = 32768;            // output of a tile, where kMaxCells allows

enum CwMode { CW_EMBED = 1, CW_GATHER = 2 };

struct CwArgs {
    const uint8_t *bytes;
    int64_t nbytes;
    const int64_t *offs;
    int32_t n;
    int32_t lut_kind;        // 1: id = lut[byte] (SINGLE, LUT256); 0: k-mer windows
    int64_t *scan_out;       // out_offsets, written by the scanning workgroups
    const int64_t *out_offs; // PACKED row starts (offset_base included)
    int64_t base;
    int64_t ncells;          // PADDED: n * W; GATHER: n_ids; PACKED: -1 (read out_offs[n])
    int64_t cap;             // cells the outputs hold
    int32_t k;
    int32_t stride;          // k (frames) or 1 (overlapping windows)
    int32_t overlap;
    int32_t revcomp;
    int32_t cls, padded, left;
    int64_t W;
    uint32_t winv;           // floor((2^32 - 1) / W) when W < 2^31, else 0
    uint32_t kinv;           // floor((2^32 - 1) / k)
    int32_t pad_id, cls_id, sep_id;
    const int32_t *lut;
    int32_t *ids;            // optional for EMBED
    int8_t *mask;            // PADDED, optional for EMBED
    const int32_t *ids_in;   // GATHER: int32 ids (or)
    const int64_t *ids_in64; // GATHER: int64 ids
    const uint8_t *table;
    int64_t n_rows;
    int64_t row_bytes;
    uint8_t *emb;
    uint32_t ru, ruinv;      // units per table row and floor((2^32 - 1) / ru)
    uint32_t step_cell, step_part;  // NT units in rows and units
    uint32_t *err_hdr;
    int32_t cells;           // cells of a tile, a multiple of CPT
    int32_t parts;           // every XCD takes one contiguous part of the tiles
    int32_t scan_units;      // PADDED, up to kFusedScanRows rows: the first workgroups scan the rows
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int UB>
struct Unit;
template <>
struct Unit<16> {
    typedef u32x4 T;
};
template <>
struct Unit<8> {
    typedef u32x2 T;
};
template <>
struct Unit<4> {
    typedef uint32_t T;
};
template <>
struct Unit<2> {
    typedef uint16_t T;
};
template <>
struct Unit<1> {
    typedef uint8_t T;
};

// x / d for x < 2^32 with dinv = floor((2^32 - 1) / d): the high product is
// the quotient or one less, and one step corrects it.
__device__ __forceinline__ uint32_t udiv(uint32_t x, uint32_t d, uint32_t dinv) {
    uint32_t q = __umulhi(x, dinv);
    if (x - q * d >= d) ++q;
    return q;
}

// x / d for x >= 0, d >= 1, with the 32-bit path when both fit.
__device__ __forceinline__ int64_t div_any(int64_t x, int64_t d, uint32_t dinv) {
    if (dinv && x < ((int64_t)1 << 32)) return udiv((uint32_t)x, (uint32_t)d, dinv);
    return x / d;
}

// Watson-Crick complement of a byte, case kept; other bytes unchanged.
__device__ __forceinline__ uint32_t complement(uint32_t b) {
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

// Row facts with offsets clamped as the row scan clamps them.
struct RowFacts {
    int64_t o0, o1, nb, len;
};

__device__ __forceinline__ RowFacts row_facts(const CwArgs &a, int64_t o0, int64_t o1) {
    RowFacts f;
    o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
    o1 = o1 < o0 ? o0 : (o1 > a.nbytes ? a.nbytes : o1);
    const int64_t L = o1 - o0;
    int64_t nb;
    if (a.lut_kind) nb = L;
    else if (a.overlap) nb = L >= a.k ? L - a.k + 1 : (L > 0 ? 1 : 0);
    else nb = div_any(L + a.k - 1, a.k, a.kinv);
    f.o0 = o0;
    f.o1 = o1;
    f.nb = nb;
    f.len = nb + 2 * a.cls;
    return f;
}
__device__ __forceinline__ RowFacts row_facts(const CwArgs &a, int64_t r) {
    return row_facts(a, a.offs[r], a.offs[r + 1]);
}

// The 16 bytes from p on, for a k-mer at p (k <= 8 needs three dwords,
// k <= 15 five). Dword addresses are clamped to the dword that holds the
// k-mer's last byte, so every read stays within the dwords the k-mer
// occupies; bytes past the k-mer are don't-cares.
template <bool K8>
__device__ __forceinline__ uint4 window16(const uint8_t *p, int32_t k) {
    constexpr int ND = K8 ? 3 : 5;
    const uintptr_t addr = reinterpret_cast<uintptr_t>(p);
    const uint32_t sh = (uint32_t)(addr & 3);
    const uint8_t *first = p - sh;
    const uint8_t *last = p + (k - 1) - ((addr + (uintptr_t)(k - 1)) & 3);
    uint32_t w[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if (i < ND) {
            const uint8_t *q = first + 4 * i;
            w[i] = *reinterpret_cast<const uint32_t *>(q < last ? q : last);
        } else {
            w[i] = 0;
        }
    }
    uint4 r;
    r.x = __builtin_amdgcn_alignbyte(w[1], w[0], sh);
    r.y = __builtin_amdgcn_alignbyte(w[2], w[1], sh);
    r.z = __builtin_amdgcn_alignbyte(w[3], w[2], sh);
    r.w = __builtin_amdgcn_alignbyte(w[4], w[3], sh);
    return r;
}

// Id of the k-mer whose bytes (in memory order) open window v; reverse
// complement: of those bytes taken back to front, each complemented.
__device__ __forceinline__ int32_t kmer_id(uint4 v, int32_t k, int32_t revcomp) {
    uint32_t code, valid;
    dev::classify16(v, code, valid);
    const uint32_t km = (1u << k) - 1u;
    if ((valid >> (32 - k)) != km) return DNATOK_ID_UNK;
    uint32_t x = code >> (32 - 2 * k);
    if (revcomp) {
        // digits in reverse order (bit reversal, then each 2-bit digit's
        // bits swapped back), each complemented (3 - d = d ^ 3)
        uint32_t y = __builtin_bitreverse32(x);
        y = ((y >> 1) & 0x55555555u) | ((y & 0x55555555u) << 1);
        x = (y >> (32 - 2 * k)) ^ ((1u << (2 * k)) - 1u);
    }
    return (int32_t)(5 + x);
}

// Row of a PACKED cell: the first r in [lo, hi] with out_offs[r + 1] - base > cell.
__device__ __forceinline__ int64_t packed_row(const CwArgs &a, int64_t lo, int64_t hi, int64_t cell) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a.out_offs[mid + 1] - a.base > cell) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// Ids of the cells cb .. cb + CPT - 1 (those below cend) and whether each
// holds a token (not a pad). First every cell is placed (row, token kind,
// and for a body token the bytes it reads; other cells point their reads
// at the offsets array, which always holds a readable word), then all
// reads are issued, then the ids are formed. Rows change within a thread's
// cells only at row ends.
template <bool K8, int CPT, bool PADDED>
__device__ __forceinline__ void thread_cells(const CwArgs &a, const int32_t *s_lut, int64_t cb, int64_t cend,
                                             int64_t row, int64_t p, RowFacts f, int32_t (&id)[CPT],
                                             bool (&tok)[CPT]) {
    // Fast path: the CPT cells are body tokens of this row whose windows
    // lie within 32 bytes (any overlapping k, frames of k <= 8, table
    // kinds): one 32-byte read, two classifications, then shifts per cell.
    {
        const int32_t kw = a.lut_kind ? 1 : a.k;
        const int32_t st = a.lut_kind ? 1 : a.stride;
        const int32_t spanb = (CPT - 1) * st + kw;
        int64_t q0 = p;
        if (PADDED && a.left) q0 = p - (a.W - f.len);
        const int64_t j0 = q0 - a.cls;
        const int64_t s0 = j0 * st;
        if (spanb <= 32 && cb + CPT <= cend && p + CPT <= (PADDED ? a.W : f.len) && q0 >= a.cls &&
            q0 + CPT <= f.len - a.cls && s0 + spanb <= f.o1 - f.o0) {
            const int64_t lo = a.revcomp ? f.o1 - s0 - spanb : f.o0 + s0;
            const uint8_t *pl = a.bytes + lo;
            const uintptr_t addr = reinterpret_cast<uintptr_t>(pl);
            const uint32_t sh = (uint32_t)(addr & 3);
            const uint8_t *first = pl - sh;
            const uint8_t *last = pl + (spanb - 1) - ((addr + (uintptr_t)(spanb - 1)) & 3);
            uint32_t w[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const uint8_t *q = first + 4 * i;
                w[i] = *reinterpret_cast<const uint32_t *>(q < last ? q : last);
            }
            if (a.lut_kind) {
                const uint32_t b4 = __builtin_amdgcn_alignbyte(w[1], w[0], sh);
#pragma unroll
                for (int i = 0; i < CPT; ++i) {
                    const int t = a.revcomp ? CPT - 1 - i : i;
                    id[i] = s_lut[(b4 >> (8 * t)) & 255u];
                    tok[i] = true;
                }
                return;
            }
            uint4 v0, v1;
            v0.x = __builtin_amdgcn_alignbyte(w[1], w[0], sh);
            v0.y = __builtin_amdgcn_alignbyte(w[2], w[1], sh);
            v0.z = __builtin_amdgcn_alignbyte(w[3], w[2], sh);
            v0.w = __builtin_amdgcn_alignbyte(w[4], w[3], sh);
            v1.x = __builtin_amdgcn_alignbyte(w[5], w[4], sh);
            v1.y = __builtin_amdgcn_alignbyte(w[6], w[5], sh);
            v1.z = __builtin_amdgcn_alignbyte(w[7], w[6], sh);
            v1.w = __builtin_amdgcn_alignbyte(w[8], w[7], sh);
            uint32_t c0, c1, va0, va1;
            dev::classify16(v0, c0, va0);
            dev::classify16(v1, c1, va1);
            const uint64_t code = ((uint64_t)c0 << 32) | c1;  // 32 digits, first byte on top
            const uint32_t valid = va0 | (va1 >> 16);         // 32 validity bits, first byte on top
            const int32_t k = a.k;
            const uint32_t km = (1u << k) - 1u;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int32_t off = (a.revcomp ? CPT - 1 - i : i) * st;  // window of cell i within the 32 bytes
                uint32_t x = (uint32_t)((code << (2 * off)) >> (64 - 2 * k));
                const bool ok = ((valid << off) >> (32 - k)) == km;
                if (a.revcomp) {
                    uint32_t y = __builtin_bitreverse32(x);
                    y = ((y >> 1) & 0x55555555u) | ((y & 0x55555555u) << 1);
                    x = (y >> (32 - 2 * k)) ^ ((1u << (2 * k)) - 1u);
                }
                id[i] = ok ? (int32_t)(5 + x) : DNATOK_ID_UNK;
                tok[i] = true;
            }
            return;
        }
    }
    const uint8_t *dummy = reinterpret_cast<const uint8_t *>(a.offs);
    const uint8_t *src[CPT];
    int32_t fixed[CPT], kk[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        src[i] = dummy;
        fixed[i] = a.pad_id;
        kk[i] = 1;
        tok[i] = false;
        if (cb + i < cend) {
            if (p == (PADDED ? a.W : f.len)) {
                // the next row (PACKED: the next non-empty one; one exists,
                // since this cell is below the total)
                p = 0;
                do {
                    ++row;
                    f = row_facts(a, row);
                } while (!PADDED && f.len == 0);
            }
            int64_t q = p;
            if (PADDED && a.left) q = p - (a.W - f.len);
            tok[i] = q >= 0 && q < f.len;
            if (tok[i]) {
                if (a.cls && q == 0) {
                    fixed[i] = a.cls_id;
                } else if (a.cls && q == f.len - 1) {
                    fixed[i] = a.sep_id;
                } else {
                    const int64_t j = q - a.cls;
                    if (a.lut_kind) {
                        src[i] = a.bytes + (a.revcomp ? f.o1 - 1 - j : f.o0 + j);
                        fixed[i] = -1;
                    } else {
                        const int64_t s0 = j * a.stride;
                        if (s0 + a.k > f.o1 - f.o0) {
                            fixed[i] = DNATOK_ID_UNK;  // short final frame, or a row shorter than k
                        } else {
                            src[i] = a.bytes + (a.revcomp ? f.o1 - s0 - a.k : f.o0 + s0);
                            fixed[i] = -1;
                            kk[i] = a.k;
                        }
                    }
                }
            }
            ++p;
        }
    }
    if (a.lut_kind) {
        uint32_t b[CPT];
#pragma unroll
        for (int i = 0; i < CPT; ++i) b[i] = *src[i];
#pragma unroll
        for (int i = 0; i < CPT; ++i) id[i] = fixed[i] >= 0 ? fixed[i] : s_lut[b[i]];
    } else {
        uint4 win[CPT];
#pragma unroll
        for (int i = 0; i < CPT; ++i) win[i] = window16<K8>(src[i], kk[i]);
#pragma unroll
        for (int i = 0; i < CPT; ++i) id[i] = fixed[i] >= 0 ? fixed[i] : kmer_id(win[i], a.k, a.revcomp);
    }
}

template <int MODE, int UB, bool K8, int CPT, bool PADDED>
__global__ __launch_bounds__(NT, CPT == 1 && PADDED ? 1 : 5) void k_cellwise(CwArgs a) {
    constexpr int kCopyUnroll = CPT == 1 ? 8 : 4;  // table units loaded before they are stored
    __shared__ int32_t s_lut[256];
    __shared__ int64_t s_row[NT * CPT];  // table row of a cell, in bytes; -1: none
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    if (MODE != CW_GATHER && (int)blockIdx.x < a.scan_units) {
        __shared__ int64_t s_tmp[kScanNT / dev::kWave + 1];
        rowscan_independent(RowLen{a.offs, a.nbytes, a.n, a.k, a.kinv, a.lut_kind ? 0 : 1, a.overlap, a.cls, a.W},
                            a.scan_out, a.base, (int)blockIdx.x, s_tmp, a.err_hdr);
        return;
    }
    const int64_t bid = (int64_t)blockIdx.x - a.scan_units;
    int64_t total = a.ncells;
    if (total < 0) total = a.out_offs[a.n] - a.base;
    const int64_t limit = total < a.cap ? total : a.cap;
    if (bid == 0 && tid == 0 && total > a.cap) dev::raise_error(a.err_hdr, DNATOK_DERR_CAPACITY);
    // The tiles there are go to the first blocks, every XCD one part of them
    // (one tile per block up to kMaxGrid blocks): a grid sized by a buffer of
    // several times the rows would put them all on the first XCDs.
    const int64_t G = min((int64_t)gridDim.x - a.scan_units, (limit + a.cells - 1) / a.cells);
    if (bid >= G) return;
    if (MODE != CW_GATHER) s_lut[tid] = a.lut[a.revcomp ? complement((uint32_t)tid) : (uint32_t)tid];
    uint32_t err = 0;
    __syncthreads();

    for (int64_t c0 = (a.parts ? dev::xcd_tile(bid, G) : bid) * a.cells; c0 < limit; c0 += G * a.cells) {
        const int64_t cend = limit - c0 < a.cells ? limit : c0 + a.cells;
        const int64_t wb = c0 + w * dev::kWave * CPT;  // the wave's first cell
        const int64_t cb = c0 + tid * CPT;             // this thread's CPT consecutive cells
        int64_t row = 0, p = 0;                        // the row of its first one, and the place there
        RowFacts f{0, 0, 0, 0};
        if (MODE != CW_GATHER && PADDED && cb < cend) {
            row = div_any(cb, a.W, a.winv);
            p = cb - row * a.W;
            f = row_facts(a, row);
        }
        if (MODE != CW_GATHER && !PADDED && wb < cend) {
            const int64_t n = a.n, we = min(wb + dev::kWave * CPT, cend) - 1;
            const int lane = tid & (dev::kWave - 1);
            auto past = [&](int64_t key) {
                return [&a, key](int64_t q) { return a.out_offs[q + 1] - a.base > key; };
            };
            // the row of the wave's first cell, looked for first among the
            // 4,096 around the one it would be in if all were equally long
            int64_t lo = 0, hi = n;
            if (n > 4096) {
                const int64_t g = min(max((int64_t)((double)wb / (double)total * (double)n) - 2048, (int64_t)0), n - 4096);
                const uint64_t b = __ballot(past(wb)(g + 64 * (int64_t)lane + 63));
                const int first = b ? __builtin_ctzll(b) : 64;
                if (first == 0) hi = g + 63;
                else if (first == 64) lo = g + 4096;
                else lo = g + 64 * first, hi = lo + 63;
            }
            const int64_t r0 = dev::wave_lower_bound(lo, hi, past(wb));
            // it and the 63 after it, one per lane
            const int64_t r = min(r0 + lane, n), r2 = min(r + 1, n);
            const int64_t start = a.out_offs[r] - a.base, end = a.out_offs[r2] - a.base, o0 = a.offs[r], o1 = a.offs[r2];
            if (__ballot(end > we)) {
                int at = 0;  // rows that end at the thread's cell or before
#pragma unroll
                for (int d = 32; d > 0; d >>= 1)
                    if (__shfl((long long)end, at + d - 1, dev::kWave) <= cb) at += d;
                row = r0 + at;
                p = cb - __shfl((long long)start, at, dev::kWave);
                const int64_t x0 = __shfl((long long)o0, at, dev::kWave), x1 = __shfl((long long)o1, at, dev::kWave);
                f = row_facts(a, x0, x1);
            } else if (cb < cend) {  // more rows than lanes
                row = packed_row(a, r0, n, cb);
                p = cb - (a.out_offs[row] - a.base);
                f = row_facts(a, row);
            }
        }
        int32_t id[CPT];
        bool tok[CPT];
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            id[i] = 0;
            tok[i] = false;
        }
        if (MODE == CW_GATHER) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                if (cb + i < cend) {
                    const int64_t x = a.ids_in64 ? a.ids_in64[cb + i] : (int64_t)a.ids_in[cb + i];
                    id[i] = (int32_t)x;
                    if (x < 0 || x >= a.n_rows) {
                        err |= DNATOK_DERR_IDS;
                        id[i] = -1;
                    }
                }
            }
        } else if (cb < cend) {
            thread_cells<K8, CPT, PADDED>(a, s_lut, cb, cend, row, p, f, id, tok);
        }
        if (MODE != CW_GATHER && cb < cend) {
            const bool full = CPT % 4 == 0 && cb + CPT <= cend;
            if (a.ids) {
                if (full && ((reinterpret_cast<uintptr_t>(a.ids + cb) & 15) == 0)) {
#pragma unroll
                    for (int g = 0; g + 3 < CPT; g += 4)
                        *reinterpret_cast<int4 *>(a.ids + cb + g) = make_int4(id[g], id[g + 1], id[g + 2], id[g + 3]);
                } else {
#pragma unroll
                    for (int i = 0; i < CPT; ++i)
                        if (cb + i < cend) a.ids[cb + i] = id[i];
                }
            }
            if (a.mask) {
                if (full && ((reinterpret_cast<uintptr_t>(a.mask + cb) & 3) == 0)) {
#pragma unroll
                    for (int g = 0; g + 3 < CPT; g += 4)
                        *reinterpret_cast<uint32_t *>(a.mask + cb + g) = (uint32_t)tok[g] | (uint32_t)tok[g + 1] << 8 |
                                                                         (uint32_t)tok[g + 2] << 16 |
                                                                         (uint32_t)tok[g + 3] << 24;
                } else {
#pragma unroll
                    for (int i = 0; i < CPT; ++i)
                        if (cb + i < cend) a.mask[cb + i] = tok[i] ? 1 : 0;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < CPT; ++i) s_row[tid * CPT + i] = id[i] >= 0 ? (int64_t)id[i] * a.row_bytes : -1;
        typedef typename Unit<UB>::T V;
        __syncthreads();
        const uint32_t units = (uint32_t)(cend - c0) * a.ru;
        uint8_t *ob = a.emb + c0 * a.row_bytes;
        uint32_t cell = udiv(tid, a.ru, a.ruinv), part = tid - cell * a.ru;
        for (uint32_t u0 = tid; u0 < units; u0 += NT * kCopyUnroll) {
            V v[kCopyUnroll];
#pragma unroll
            for (int t = 0; t < kCopyUnroll; ++t) {
                const int64_t row = u0 + t * NT < units ? s_row[cell] : -1;
                if (row >= 0) v[t] = *reinterpret_cast<const V *>(a.table + row + part * UB);
                else v[t] = V{};
                cell += a.step_cell;  // the unit NT further on
                part += a.step_part;
                if (part >= a.ru) {
                    part -= a.ru;
                    ++cell;
                }
            }
#pragma unroll
            for (int t = 0; t < kCopyUnroll; ++t) {
                const uint32_t u = u0 + t * NT;
                if (u < units) __builtin_nontemporal_store(v[t], reinterpret_cast<V *>(ob) + u);
            }
        }
        __syncthreads();
    }
    if (err) dev::raise_error(a.err_hdr, err);
}

template <int MODE, int UB, bool K8>
int launch_cw(const CwArgs &a, int64_t max_cells, hipStream_t stream) {
    const int64_t most = a.parts ? kMaxGrid : (int64_t)kWalkersPerCu * device_cu_count();
    const int64_t g = std::min(std::max<int64_t>(1, (max_cells + a.cells - 1) / a.cells), most) + a.scan_units;
    constexpr bool GATHER = MODE == CW_GATHER;
    auto *one = a.padded || GATHER ? k_cellwise<MODE, UB, K8, 1, true> : k_cellwise<MODE, UB, K8, 1, GATHER>;
    auto *four = a.padded || GATHER ? k_cellwise<MODE, UB, K8, 4, true> : k_cellwise<MODE, UB, K8, 4, GATHER>;
    // Four workgroups a CU (held by the LDS they ask for) but for PACKED k-mers,
    // which take longest to place: the fewer store, the nearer they come to a
    // fill. 4,096 rows of 512 bases, 256-byte table rows, five and four: PADDED
    // 87.7 and 86.0 us, PACKED 100.7 and 93.9; 40,000 rows of 1,000 bases PACKED
    // as 6-mers 311 and 355. (Three PADDED: 79.1 there, but 5% longer at 8,192
    // bases a row.)
    const bool hold = a.cells <= NT && !GATHER && (a.padded || a.lut_kind);
    const size_t lds = hold ? 34 * 1024 : 0;
    hipLaunchKernelGGL(a.cells <= NT ? one : four, dim3((unsigned)g), dim3(NT), lds, stream, a);
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

// k-mers of up to 8 bases read three dwords per token, longer ones five.
template <int MODE, int UB>
int launch_cw_k(const CwArgs &a, int64_t max_cells, hipStream_t stream) {
    if (MODE == CW_GATHER || a.lut_kind || a.k <= 8) return launch_cw<MODE, UB, true>(a, max_cells, stream);
    return launch_cw<MODE, UB, MODE == CW_GATHER>(a, max_cells, stream);
}

template <int MODE>
int launch_cw_units(CwArgs &a, int64_t max_cells, hipStream_t stream) {
    // widest unit dividing the row size and both row bases
    const uintptr_t al = reinterpret_cast<uintptr_t>(a.table) | reinterpret_cast<uintptr_t>(a.emb) |
                         (uintptr_t)a.row_bytes;
    int ub = 16;
    while (ub > 1 && (al & (uintptr_t)(ub - 1))) ub >>= 1;
    a.ru = (uint32_t)(a.row_bytes / ub);
    a.ruinv = 0xFFFFFFFFu / a.ru;
    a.step_cell = NT / a.ru;
    a.step_part = NT % a.ru;
    // 32 KiB a tile, one cell per thread: with four, 32 of 256 threads placed a
    // tile of 256-byte rows (3.5M 6-mers of 100,000 reads 141 us PACKED, this
    // way 89). Rows of less than 128 bytes, four cells per thread, and where
    // they are placed 1,024 of them, up to 16 KiB a tile in the grid's order, as
    // placing outweighs the stores (41M cells of 16 bytes PACKED 195 us, in
    // parts 207; 5M given ids of 64 bytes 55 us in tiles of 512, of 1,024 62).
    const int64_t fit = std::max<int64_t>(4, kTileBytes / a.row_bytes / 4 * 4);
    const bool small = MODE != CW_GATHER && a.row_bytes < kTileBytes / NT;
    a.cells = small ? kMaxCells : (int32_t)std::min<int64_t>(fit, kMaxCells);
    a.parts = !small || a.cells * a.row_bytes > kTileBytes / 2;
    switch (ub) {
    case 16: return launch_cw_k<MODE, 16>(a, max_cells, stream);
    case 8: return launch_cw_k<MODE, 8>(a, max_cells, stream);
    case 4: return launch_cw_k<MODE, 4>(a, max_cells, stream);
    case 2: return launch_cw_k<MODE, 2>(a, max_cells, stream);
    default: return launch_cw_k<MODE, 1>(a, max_cells, stream);
    }
}

// Common set-up of the encode-side modes: row scan (out_offsets), then
// the cell arguments.
int setup_encode(CwArgs &a, const dnatok_vocab *v, const uint8_t *d_bytes, int64_t nbytes, const int64_t *d_offsets,
                 int32_t n, int64_t *d_out_offsets, const dnatok_encode_opts &o, hipStream_t stream,
                 int64_t *max_cells) {
    const bool kmer = v->kind == DNATOK_KMER;
    a = CwArgs{};
    a.bytes = d_bytes;
    a.nbytes = nbytes;
    a.offs = d_offsets;
    a.n = n;
    a.lut_kind = kmer ? 0 : 1;
    a.out_offs = d_out_offsets;
    a.base = o.offset_base;
    a.k = kmer ? v->k : 1;
    a.overlap = (o.variant & DNATOK_VARIANT_OVERLAP) ? 1 : 0;
    a.stride = a.overlap ? 1 : a.k;
    a.kinv = 0xFFFFFFFFu / (uint32_t)a.k;
    a.revcomp = (o.variant & DNATOK_VARIANT_REVCOMP) ? 1 : 0;
    a.cls = o.add_cls_sep ? 1 : 0;
    a.padded = o.layout == DNATOK_PADDED ? 1 : 0;
    a.left = o.pad_side == DNATOK_PAD_LEFT ? 1 : 0;
    a.W = a.padded ? o.pad_to : 0;
    a.winv = (a.padded && a.W < ((int64_t)1 << 31)) ? 0xFFFFFFFFu / (uint32_t)a.W : 0;
    a.pad_id = v->pad_id;
    a.cls_id = v->cls_id;
    a.sep_id = v->sep_id;
    a.lut = v->d_lut;

    Workspace *ws = nullptr;
    int rc = get_workspace(stream, 1, &ws);
    if (rc) return rc;
    a.scan_units = a.padded && n <= kFusedScanRows ? (int32_t)rowscan_units(n) : 0;
    a.scan_out = d_out_offsets;
    if (!a.scan_units) {
        RowScanSpec sp;
        sp.offs = d_offsets;
        sp.n = n;
        sp.nbytes = nbytes;
        sp.out = d_out_offsets;
        sp.k = a.k;
        sp.kmer = kmer ? 1 : 0;
        sp.overlap = a.overlap;
        sp.cls = a.cls;
        sp.padded = a.padded;
        sp.W = a.W;
        sp.base = a.base;
        rc = launch_rowscan_spec(sp, stream);
        if (rc) return rc;
    }
    a.err_hdr = ws->d_hdr;
    a.ncells = a.padded ? (int64_t)n * a.W : -1;
    // PACKED: the most that rows of nbytes together can have
    const int64_t stride = kmer ? a.stride : 1;
    *max_cells = a.padded ? a.ncells : nbytes / stride + (stride > 1 || a.overlap ? n : 0) + 2 * (int64_t)a.cls * n;
    return DNATOK_OK;
}

}  // namespace

int launch_embed(const dnatok_vocab *v, const uint8_t *d_bytes, int64_t nbytes, const int64_t *d_offsets, int32_t n,
                 const void *d_table, int64_t n_rows, int64_t row_bytes, void *d_out, int64_t out_rows,
                 int64_t *d_out_offsets, int32_t *d_ids, int8_t *d_mask, const dnatok_encode_opts &o,
                 hipStream_t stream) {
    CwArgs a;
    int64_t max_cells = 0;
    int rc = setup_encode(a, v, d_bytes, nbytes, d_offsets, n, d_out_offsets, o, stream, &max_cells);
    if (rc) return rc;
    a.ids = d_ids;
    a.mask = a.padded ? d_mask : nullptr;
    a.cap = out_rows;
    a.table = static_cast<const uint8_t *>(d_table);
    a.n_rows = n_rows;
    a.row_bytes = row_bytes;
    a.emb = static_cast<uint8_t *>(d_out);
    if (max_cells > out_rows) max_cells = out_rows;
    return launch_cw_units<CW_EMBED>(a, max_cells, stream);
}

int launch_embed_ids(const int32_t *d_ids, const int64_t *d_ids64, int64_t n_ids, const void *d_table,
                     int64_t n_rows, int64_t row_bytes, void *d_out, hipStream_t stream) {
    CwArgs a = CwArgs{};
    Workspace *ws = nullptr;
    int rc = get_workspace(stream, 1, &ws);
    if (rc) return rc;
    a.err_hdr = ws->d_hdr;
    a.ids_in = d_ids;
    a.ids_in64 = d_ids64;
    a.ncells = n_ids;
    a.cap = n_ids;
    a.table = static_cast<const uint8_t *>(d_table);
    a.n_rows = n_rows;
    a.row_bytes = row_bytes;
    a.emb = static_cast<uint8_t *>(d_out);
    return launch_cw_units<CW_GATHER>(a, n_ids, stream);
}

}  // namespace dnatok
