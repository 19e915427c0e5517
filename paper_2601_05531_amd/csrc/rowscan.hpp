// Row scan of the closed-form token counts (shared by the encode, the
// embedding lookup and the stand-alone scan launches): each row's length is L, its
// number of k-frames ceil(L / k), or its number of stride-1 windows, plus
// the specials; out_offsets is their exclusive scan. Offsets are validated
// and clamped here, so every kernel that places cells from them agrees.
#pragma once

#include "common.hpp"
#include "device.hpp"

namespace dnatok {

namespace {

constexpr int kScanNT = 256;                                 // block size of every launch that scans
constexpr int kRowsPerThread = 16;                           // rows per thread per pass
constexpr int64_t kUnitRows = (int64_t)kScanNT * kRowsPerThread;

// x / k for k >= 1 with kinv = floor((2^32 - 1) / k): the high product is
// floor(x / k) or one less (x < 2^32), and one step corrects it. Quotients
// of 2^31 or more take the plain division.
__device__ __forceinline__ int64_t div_k(int64_t x, int32_t k, uint32_t kinv) {
    if (x < 0x7FFFFFFF) {
        const uint32_t ux = (uint32_t)x;
        uint32_t q = __umulhi(ux, kinv);
        if (ux - q * (uint32_t)k >= (uint32_t)k) ++q;
        return (int64_t)q;
    }
    return x / k;
}

struct RowScanArgs {
    const int64_t *offs;
    int32_t n;
    int64_t nbytes;
    int64_t *out_offs;
    int32_t k;
    uint32_t kinv;  // floor((2^32 - 1) / k)
    int32_t kmer;     // frames of k (2: at least one per row)
    int32_t overlap;  // k-mer windows of stride 1: L - k + 1 (one for 0 < L < k)
    int32_t cls;
    int32_t padded;
    int64_t W;
    int64_t base;
    int64_t nunits;
    dev::TileQueue q;
};

// Lengths of the up-to-kUnitRows rows starting at row0 (validated), their
// exclusive scan written to out_offs after `Prefix(total)` supplies the
// unit's starting value. Returns the unit's token total.
template <class Prefix>
__device__ __forceinline__ int64_t rowscan_unit(const RowScanArgs &a, int64_t row0, int64_t *s_tmp, uint32_t &err,
                                                Prefix prefix) {
    const int tid = threadIdx.x;
    const int64_t i0 = row0 + (int64_t)tid * kRowsPerThread;
    // all of this thread's offsets first, from indices clamped to the batch,
    // so the loads go out together instead of one per row behind its test
    int64_t off[kRowsPerThread + 1];
#pragma unroll
    for (int j = 0; j <= kRowsPerThread; ++j) {
        const int64_t i = i0 + j;
        off[j] = a.offs[i < a.n ? i : a.n];
    }
    int64_t len[kRowsPerThread];
    int64_t mine = 0;
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        const int64_t i = i0 + j;
        len[j] = 0;
        if (i < a.n) {
            int64_t o0 = off[j], o1 = off[j + 1];
            if (o0 < 0 || o1 < o0 || o1 > a.nbytes) err |= DNATOK_DERR_OFFSETS;
            o0 = o0 < 0 ? 0 : (o0 > a.nbytes ? a.nbytes : o0);
            o1 = o1 < o0 ? o0 : (o1 > a.nbytes ? a.nbytes : o1);
            const int64_t L = o1 - o0;
            int64_t nb = L;
            if (a.kmer) nb = a.overlap ? (L >= a.k ? L - a.k + 1 : (L > 0 ? 1 : 0)) : div_k(L + a.k - 1, a.k, a.kinv);
            if (a.kmer == 2 && nb == 0) nb = 1;
            len[j] = nb + 2 * a.cls;
            if (a.padded && len[j] > a.W) err |= DNATOK_DERR_ROW_WIDTH;
        }
        mine += len[j];
    }
    int64_t total;
    const int64_t pre = dev::block_excl_scan<kScanNT>(mine, s_tmp, &total);
    int64_t run = a.base + prefix(total) + pre;
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        const int64_t i = i0 + j;
        if (i < a.n) a.out_offs[i] = run;
        run += len[j];
    }
    return total;
}

// Length in tokens of a row, and the flags its offsets raise.
struct RowLen {
    const int64_t *offs;
    int64_t nbytes;
    int32_t n;
    int32_t k;
    uint32_t kinv;
    int32_t kmer, overlap, cls;
    int64_t W;  // PADDED: the widest row (INT64_MAX otherwise)
    __device__ __forceinline__ int64_t of(int64_t o0, int64_t o1, uint32_t &err) const {
        if (o0 < 0 || o1 < o0 || o1 > nbytes) err |= DNATOK_DERR_OFFSETS;
        o0 = o0 < 0 ? 0 : (o0 > nbytes ? nbytes : o0);
        o1 = o1 < o0 ? o0 : (o1 > nbytes ? nbytes : o1);
        const int64_t L = o1 - o0;
        int64_t nb = L;
        if (kmer) nb = overlap ? (L >= k ? L - k + 1 : (L > 0 ? 1 : 0)) : div_k(L + k - 1, k, kinv);
        if (kmer == 2 && nb == 0) nb = 1;
        const int64_t l = nb + 2 * cls;
        if (l > W) err |= DNATOK_DERR_ROW_WIDTH;
        return l;
    }
    __device__ __forceinline__ int64_t len(int64_t i, uint32_t &err) const { return of(offs[i], offs[i + 1], err); }
};

// Offsets of the kScanRows rows of one unit by one workgroup that no other
// waits for: it adds up the rows before the unit itself (eight in flight per
// thread) instead of taking the sum over from its predecessors. A batch of a
// few thousand rows is bound by the latency of its dependent steps, and this
// form has three (offsets, block scan, stores): 3,001 rows take 5.4 us,
// where the chained units with their ticket and look-back took 10.4. The
// reads grow with the square of the rows (8 MB at 65,536). In a launch of its
// own it is the shorter form up to kIndependentMaxRows: PACKED encodes of rows
// of about 1,000 bases, this way / chained, in us, single-nucleotide and 6-mer
// ids: 8,192 rows 18.4 / 22.8 and 19.3 / 22.5, 16,384 31.6 / 32.4 and 27.6 /
// 25.1, 65,536 107 / 84 and 80 / 43. In front of the workgroups of an encode
// or a lookup, which hide it, up to kFusedScanRows: 16,384 rows as 6-mers
// PADDED 16.9, by a launch of its own 25.7; 65,536 49.6 and 50.3.
constexpr int kScanRows = 1024;
constexpr int kScanRowsPerThread = kScanRows / kScanNT;
constexpr int32_t kIndependentMaxRows = 12288;
constexpr int32_t kFusedScanRows = 65536;
[[maybe_unused]] __host__ __device__ inline int64_t rowscan_units(int64_t n) {
    return n > 0 ? (n + kScanRows - 1) / kScanRows : 1;
}
[[maybe_unused]] __device__ __forceinline__ void rowscan_independent(const RowLen &rl, int64_t *out, int64_t base,
                                                                     int64_t unit, int64_t *s_tmp, uint32_t *err_hdr) {
    const int tid = threadIdx.x;
    const int64_t row0 = unit * kScanRows, n = rl.n;
    uint32_t err = 0, ignore = 0;  // each unit reports its own rows
    // this unit's offsets and the rows before it are asked for together
    int64_t off[kScanRowsPerThread + 1];
    const int64_t i0 = row0 + (int64_t)tid * kScanRowsPerThread;
#pragma unroll
    for (int j = 0; j <= kScanRowsPerThread; ++j) off[j] = rl.offs[min(i0 + j, n)];
    int64_t before = 0;
    for (int64_t r = tid; r < row0; r += 8 * kScanNT) {
        int64_t x[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = min(r + u * kScanNT, row0 - 1);
            x[u] = rl.offs[i];
            y[u] = rl.offs[i + 1];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (r + u * kScanNT < row0) before += rl.of(x[u], y[u], ignore);
    }
    int64_t len[kScanRowsPerThread], mine = 0;
#pragma unroll
    for (int j = 0; j < kScanRowsPerThread; ++j) {
        len[j] = i0 + j < n ? rl.of(off[j], off[j + 1], err) : 0;
        mine += len[j];
    }
    int64_t total;
    int64_t run = base + dev::block_excl_scan<kScanNT>(mine, s_tmp, &total);
    if (row0 > 0) run += dev::block_sum<kScanNT>(before, s_tmp);
#pragma unroll
    for (int j = 0; j < kScanRowsPerThread; ++j) {
        if (i0 + j < n) out[i0 + j] = run;
        run += len[j];
        // the last row's owner (or, without rows, the first thread) ends the offsets
        if (i0 + j == n - 1 || (n == 0 && tid == 0 && j == 0)) out[n] = run;
    }
    if (err) dev::raise_error(err_hdr, err);
}

}  // namespace

}  // namespace dnatok
