// Row scan of a ragged batch (token counts per row to output offsets), the
// tile size of an encode, and its dispatch to the wave-tile kernel.
//
// Every row's token count has a closed form (L, ceil(L/k) or L - k + 1, plus
// 2 with CLS/SEP), so out_offsets is a scan over rows: up to 12,288 rows by
// workgroups that do not wait for each other (k_rowscan_units), longer
// batches in units of 4,096 rows handed out by ticket and chained with a
// decoupled look-back (k_rowscan).
#include "common.hpp"
#include "device.hpp"
#include "rowscan.hpp"

namespace dnatok {

namespace {

constexpr int NT = 256;
static_assert(NT == kScanNT, "the row scan's block size");

__global__ __launch_bounds__(NT) void k_rowscan(RowScanArgs a) {
    __shared__ int64_t s_tmp[NT / dev::kWave + 1];
    __shared__ int64_t s_unit, s_excl;
    const int tid = threadIdx.x;
    const uint32_t parity = dev::ld_relaxed32(a.q.hdr + 2);
    uint64_t *st = parity ? a.q.status1 : a.q.status0;
    uint64_t *st_other = parity ? a.q.status0 : a.q.status1;
    uint32_t err = 0;
    for (;;) {
        if (tid == 0) s_unit = (int64_t)atomicAdd(a.q.hdr + 0, 1u);
        __syncthreads();
        const int64_t u = s_unit;
        __syncthreads();
        if (u >= a.nunits) break;
        for (int64_t j = u + (int64_t)tid * a.nunits; j < a.q.clear_n; j += (int64_t)NT * a.nunits) st_other[j] = 0;
        // Unit prefix through the decoupled look-back over units (wave 0).
        const int64_t total = rowscan_unit(a, u * kUnitRows, s_tmp, err, [&](int64_t tot) {
            if (threadIdx.x < dev::kWave) {
                if (threadIdx.x == 0) dev::publish_aggregate(st, u, tot);
                const int64_t ex = dev::wave_lookback(st, u, tot, a.q.hdr);
                if (threadIdx.x == 0) s_excl = ex;
            }
            __syncthreads();
            return s_excl;
        });
        if (u == a.nunits - 1 && tid == 0) a.out_offs[a.n] = a.base + s_excl + total;
        __syncthreads();
    }
    if (err) dev::raise_error(a.q.hdr, err);
    if (tid == 0) dev::finish_block(a.q.hdr);
}

}  // namespace

namespace {
struct IndependentArgs {
    RowLen rl;
    int64_t *out;
    int64_t base;
    uint32_t *hdr;
};
__global__ __launch_bounds__(NT) void k_rowscan_units(IndependentArgs a) {
    __shared__ int64_t s_tmp[NT / dev::kWave + 1];
    rowscan_independent(a.rl, a.out, a.base, blockIdx.x, s_tmp, a.hdr);
}
}  // namespace

int launch_rowscan_spec(const RowScanSpec &sp, hipStream_t stream) {
    RowScanArgs s;
    s.offs = sp.offs;
    s.n = sp.n;
    s.nbytes = sp.nbytes;
    s.out_offs = sp.out;
    s.k = sp.k > 0 ? sp.k : 1;
    s.kinv = 0xFFFFFFFFu / (uint32_t)s.k;
    s.kmer = sp.kmer;
    s.overlap = sp.overlap;
    s.cls = sp.cls;
    s.padded = sp.padded;
    s.W = sp.W;
    s.base = sp.base;
    s.nunits = ((int64_t)sp.n + kUnitRows - 1) / kUnitRows;
    if (s.nunits < 1) s.nunits = 1;
    Workspace *ws = nullptr;
    int rc = get_workspace(stream, s.nunits, &ws);
    if (rc) return rc;
    if (sp.n <= kIndependentMaxRows) {
        IndependentArgs ia{RowLen{sp.offs, sp.nbytes, sp.n, s.k, s.kinv, sp.kmer, sp.overlap, sp.cls,
                                  sp.padded ? sp.W : INT64_MAX},
                           sp.out, sp.base, ws->d_hdr};
        hipLaunchKernelGGL(k_rowscan_units, dim3((unsigned)rowscan_units(sp.n)), dim3(NT), 0, stream, ia);
        DNATOK_HIP(hipGetLastError());
        return DNATOK_OK;
    }
    s.q.hdr = ws->d_hdr;
    s.q.status0 = ws->d_status;
    s.q.status1 = ws->d_status + ws->cap;
    if (s.nunits > ws->high_water) ws->high_water = s.nunits;
    s.q.clear_n = ws->high_water;
    int per_cu = 0;
    DNATOK_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rowscan, NT, 0));
    int64_t g = (int64_t)device_cu_count() * (per_cu > 0 ? per_cu : 1);
    if (g > s.nunits) g = s.nunits;
    hipLaunchKernelGGL(k_rowscan, dim3((unsigned)g), dim3(NT), 0, stream, s);
    DNATOK_HIP(hipGetLastError());
    return DNATOK_OK;
}

int launch_rowscan(const int64_t *d_offsets, int32_t n, int64_t nbytes, int64_t *d_out, int32_t divisor, int32_t cls,
                   hipStream_t stream, bool at_least_one) {
    RowScanSpec sp;
    sp.offs = d_offsets;
    sp.n = n;
    sp.nbytes = nbytes;
    sp.out = d_out;
    sp.k = divisor;
    sp.kmer = at_least_one ? 2 : 1;
    sp.overlap = 0;
    sp.cls = cls;
    sp.padded = 0;
    sp.W = 0;
    sp.base = 0;
    return launch_rowscan_spec(sp, stream);
}

// Input bytes a workgroup of the wave-tile kernel takes (4 KiB times a power
// of two up to 8; a wave has a quarter of them, with several vocabularies the
// workgroup shares them). Untuned: about 2,048 output cells per wave, halved
// while the batch gives a CU fewer than two workgroups. Measured, in us at
// 4 / 8 / 16 / 32 KiB on 4,096 x 8,192 bases: single-nucleotide ids 42 / 40 /
// 42 / 40, overlapping 6-mers 57 / 43 / 49 / 46, 6-mers 37 / 25 / 17 / 16,
// k = 3..6 in one pass 54 / 42 / 47 / 49.
int64_t encode_tile_bytes(const dnatok_vocab *v, int64_t nbytes, int nv, int32_t variant) {
    const int32_t tile = v->tune_tile.load(std::memory_order_relaxed);
    if (tile > 0) return tile;
    const bool frames = v->kind == DNATOK_KMER && !(variant & DNATOK_VARIANT_OVERLAP);
    int64_t want = nv > 1 || !frames || v->k < 2 ? 8192 : v->k < 3 ? 16384 : 32768;
    const int64_t target = nbytes / (2 * (int64_t)device_cu_count());
    while (want > 4096 && want > target) want >>= 1;
    return want;
}

int launch_encode_multi(const dnatok_vocab *const *vs, int nv, const uint8_t *d_bytes, int64_t nbytes,
                        const int64_t *d_offsets, int32_t n, int32_t *const *d_ids, const int64_t *caps,
                        int64_t *const *d_out_offsets, int8_t *const *d_masks, const dnatok_encode_opts *os,
                        hipStream_t stream) {
    return launch_encode_rows(vs, nv, d_bytes, nbytes, d_offsets, n, d_ids, caps, d_out_offsets, d_masks, os,
                              encode_tile_bytes(vs[0], nbytes, nv, os[0].variant), stream);
}

int launch_encode(const dnatok_vocab *v, const uint8_t *d_bytes, int64_t nbytes, const int64_t *d_offsets,
                  int32_t n, int32_t *d_ids, int64_t cap, int64_t *d_out_offsets, int8_t *d_mask,
                  const dnatok_encode_opts &o, hipStream_t stream) {
    return launch_encode_multi(&v, 1, d_bytes, nbytes, d_offsets, n, &d_ids, &cap, &d_out_offsets, &d_mask, &o,
                               stream);
}

}  // namespace dnatok
