// Device lookup of a symbol pair's merge rank, shared by the BPE kernels.
#pragma once

#include "common.hpp"
#include "device.hpp"

namespace dnatok {

namespace {

struct RankTab {
    const uint4 *bucket;
    const uint32_t *pair;
    uint32_t nbk;
};

// Rank of the pair (a, b), or kNoRank. Specials and N never merge.
__device__ __forceinline__ uint32_t pair_rank(const RankTab &t, uint32_t a, uint32_t b) {
    if (a < 5 || a == 9 || b < 5 || b == 9) return kNoRank;
    const uint32_t key = a | (b << 16);
    uint32_t b1, b2;
    bpe_buckets(key, t.nbk, &b1, &b2);
    const uint4 x = t.bucket[b1], y = t.bucket[b2];
    uint32_t r = kNoRank;
    r = (x.x == key) ? x.y : r;
    r = (x.z == key) ? x.w : r;
    r = (y.x == key) ? y.y : r;
    r = (y.z == key) ? y.w : r;
    return r;
}

using dev::wave_sync;

}  // namespace

}  // namespace dnatok
