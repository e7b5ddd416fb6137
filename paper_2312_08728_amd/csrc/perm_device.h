// The generator of the seeded partitions, for the kernel that writes them out (perm_kernel.hip) and those that work out the entries they
// need (gram_fused_kernel.hip, gram_direct_kernel in gram_kernels.hip): a keyed 8-round balanced Feistel network on 2 h bits
// (2^(2h) < 4 * rows) restricted to [0, rows) by cycle walking, in uint32 arithmetic only.
#pragma once

#include "bmgd_internal.h"

namespace bmgd {
namespace {

__host__ __device__ inline uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}

struct KeyRow {
    uint32_t k[kPermRounds];
};

__device__ inline uint32_t feistel(uint32_t x, const KeyRow& key, uint32_t h, uint32_t mask)
{
    uint32_t left = x >> h, right = x & mask;
#pragma unroll
    for (int i = 0; i < kPermRounds; ++i) {
        const uint32_t f = mix32(right ^ key.k[i]) & mask;
        const uint32_t t = left ^ f;
        left = right;
        right = t;
    }
    return (left << h) | right;
}

// Entry j < rows of the partition: j lies on a cycle of the bijection that returns to j, so the walk always re-enters [0, rows).
__device__ inline uint32_t perm_entry(uint32_t j, const KeyRow& key, uint32_t h, uint32_t rows)
{
    const uint32_t mask = (1u << h) - 1u;
    uint32_t x = feistel(j, key, h, mask);
    while (x >= rows) x = feistel(x, key, h, mask);
    return x;
}

}  // namespace
}  // namespace bmgd
