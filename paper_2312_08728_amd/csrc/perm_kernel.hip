// Device-side seeded partition of a buffer into mini-batches.
//
// Algorithm 1 draws a fresh random partition of the buffer at the start of every pass; Section 2.2
// asks for disjoint parts that cover the buffer.  The generator (perm_device.h) is integer arithmetic only, so that the
// index arrays are reproducible bit for bit.  Mini-batch m is perm[(m-1) n : min(m n, rows)).
#include "perm_device.h"

#include <algorithm>

namespace bmgd {

namespace {

// With `subset` the partition is one of the rows subset[0 .. rows) of a larger buffer: out holds subset[PERM[j]].
// An entry outside [0, limit) is replaced by row 0 and reported through *bad (the host turns that into an error).
__global__ void __launch_bounds__(256) perm_kernel(int32_t* __restrict__ out, uint32_t rows, uint32_t h,
                                                   PermKeys keys, const int32_t* __restrict__ subset, uint32_t limit,
                                                   unsigned* bad)
{
    const uint32_t pass = blockIdx.y;
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= rows) return;
    KeyRow key;
#pragma unroll
    for (int i = 0; i < kPermRounds; ++i) key.k[i] = keys.key[pass][i];
    uint32_t x = perm_entry(j, key, h, rows);
    if (subset) {
        const uint32_t v = (uint32_t)subset[x];
        if (v >= limit) __hip_atomic_store(bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = v < limit ? v : 0u;
    }
    out[(size_t)pass * rows + j] = (int32_t)x;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint4* __restrict__ dst, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = make_uint4(0, 0, 0, 0);
}

// avg <- theta for the first snapshot, else avg + (theta - avg) * inv with inv = 1 / (snapshots so far + 1)
__global__ void __launch_bounds__(256) running_mean_kernel(float* __restrict__ avg, const float* __restrict__ theta, size_t n,
                                                           float inv, int first)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float t = theta[i];
        avg[i] = first ? t : avg[i] + (t - avg[i]) * inv;
    }
}

// Rows of C values out of rows of ld, packed, and the two words of failure flags, into host memory the device can write:
// dst[i] = src[(row0 + i / C) ld + i % C].  Bound by the link (3,072 rows of 1,000 floats, in 1 MB parts: 0.7 ms with the copies on the host).
__global__ void __launch_bounds__(256) export_kernel(float* __restrict__ dst, const float* __restrict__ src, unsigned row0, unsigned C,
                                                     unsigned ld, unsigned count, unsigned* __restrict__ flags_out,
                                                     const unsigned* __restrict__ flags)
{
    if (blockIdx.x == 0 && threadIdx.x < 2) flags_out[threadIdx.x] = flags[threadIdx.x];
    const unsigned stride = gridDim.x * blockDim.x;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const unsigned r = i / C;
        dst[i] = src[(size_t)(row0 + r) * ld + (i - r * C)];
    }
}

// The other way: dst[(row0 + i / C) ld + i % C] = src[i].
__global__ void __launch_bounds__(256) import_kernel(float* __restrict__ dst, const float* __restrict__ src, unsigned row0, unsigned C,
                                                     unsigned ld, unsigned count)
{
    const unsigned stride = gridDim.x * blockDim.x;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const unsigned r = i / C;
        dst[(size_t)(row0 + r) * ld + (i - r * C)] = src[i];
    }
}

}  // namespace

hipError_t launch_export(float* dst, const float* src, int64_t row0, int64_t rows, int64_t C, int64_t ld, unsigned* flags_out,
                         const unsigned* flags, hipStream_t stream)
{
    const unsigned count = (unsigned)(rows * C);
    const unsigned blocks = std::max(1u, std::min((count + 255) / 256, 1024u));
    hipLaunchKernelGGL(export_kernel, dim3(blocks), dim3(256), 0, stream, dst, src, (unsigned)row0, (unsigned)std::max<int64_t>(C, 1),
                       (unsigned)ld, count, flags_out, flags);
    return hipGetLastError();
}

hipError_t launch_import(float* dst, const float* src, int64_t row0, int64_t rows, int64_t C, int64_t ld, hipStream_t stream)
{
    const unsigned count = (unsigned)(rows * C);
    if (count == 0) return hipSuccess;
    const unsigned blocks = std::min((count + 255) / 256, 1024u);
    hipLaunchKernelGGL(import_kernel, dim3(blocks), dim3(256), 0, stream, dst, src, (unsigned)row0, (unsigned)C, (unsigned)ld, count);
    return hipGetLastError();
}

hipError_t launch_running_mean(float* avg, const float* theta, size_t n, float inv, bool first, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(running_mean_kernel, dim3(blocks), dim3(256), 0, stream, avg, theta, n, inv, first ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void* dst, size_t bytes, hipStream_t stream)
{
    if (bytes == 0) return hipSuccess;
    if ((reinterpret_cast<uintptr_t>(dst) % 16) != 0 || bytes % 16 != 0) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16;
    const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 2048);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<uint4*>(dst), n16);
    return hipGetLastError();
}

void perm_round_keys(uint64_t seed, uint32_t b, uint32_t t, uint32_t out[kPermRounds])
{
    uint32_t a = mix32((uint32_t)(seed & 0xFFFFFFFFu) ^ 0x9E3779B9u);
    a = mix32(a ^ (uint32_t)(seed >> 32));
    a = mix32(a + b);
    a = mix32(a ^ t);
    for (int i = 0; i < kPermRounds; ++i) out[i] = mix32(a + (uint32_t)i * 0x9E3779B9u);
}

int perm_half_width(int64_t rows)
{
    int bits = 0;
    for (uint64_t v = (uint64_t)(rows - 1); v != 0; v >>= 1) ++bits;
    const int h = (bits + 1) / 2;
    return h < 1 ? 1 : h;
}

hipError_t launch_perm(int32_t* out, int64_t rows, int npass, const PermKeys& keys, hipStream_t stream, const int32_t* subset,
                       int64_t limit, unsigned* bad)
{
    if (rows <= 0 || npass <= 0) return hipSuccess;
    if (npass > kMaxPassesPerLaunch || rows > (int64_t(1) << 30)) return hipErrorInvalidValue;
    if (subset && (!bad || limit < rows || limit > (int64_t(1) << 30))) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((rows + 255) / 256), (unsigned)npass);
    hipLaunchKernelGGL(perm_kernel, grid, dim3(256), 0, stream, out, (uint32_t)rows,
                       (uint32_t)perm_half_width(rows), keys, subset, (uint32_t)limit, bad);
    return hipGetLastError();
}

}  // namespace bmgd
