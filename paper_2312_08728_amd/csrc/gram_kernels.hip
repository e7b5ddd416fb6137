// Least squares with few features: the update in its linear-system form.
//
// For the squared loss the mini-batch update of eq. (2.1) is eq. (3.1):
//     theta <- (I - alpha Sxx_m) theta + alpha Sxy_m,   Sxx_m = n_b^-1 sum x x',  Sxy_m = n_b^-1 sum x y
// over the rows of mini-batch m.  Sxx_m and Sxy_m do not depend on theta, so when p is small (p^2 << n p)
// they are formed for every mini-batch of a pass by a fully parallel pre-pass over the buffer -- a dense
// contraction [X y]' [X y] per mini-batch, on the matrix cores in fp32 -- and the strictly sequential chain
// then costs p^2 multiply-adds and 4 p^2 bytes per step inside ONE workgroup: no exchange between workgroups
// at all.  Same arithmetic as the row form up to the order of summation.
#include "bmgd_internal.h"
#include "gram_chain.h"
#include "lds_load.h"
#include "perm_device.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <utility>

namespace bmgd {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct GramTiles {
    int ntiles;                     // upper-triangle 16 x 16 tiles of the (p + 1) x (p + 1) moment matrix
    int tsplit;                     // workgroups per mini-batch; each takes TPW consecutive entries of `tile`
    unsigned short tile[48];        // I | J << 8, I <= J; padding entries repeat tile 0 and are not written out
};

constexpr int kRowsPerChunk = 16;   // rows staged per wavefront at a time: four K = 4 matrix instructions
constexpr int kGramWaves = 4;

// Moment matrices of one mini-batch (one pass): the wavefronts take 16-row chunks in turn and accumulate
// their TPW tiles of [X y]' [X y]; the four partial sums meet in LDS, are divided by n_b and written in the
// chain's layout (both triangles).  MFMA operand layout (v_mfma_f32_16x16x4_f32): a = A[lane % 16][lane / 16],
// b = B[lane / 16][lane % 16], c[v] = C[4 (lane / 16) + v][lane % 16]; here A = (staged rows)' and B = staged rows.
// VEC: p is a multiple of 4 and rows are moved as float4 (a quarter of the load, address and store instructions; the
// kernel is bound by instruction issue, not by any one unit).
template <int TPW, bool WIDE, bool VEC>
__global__ void __launch_bounds__(64 * kGramWaves) gram_mfma_kernel(const float* __restrict__ X, const float* __restrict__ y,
                                                                     const int* __restrict__ perm, float* __restrict__ out,
                                                                     int rows, int n, int perm_stride, int M, int n_items,
                                                                     int stride, GramLayout L, GramTiles T, int dense_q)
{
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Workgroups go to the eight XCDs in turn (blockIdx % 8), each with an L2 of its own: the tsplit workgroups
    // that read the same mini-batch are consecutive on one XCD, so all but the first find its rows in that L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int part = slot % T.tsplit;
    const int mb = (slot / T.tsplit) * 8 + xcd;
    if (mb >= n_items) return;
    const int m = mb % M, pass = mb / M;
    const int p = L.p;
    const int nb = min(n, rows - m * n);
    const int* idx = perm + (size_t)pass * perm_stride + (size_t)m * n;
    float* xs = lds + wave * kRowsPerChunk * stride;             // this wavefront's staging area
    constexpr int CL = WIDE ? 2 : 1;                              // 64-column groups of a row

    for (int e = lane; e < kRowsPerChunk * stride; e += 64) xs[e] = 0.f;   // padding columns stay zero

    int tI[TPW], tJ[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int g = part * TPW + t;
        const unsigned short code = T.tile[g < T.ntiles ? g : 0];
        tI[t] = 16 * (code & 0xFF);
        tJ[t] = 16 * (code >> 8);
    }
    floatx4 acc[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int nchunks = (nb + kRowsPerChunk - 1) / kRowsPerChunk;
    float v[kRowsPerChunk][CL];                      // (not VEC)
    float yv = 0.f;
    // VEC: the 16 * p / 4 float4 of a chunk are dealt to the lanes in turn; which row and which columns lane l's i-th
    // float4 belongs to does not change from chunk to chunk
    constexpr int NV = WIDE ? 8 : 4;                 // float4 per lane and chunk: 16 * (p / 4) / 64 rounded up for the largest p
    float4 v4[VEC ? NV : 1];
    int vrow[VEC ? NV : 1], vcol[VEC ? NV : 1];      // row of the chunk (as a byte offset of its lane for the shuffle), first column
    if constexpr (VEC) {
        const int p4 = p >> 2;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int e = min(lane + 64 * i, kRowsPerChunk * p4 - 1);    // (beyond the chunk: the last float4 again, same value)
            const int r = e / p4;
            vrow[i] = r;
            vcol[i] = 4 * (e - r * p4);
        }
    }
    auto request = [&](int chunk) {
        if constexpr (VEC) {
            const int i = min(chunk * kRowsPerChunk + (lane & 15), nb - 1);
            const int row = idx[i];
            yv = y[row];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int rr = __builtin_amdgcn_ds_bpermute(4 * vrow[q], row);   // the row index held by lane vrow[q]
                v4[q] = *reinterpret_cast<const float4*>(X + (size_t)rr * p + vcol[q]);
            }
        } else {
            // unconditional loads from clamped rows and columns; what lies outside the mini-batch is zeroed on use
            const int i = min(chunk * kRowsPerChunk + (lane & 15), nb - 1);
            const int row = idx[i];
            yv = y[row];
#pragma unroll
            for (int r = 0; r < kRowsPerChunk; ++r) {
                const int rr = __builtin_amdgcn_readlane(row, r);
                const float* src = X + (size_t)rr * p;
#pragma unroll
                for (int j = 0; j < CL; ++j) v[r][j] = src[min(lane + 64 * j, p - 1)];
            }
        }
    };
    auto stage = [&](int chunk) {
        const int left = nb - chunk * kRowsPerChunk;              // rows of this chunk inside the mini-batch
        if constexpr (VEC) {
            if (left < kRowsPerChunk) {                           // (uniform) the last chunk: rows beyond the mini-batch are zeroed
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    if (vrow[q] >= left) v4[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int q = 0; q < NV; ++q) *reinterpret_cast<float4*>(xs + vrow[q] * stride + vcol[q]) = v4[q];
            __builtin_amdgcn_wave_barrier();
            if (lane < kRowsPerChunk) xs[lane * stride + p] = lane < left ? yv : 0.f;
        } else {
#pragma unroll
            for (int r = 0; r < kRowsPerChunk; ++r) {
#pragma unroll
                for (int j = 0; j < CL; ++j) {
                    // no branch: lanes beyond p write a zero into a padding column (or into the column of y, which
                    // the store below then overwrites)
                    const int c = lane + 64 * j;
                    xs[r * stride + min(c, stride - 1)] = (c < p && r < left) ? v[r][j] : 0.f;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (lane < kRowsPerChunk) xs[lane * stride + p] = lane < left ? yv : 0.f;
        }
    };

    if (wave < nchunks) request(wave);
    for (int chunk = wave; chunk < nchunks; chunk += kGramWaves) {
        __builtin_amdgcn_wave_barrier();
        stage(chunk);
        __builtin_amdgcn_wave_barrier();
        if (chunk + kGramWaves < nchunks) request(chunk + kGramWaves);
#pragma unroll
        for (int kk = 0; kk < kRowsPerChunk / 4; ++kk) {
            const float* rowp = xs + (4 * kk + (lane >> 4)) * stride + (lane & 15);
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const float a = rowp[tI[t]];
                const float b = rowp[tJ[t]];
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[t], 0, 0, 0);
            }
        }
    }

    // sum over the wavefronts, scale, write out
    __syncthreads();
    floatx4* red = reinterpret_cast<floatx4*>(lds);               // [wave][TPW][64]
#pragma unroll
    for (int t = 0; t < TPW; ++t) red[(wave * TPW + t) * 64 + lane] = acc[t];
    __syncthreads();
    const float inv = 1.f / (float)nb;
    // dense_q > 0: the matrix [Sxx_m | -Sxy_m] goes out dense, row-major with row stride dense_q, for the kernel that
    // multiplies steps together (gram_products.hip); rows and columns beyond it are never written (they stay zero)
    float* o = out + (size_t)(pass * M + m) * (dense_q > 0 ? (size_t)dense_q * dense_q : (size_t)L.step_floats);
    const int my_tiles = min(TPW, T.ntiles - part * TPW);
    for (int t = wave; t < my_tiles; t += kGramWaves) {
        floatx4 s = red[t * 64 + lane];
#pragma unroll
        for (int w = 1; w < kGramWaves; ++w) s += red[(w * TPW + t) * 64 + lane];
        const unsigned short code = T.tile[part * TPW + t];
        const int I = 16 * (code & 0xFF), J = 16 * (code >> 8);
        const int c = J + (lane & 15);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = I + 4 * (lane >> 4) + q;
            const float val = s[q] * inv;
            if (dense_q > 0) {
                if (r < p && c < p) {
                    o[r * dense_q + c] = val;
                    if (I != J) o[c * dense_q + r] = val;
                } else if (r < p && c == p) {
                    o[r * dense_q + p] = -val;
                }
            } else if (r < p && c < p) {
                o[gram_pos(L, r, c)] = val;
                if (I != J) o[gram_pos(L, c, r)] = val;
            } else if (r < p && c == p) {
                o[L.b_off + r] = val;
            }
        }
    }
}

template <int TPR, int KQ, int KS, int AHEAD, bool TAB, int RULE>
__global__ void __launch_bounds__(1024) gram_chain_kernel(const float* __restrict__ gram, float* __restrict__ theta,
                                                          GramLayout L, int nsteps, int period, float alpha,
                                                          const float* __restrict__ lr_tab, int lr_base, int lr_len, OptArgs opt)
{
    gram_chain_steps<TPR, KQ, KS, AHEAD, TAB ? kRateTable : kRateConstant, RULE>(gram, theta, L, nsteps, period, alpha, lr_tab, lr_base,
                                                                                 lr_len, nullptr, opt);
}

// The same matrices with the rows gathered straight into matrix operands, for up to 47 features and 64 mini-batches a pass or more.
//
// With A = rows' and B = rows a lane's element of both operands is the same, so 16 columns of four rows are one load per lane and serve a
// whole row and column of tiles: no way through shared memory, and a wavefront keeps ALL tiles of its rows' matrix in registers.  What
// bounds it is the gather of short rows.  A mini-batch may be split over S = 2 workgroups by rows (direct_split), so that a few long ones fill
// the device too; the second of two workgroups to finish adds the first one's sums, which it finds where the result goes (a + b = b + a: the
// same bits whichever comes first).  Rows are requested one stage (U groups of four rows) ahead.  The entries of the partition are worked
// out here, 64 at a time per wavefront: the partition's own kernel and what lies behind it are 10 to 16 us per buffer.
// us per buffer of three passes, products behind it, staged kernel with partitions from memory / this one (p, n, mini-batches): 143 / 78
// (5, 5000, 128), 111 / 98 (10, 20, 511), 127 / 115 (20, 300, 511), 79 / 75 (20, 1000, 256), 285 / 208 (20, 5000, 256), 80 / 72 (33, 1500,
// 128), 95 / 97 (33, 300, 256), 93 / 91 (40, 80, 256), 104 / 101 (47, 94, 256), 138 / 108 (47, 3000, 128).  Not with more features: from
// five tile rows on its loads and matrix instructions do not overlap as they should (p = 64: 53 / 86 us of kernel, p = 100: 90 / 136); four
// tile rows (p = 48 to 63) were not built.
struct DirectArgs {
    const float* X;
    const float* y;
    PermKeys keys;
    uint32_t h;
    const int32_t* subset;
    uint32_t limit;
    unsigned* bad;
    float* out;
    unsigned* tickets;                               // S = 2: [n_items][2][kDirectWaves], zero between launches
    GramLayout L;
    int rows, n, M, dense_q, n_items;
    const int32_t* perm;                             // (gram_rows_kernel)
    int perm_stride;
};

constexpr int kDirectWaves = 4, kSumTiles = 16;

// The end of a workgroup of either moments kernel: its TPW tiles from number t_first on (group h of the mini-batch's tiles), summed over
// its four wavefronts, joined with the other workgroup's (S = 2), scaled and written.  lds: two KB for each of the tiles summed at a time.
template <int NT, int TPW, int S>
__device__ __forceinline__ void finish_tiles(const DirectArgs& a, floatx4 (&acc)[TPW], int t_first, int h, float* lds, int item, int nb, int wave, int lane)
{
    constexpr int TILES = NT * (NT + 1) / 2;
    const int p = a.L.p, i16 = lane & 15, quad = lane >> 4;
    // the four wavefronts' sums: two halves through shared memory, then every wavefront a quarter of the tiles; as many tiles at a time as
    // kSumTiles says
    constexpr int MINE = (TPW + kDirectWaves - 1) / kDirectWaves, PART = TPW < kSumTiles ? TPW : kSumTiles;
    floatx4* red = reinterpret_cast<floatx4*>(lds);
    float s[MINE][4];
    int tI[MINE], tJ[MINE];
#pragma unroll
    for (int t0 = 0; t0 < TPW; t0 += kSumTiles) {
        if (t0 > 0) __syncthreads();
        if (wave >= 2) {
#pragma unroll
            for (int t = t0; t < TPW && t < t0 + PART; ++t) red[((wave - 2) * PART + t - t0) * 64 + lane] = acc[t];
        }
        __syncthreads();
        if (wave < 2) {
#pragma unroll
            for (int t = t0; t < TPW && t < t0 + PART; ++t) {
                acc[t] += red[(wave * PART + t - t0) * 64 + lane];
                red[(wave * PART + t - t0) * 64 + lane] = acc[t];
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = t0 / kDirectWaves; q < MINE && q < (t0 + kSumTiles) / kDirectWaves; ++q) {
            const int i = min(q * kDirectWaves + wave, TPW - 1), t = min(t_first + i, TILES - 1);
            const floatx4 v = red[(i - t0) * 64 + lane] + red[(PART + i - t0) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[q][e] = v[e];
            int I = 0, first = 0;                    // tile t is (I, J): rows of tiles have NT, NT - 1, ... entries
#pragma unroll
            for (int k = 0; k < NT - 1; ++k)
                if (t - first >= NT - I) { first += NT - I; ++I; }
            tI[q] = 16 * I;
            tJ[q] = 16 * (I + t - first);
        }
    }
    float* o = a.out + (size_t)item * (a.dense_q > 0 ? (size_t)a.dense_q * a.dense_q : (size_t)a.L.step_floats);
    auto where = [&](int r, int c) { return a.dense_q > 0 ? r * a.dense_q + c : c == p ? a.L.b_off + r : gram_pos(a.L, r, c); };
    auto each = [&](auto&& f) {
#pragma unroll
        for (int q = 0; q < MINE; ++q) {
            const int c = tJ[q] + i16;
            const bool here = q * kDirectWaves + wave < TPW && t_first + q * kDirectWaves + wave < TILES && c <= p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = tI[q] + 4 * quad + e;
                if (here && r < p) f(q, e, r, c);
            }
        }
    };
    const float inv = 1.f / (float)nb;
    const __amdgpu_buffer_rsrc_t ob = __builtin_amdgcn_make_buffer_rsrc(o, 0, (int)((a.dense_q > 0 ? a.dense_q * a.dense_q : a.L.step_floats) * 4), 0x00020000);
    constexpr int kAgent = 0x10;                     // cache policy sc1: past this die's cache
    if constexpr (S == 2) {
        // Per wavefront, group of tiles and mini-batch a word: arrivals add 1, who comes first leaves its sums and then adds kLeft; who comes
        // second (the first one is past its arrival and waits for nothing, so this wait ends) adds them to its own and clears the word.
        constexpr unsigned kLeft = 4;
        unsigned* ticket = a.tickets + (item * 2 + h) * kDirectWaves + wave;
        unsigned order = 0u;
        if (lane == 0) order = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        order = (unsigned)__builtin_amdgcn_readfirstlane((int)order);
        if (order == 0u) {
            each([&](int q, int e, int r, int c) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, s[q][e]), ob, (unsigned)where(r, c) * 4u, 0, kAgent); });
            __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
            asm volatile("" ::: "memory");
            if (lane == 0) __hip_atomic_fetch_add(ticket, kLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        while (__hip_atomic_load(ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < kLeft) __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
        float other[MINE][4];
        each([&](int q, int e, int r, int c) { other[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ob, (unsigned)where(r, c) * 4u, 0, kAgent)); });
        each([&](int q, int e, int, int) { s[q][e] += other[q][e]; });
        if (lane == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // (written past this die's cache as well: a plain store could leave one behind it that the other workgroup's sums would be merged into)
    each([&](int q, int e, int r, int c) {
        const float val = s[q][e] * inv;
        const float put = c == p && a.dense_q > 0 ? -val : val;   // dense: [Sxx | -Sxy], for the kernel that multiplies steps together
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, put), ob, (unsigned)where(r, c) * 4u, 0, S == 2 ? kAgent : 0);
        if (tI[q] != tJ[q] && c < p)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, val), ob, (unsigned)where(c, r) * 4u, 0, S == 2 ? kAgent : 0);
    });
}

template <int NT, int S>
__global__ void __launch_bounds__(64 * kDirectWaves, 2) gram_direct_kernel(DirectArgs a)
{
    constexpr int TILES = NT * (NT + 1) / 2;
    constexpr int U = 8;                             // groups of four rows per stage
    constexpr int STAGES = 64 / (4 * U);             // stages per 64 entries of the partition
    __shared__ __align__(16) float lds[2 * TILES * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int item = blockIdx.x / S, part = blockIdx.x % S;
    const int pass = item / a.M, m = item - pass * a.M;
    const int p = a.L.p;
    const int nb = min(a.n, a.rows - m * a.n);
    const int i16 = lane & 15, quad = lane >> 4;
    // this wavefront's rows: whole groups of four, one share of S * kDirectWaves
    const int share = (nb + 4 * S * kDirectWaves - 1) / (4 * S * kDirectWaves) * 4;
    const int r_begin = min(nb, (part * kDirectWaves + wave) * share), r_end = min(nb, r_begin + share);
    const int last_col = min(16 * (NT - 1) + i16, p - 1);             // (beyond p: values that go into entries nobody reads)
    const bool is_y = 16 * (NT - 1) + i16 == p;
    KeyRow key;
#pragma unroll
    for (int i = 0; i < kPermRounds; ++i) key.k[i] = a.keys.key[pass][i];

    floatx4 acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    struct Stage {
        float x[U][NT];
    };
    uint32_t idx = 0;                                // lane l: row l of the 64 that are being requested
    float yv = 0.f, y_use = 0.f;                     // and its response; of the 64 that are being used
    auto entries = [&](int r0) {                     // rows r0 .. r0 + 63 of this wavefront (clamped)
        const int j = min(r0 + lane, r_end - 1);
        idx = perm_entry((uint32_t)(m * a.n + j), key, a.h, (uint32_t)a.rows);
        if (a.subset) {
            const uint32_t v = (uint32_t)a.subset[idx];
            if (v >= a.limit) __hip_atomic_store(a.bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            idx = v < a.limit ? v : 0u;
        }
        yv = a.y[idx];
    };
    auto request = [&](Stage& st, int k) {           // stage k of the 64 entries
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t r = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (4 * (k * U + u) + quad), (int)idx);
            const float* row = a.X + (size_t)r * (size_t)p;
#pragma unroll
            for (int f = 0; f < NT - 1; ++f) st.x[u][f] = row[i16 + 16 * f];
            st.x[u][NT - 1] = row[last_col];
        }
    };
    auto use = [&](Stage& st, int k, int left) {     // left: rows from the stage's first on
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float yy = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * (4 * (k * U + u) + quad), __builtin_bit_cast(int, y_use)));
            st.x[u][NT - 1] = is_y ? yy : st.x[u][NT - 1];
        }
        if (left < 4 * U) {                          // (uniform) the last stage: rows beyond the share count as zero
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int f = 0; f < NT; ++f) st.x[u][f] = 4 * u + quad < left ? st.x[u][f] : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int t = 0;
#pragma unroll
            for (int I = 0; I < NT; ++I) {
#pragma unroll
                for (int J = I; J < NT; ++J, ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(st.x[u][I], st.x[u][J], acc[t], 0, 0, 0);
            }
        }
    };
    if (r_begin < r_end) {
        // Two stages in registers, used in turn: a stage is requested while the other is used.  (A stage beyond the last one repeats rows
        // of the share and is not used.)
        static_assert(STAGES % 2 == 0, "a stage of each kind in turn");
        Stage A, B;
        entries(r_begin);
        request(A, 0);
        for (int r0 = r_begin; r0 < r_end; r0 += 64) {
            y_use = yv;
#pragma unroll
            for (int k = 0; k < STAGES; k += 2) {
                request(B, k + 1);
                if (r0 + 4 * U * k < r_end) use(A, k, r_end - (r0 + 4 * U * k));
                if (k + 2 < STAGES) request(A, k + 2);
                else { entries(min(r0 + 64, r_end - 1)); request(A, 0); }
                if (r0 + 4 * U * (k + 1) < r_end) use(B, k + 1, r_end - (r0 + 4 * U * (k + 1)));
            }
        }
    }

    finish_tiles<NT, TILES, S>(a, acc, 0, 0, lds, item, nb, wave, lane);
}

// The same matrices for 96 features and more: every wavefront for itself, on its own rows and its own piece of shared memory, without a barrier.
//
// The staged kernel reads both operands of every product from shared memory and is bound by the instructions around its matrix instructions
// (busy for 32 % of its time).  Here a lane's element of both operands is the same, one read for 16 columns of four rows, and the compiler knows
// the tiles; rows come from memory straight to shared memory, up to three chunks of eight ahead, and the next operands are read while four rows are
// multiplied.  The tiles are dealt to two workgroups (tile t = H TPW ... of the upper triangle, row by row): their sums leave room for three
// workgroups per compute unit; all tiles in one need no row twice, but come out less even on the compute units (p = 100, 300 mini-batches of 1,000
// rows: 68 against 75 us; two workgroups by rows as well: 79; one compute unit then holds three of the 600 workgroups, 41 us of matrix instructions
// at 2.15 GHz, others two).  The second group does not load the columns that only the first needs.  Both groups of a mini-batch run on one die, next
// to each other, so its rows come from memory once.  Entries of the partition come from memory: worked out here they cost 10 walks of the generator
// per 64 rows (94 us).  us per launch, staged kernel / this one: 87 / 69 (p = 100, 300 mini-batches of 1,000 rows), 128 / 104 (p = 127).  For fewer
// tiles it is not faster (p = 64: 38 / 43, p = 90: 36 / 43): a wavefront's loads and waits are then as long as its products.
template <int N> struct IntC { static constexpr int value = N; };

constexpr int kTileGroups = 2, kChunkRows = 8, kRing = 3;             // (a third workgroup fits a compute unit with a ring of three)
static_assert(kChunkRows == 8, "two groups of four rows");
constexpr int kBlockChunks = 2 * kRing, kBlockRows = kBlockChunks * kChunkRows;   // rows whose entries are fetched together
static_assert(kBlockRows <= 64, "one load of a wavefront fetches a block's entries, one its responses");

constexpr int tile_row(int NT, int t)                // I of tile t of the upper triangle, row by row
{
    int I = 0;
    while (t >= NT - I) { t -= NT - I; ++I; }
    return I;
}
constexpr int tile_col(int NT, int t)
{
    int I = 0;
    while (t >= NT - I) { t -= NT - I; ++I; }
    return I + t;
}

// acc[t] of tiles FROM, FROM + 1, ... += their share of four rows (which values of a lane that is has to be known to the compiler)
template <int NT, int FROM, int TPW, size_t... I>
__device__ __forceinline__ void multiply_tiles(floatx4 (&acc)[TPW], const float (&v)[NT], std::index_sequence<I...>)
{
    ((acc[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[IntC<tile_row(NT, FROM + (int)I)>::value], v[IntC<tile_col(NT, FROM + (int)I)>::value], acc[I], 0, 0, 0)), ...);
}

template <int NT, int H, bool VEC, int TPW>
__device__ __forceinline__ void rows_tiles(const DirectArgs& a, floatx4 (&acc)[TPW], unsigned char* mine, unsigned mine_lds, int pass, int m,
                                           int r_begin, int r_end, int lane)
{
    constexpr int TILES = NT * (NT + 1) / 2;
    constexpr int FIRST = tile_row(NT, H * TPW);     // the first tile row, and with it the first 16 columns, that this group needs
    constexpr int W = NT - FIRST;                    // 16-column blocks of a staged row
    constexpr int kChunk = kChunkRows * W * 64;      // bytes of a chunk
    constexpr int NI = VEC ? (W + 1) / 2 : 2 * W;    // load instructions of a chunk: the last one by half a wavefront if VEC and W is odd
    constexpr int kYAt = kRing * kChunkRows * NT * 64, kIdxAt = kYAt + 512;
    const int p = a.L.p, i16 = lane & 15, quad = lane >> 4;
    const bool is_y = 16 * (NT - 1) + i16 == p;
    // where in a chunk this lane's element of load q goes, and so which row (as a byte offset for the exchange of lanes) and columns it is
    int vrow[NI], vcol[NI];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const int e = lane + 64 * q;
        vrow[q] = 4 * (VEC ? e / (4 * W) : e / (16 * W));
        vcol[q] = 16 * FIRST + (VEC ? min(4 * (e % (4 * W)), p - 4 - 16 * FIRST) : min(e % (16 * W), p - 1 - 16 * FIRST));   // (beyond p: values that go into entries nobody reads)
    }
    const int* const from = a.perm + (size_t)pass * a.perm_stride + (size_t)m * a.n;
    auto uniform = [](unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); };
    auto request_entries = [&](int block) {          // rows kBlockRows * block .. of the share (clamped; lanes beyond the block's rows are not looked at)
        load_word_to_lds(from + min(r_begin + kBlockRows * block + lane, r_end - 1), uniform(mine_lds + kIdxAt + (unsigned)(block & 1) * 256u));
    };
    auto request_y = [&](int block) {
        const int row = *reinterpret_cast<const int*>(mine + kIdxAt + (block & 1) * 256 + 4 * lane);
        load_word_to_lds(reinterpret_cast<const int*>(a.y) + row, uniform(mine_lds + kYAt + (unsigned)(block & 1) * 256u));
    };
    unsigned row_of[NI];
    auto look_up = [&](int block, int k) {           // the rows of chunk k of a block
#pragma unroll
        for (int q = 0; q < NI; ++q) row_of[q] = *reinterpret_cast<const unsigned*>(mine + kIdxAt + (block & 1) * 256 + 4 * kChunkRows * k + vrow[q]);
    };
    auto request = [&](int k) {                      // ... which have been looked up
        const unsigned to = uniform(mine_lds + (unsigned)(k % kRing) * kChunk);
#pragma unroll
        for (int q = 0; q < NI; ++q) {
            const float* src = a.X + (size_t)row_of[q] * (size_t)p + vcol[q];
            if constexpr (!VEC) load_word_to_lds(reinterpret_cast<const int*>(src), to + 256u * q);
            else if (64 * (q + 1) <= 4 * W * kChunkRows || lane < 32) load_to_lds(reinterpret_cast<const unsigned short*>(src), to + 1024u * q);
        }
    };
    auto read = [&](float (&v)[NT], int block, int k, int g) {       // four rows
        const float* row = reinterpret_cast<const float*>(mine + (k % kRing) * kChunk) + (4 * g + quad) * (16 * W) + i16;
        const float* end = is_y ? reinterpret_cast<const float*>(mine + kYAt + (block & 1) * 256) + kChunkRows * k + 4 * g + quad : row + 16 * (W - 1);
#pragma unroll
        for (int f = FIRST; f < NT - 1; ++f) v[f] = row[16 * (f - FIRST)];
        v[NT - 1] = *end;
    };
    auto use = [&](float (&v)[NT], int left) {       // left: rows from these on
        if (left <= 0) return;
        if (left < 4) {                              // (uniform) the last ones: rows beyond the share count as zero
#pragma unroll
            for (int f = FIRST; f < NT; ++f) v[f] = quad < left ? v[f] : 0.f;
        }
        multiply_tiles<NT, H * TPW>(acc, v, std::make_index_sequence<TPW < TILES - H * TPW ? TPW : TILES - H * TPW>{});
    };
    auto landed = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    request_entries(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    request_y(0);
#pragma unroll
    for (int k = 0; k < kRing; ++k) {
        look_up(0, k);
        request(k);
    }
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 1) * NI) : "memory");
    float first[NT], second[NT];
    read(first, 0, 0, 0);
    for (int block = 0; r_begin + kBlockRows * block < r_end; ++block) {
        const int left = r_end - r_begin - kBlockRows * block;
        request_entries(block + 1);
#pragma unroll
        for (int k = 0; k < kBlockChunks; ++k) {
            // Operands of the next four rows, and the rows of the chunk that is requested next, are read from shared memory while four rows are
            // multiplied.  Chunk k + kRing goes where chunk k is, whose reads have returned by then; the rows of chunk k + 1, requested before
            // kRing - 1 others, have come behind the wait (and by k = kRing - 1 the next entries, requested before chunk kRing).
            constexpr int kNext = kBlockChunks - kRing;
            read(second, block, k, 1);
            look_up(block + (k + kRing) / kBlockChunks, (k + kRing) % kBlockChunks);
            use(first, left - kChunkRows * k);
            landed();
            if (k == kNext) request_y(block + 1);
            request((k + kRing) % kBlockChunks);
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 1) * NI) : "memory");
            read(first, block + (k + 1) / kBlockChunks, (k + 1) % kBlockChunks, 0);
            use(second, left - kChunkRows * k - 4);
        }
    }
}

template <int NT>
constexpr int rows_lds_bytes()
{
    constexpr int TPW = (NT * (NT + 1) / 2 + kTileGroups - 1) / kTileGroups;
    constexpr int ring = kDirectWaves * (kRing * kChunkRows * NT * 64 + 1024), sums = 2 * (TPW < kSumTiles ? TPW : kSumTiles) * 1024;
    static_assert(ring <= 65536 && sums <= 65536, "more has to be asked for, kernel by kernel");
    return ring > sums ? ring : sums;
}

template <int NT, int S, bool VEC>
__global__ void __launch_bounds__(64 * kDirectWaves, 2) gram_rows_kernel(DirectArgs a)
{
    constexpr int T = kTileGroups, TPW = (NT * (NT + 1) / 2 + T - 1) / T;
    extern __shared__ __align__(16) unsigned char smem[];
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int h = slot % T, part = slot / T % S, item = slot / (T * S) * 8 + xcd;
    if (item >= a.n_items) return;
    const int pass = item / a.M, m = item - pass * a.M;
    const int nb = min(a.n, a.rows - m * a.n);
    // this wavefront's rows: whole groups of four, one share of S * kDirectWaves
    const int share = (nb + 4 * S * kDirectWaves - 1) / (4 * S * kDirectWaves) * 4;
    const int r_begin = min(nb, (part * kDirectWaves + wave) * share), r_end = min(nb, r_begin + share);
    constexpr int kMine = kRing * kChunkRows * NT * 64 + 1024;
    unsigned char* const mine = smem + wave * kMine;
    const unsigned mine_lds = (unsigned)(size_t)(lds_byte*)smem + (unsigned)(wave * kMine);
    floatx4 acc[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (r_begin < r_end) {
        if (h == 0) rows_tiles<NT, 0, VEC, TPW>(a, acc, mine, mine_lds, pass, m, r_begin, r_end, lane);
        else rows_tiles<NT, 1, VEC, TPW>(a, acc, mine, mine_lds, pass, m, r_begin, r_end, lane);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (rows requested beyond the last ones)
    __syncthreads();
    finish_tiles<NT, TPW, S>(a, acc, h * TPW, h, reinterpret_cast<float*>(smem), item, nb, wave, lane);
}

using DirectFn = void (*)(DirectArgs);

template <int S>
DirectFn direct_kernel(int NT)
{
    switch (NT) {
    case 1: return gram_direct_kernel<1, S>;
    case 2: return gram_direct_kernel<2, S>;
    case 3: return gram_direct_kernel<3, S>;
    }
    return nullptr;
}

// By the mini-batches of one pass, so that a pass gives the same bits whatever it is launched with.
bool direct_moments(int p, int M) { return p <= 47 && M >= 64; }

// Two workgroups for a mini-batch, by rows, while a launch is a few rounds of workgroups (two per compute unit) at most, if the mini-batch is
// long: for a short one the second trip through memory costs more than the rows it spreads.  us of a buffer waited for, three passes, one /
// two workgroups: 236 / 254 (p = 37, n = 74, 511 mini-batches), 159 / 171 (256), 122 / 122 (p = 33, n = 500, 128), 137 / 131 (n = 1000, 128),
// 195 / 207 (p = 47, n = 1000, 256), 202 / 191 (p = 33, n = 1500, 192), 198 / 175 (n = 3000, 128), 410 / 391 (384).
int direct_split(int M, int n) { return n >= (M <= 160 ? 768 : 1024) && M < 512 ? 2 : 1; }

// tiles per workgroup for NT tile rows: {few workgroups, many workgroups}
void tile_split(int ntiles, int wgs_per_split, int* tsplit, int* tpw)
{
    // at most 10 tiles per workgroup: measured faster than wider workgroups (more of them, two per SIMD)
    static const int options[10][3] = {{1, 1, 1}, {3, 1, 1}, {6, 1, 1}, {10, 1, 2}, {15, 3, 3},
                                       {21, 3, 3}, {28, 4, 4}, {36, 4, 4}, {45, 5, 5}, {0, 0, 0}};
    for (int i = 0; options[i][0]; ++i)
        if (options[i][0] == ntiles) {
            const int few = options[i][1], many = options[i][2];
            *tsplit = wgs_per_split * few >= 256 ? few : many;
            *tpw = (ntiles + *tsplit - 1) / *tsplit;
            return;
        }
    *tsplit = 0;
    *tpw = 0;
}

template <int TPW>
hipError_t launch_gram_mfma(bool wide, dim3 grid, size_t lds, hipStream_t stream, const float* X, const float* y, const int32_t* perm,
                            float* out, int rows, int n, int perm_stride, int M, int n_items, int stride, const GramLayout& L,
                            const GramTiles& T, int dense_q, hipEvent_t start, hipEvent_t stop)
{
    // the events ride on the dispatch itself: no separate markers in the queue
    const bool vec = L.p % 4 == 0;
#define GRAM_LAUNCH(W, V)                                                                                                          \
    hipExtLaunchKernelGGL((gram_mfma_kernel<TPW, W, V>), grid, dim3(64 * kGramWaves), (uint32_t)lds, stream, start, stop, 0u, X, y,  \
                          perm, out, rows, n, perm_stride, M, n_items, stride, L, T, dense_q)
    if (wide && vec) GRAM_LAUNCH(true, true);
    else if (wide) GRAM_LAUNCH(true, false);
    else if (vec) GRAM_LAUNCH(false, true);
    else GRAM_LAUNCH(false, false);
#undef GRAM_LAUNCH
    return hipGetLastError();
}

// p > 95 (seven to nine tile rows): the kernel, its shared memory
template <int S>
DirectFn rows_kernel(int NT, bool vec, int* lds)
{
    switch (NT) {
    case 7: *lds = rows_lds_bytes<7>(); return vec ? gram_rows_kernel<7, S, true> : gram_rows_kernel<7, S, false>;
    case 8: *lds = rows_lds_bytes<8>(); return vec ? gram_rows_kernel<8, S, true> : gram_rows_kernel<8, S, false>;
    case 9: *lds = rows_lds_bytes<9>(); return vec ? gram_rows_kernel<9, S, true> : nullptr;     // (p = 128)
    }
    return nullptr;
}

// Where the kernel above takes p > 95 from the staged one: many mini-batches, or few long ones, which it splits over two workgroups by rows.
// With few rows in a mini-batch the staged kernel's more workgroups, each with fewer tiles, get going sooner.  By the mini-batches of one pass, as
// above, and so that launches of one to four passes come out at most 4 % slower (swept over M = 1 to 1000).  Two workgroups to a mini-batch
// come out uneven on 256 compute units where the last round of a pass's is less than full (`even`): that costs more than the kernel gains with its
// 45 tiles at p = 128, and where the staged kernel gains most from its finer shares, rows of up to 111 values that are not moved in fours.  us of
// moments for one pass / three, staged kernel and this one (mini-batches, rows; -: not chosen).  p = 100: 36 / 84 and 35 / 77 (100, 1000), 32 / 71 and
// 25 / 54 (200, 300), - 25 / 63 and 25 / 49 (128, 500), - 17 / 37 and 19 / 33 (100, 256), - 28 / 58 and 35 / 53 (64, 1000); split: 136 / 139 and 101 / 102
// (8, 8000), 73 / 77 and 61 / 64 (16, 4000), 43 / 63 and 42 / 60 (32, 2000), - 36 / 76 and 38 / 67 (48, 1500).  p = 111: - 33 / 79 and 38 / 72 (150, 500).
// p = 112: - 64 / 127 and 66 / 140 (84, 2000).  p = 127: 51 / 125 and 46 / 116 (100, 1000), 225 / 229 and 136 / 137 (8, 8000), 118 / 125 and 81 / 84 (16,
// 4000).  p = 128: 59 / 157 and 50 / 131 (256, 500), - 39 / 98 and 47 / 89 (150, 500); split: 146 / 152 and 131 / 133 (8, 8000), - 44 / 46 and 55 / 56 (8, 2000).
bool rows_moments(int p, int M, int n)
{
    if (p <= 95) return false;
    if (M < 85) return n >= (p == 128 ? 8000 : M <= 48 ? 2000 : 5000);
    if ((int64_t)M * n < 50000 || (M <= 128 && n < 560)) return false;
    const int rounds = (2 * M + 255) / 256;
    const bool even = 2 * M * 5 >= rounds * 256 * 4;
    if (p == 128) return even;
    if (p < 112 && p % 4 != 0) return even && (n >= 600 || M >= 600);
    return true;
}

int rows_split(int M) { return M < 85 ? 2 : 1; }

template <int TPR, int KQ, int KS>
hipError_t launch_chain(const GramLayout& L, const float* gram, float* theta, int nsteps, int period, float alpha, const float* lr_tab,
                        int lr_base, int lr_len, const OptArgs& opt, hipStream_t stream, hipEvent_t start, hipEvent_t stop)
{
    constexpr int per_step = 4 * KQ + KS + 1;
    constexpr int AHEAD = per_step <= 9 ? 8 : per_step <= 14 ? 6 : 4;
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, dim3(1), dim3(L.nthr), 0u, stream, start, stop, 0u, gram, theta, L, nsteps, period, alpha, lr_tab,
                              lr_base, lr_len, opt);
    };
    const int rule = opt.kind == kOptSgd ? kRulePlain : opt.kind == kOptAdam ? kRuleAdam : kRuleMomentum;
    if (lr_tab) {
        if (rule == kRulePlain) go(gram_chain_kernel<TPR, KQ, KS, AHEAD, true, kRulePlain>);
        else if (rule == kRuleMomentum) go(gram_chain_kernel<TPR, KQ, KS, AHEAD, true, kRuleMomentum>);
        else go(gram_chain_kernel<TPR, KQ, KS, AHEAD, true, kRuleAdam>);
    } else {
        if (rule == kRulePlain) go(gram_chain_kernel<TPR, KQ, KS, AHEAD, false, kRulePlain>);
        else if (rule == kRuleMomentum) go(gram_chain_kernel<TPR, KQ, KS, AHEAD, false, kRuleMomentum>);
        else go(gram_chain_kernel<TPR, KQ, KS, AHEAD, false, kRuleAdam>);
    }
    return hipGetLastError();
}

template <int TPR, int KQ>
hipError_t launch_chain_ks(const GramLayout& L, const float* gram, float* theta, int nsteps, int period, float alpha,
                           const float* lr_tab, int lr_base, int lr_len, const OptArgs& opt, hipStream_t stream, hipEvent_t start,
                           hipEvent_t stop)
{
    switch (L.ks) {
    case 0: return launch_chain<TPR, KQ, 0>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
    case 1: return launch_chain<TPR, KQ, 1>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
    case 2: return launch_chain<TPR, KQ, 2>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
    case 3: return launch_chain<TPR, KQ, 3>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
    case 4: return launch_chain<TPR, KQ, 4>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool gram_eligible(int model, int64_t p, int64_t n)
{
    return model == 0 && p <= kGramMaxP && n >= 2 * p;
}

size_t gram_bytes_per_batch(int64_t p)
{
    return (size_t)make_layout((int)p).step_floats * sizeof(float);
}

int gram_dense_order(int64_t p) { return (int)((p + 1 + 15) / 16 * 16); }

size_t gram_dense_bytes_per_batch(int64_t p)
{
    const size_t q = (size_t)gram_dense_order(p);
    return q * q * sizeof(float);
}

int gram_chain_threads(int64_t p)
{
    return make_layout((int)p).nthr;
}

bool gram_moments_draw(int64_t p, int64_t rows, int64_t n) { return direct_moments((int)p, (int)((rows + n - 1) / n)); }

hipError_t gram_launch_moments(const float* X, const float* y, const int32_t* perm, const GramPartition& from, float* gram, unsigned* tickets,
                               int rows, int p, int n, int npass, int perm_stride, hipStream_t stream, hipEvent_t start, hipEvent_t stop,
                               bool dense)
{
    const int dense_q = dense ? gram_dense_order(p) : 0;
    if (p < 1 || p > kGramMaxP) return hipErrorInvalidValue;
    const GramLayout L = make_layout(p);
    const int M = (rows + n - 1) / n;
    const int gpass = perm_stride == 0 ? 1 : npass;      // one partition for all passes: one set of matrices
    const int NT = (p + 1 + 15) / 16;                    // tile rows of the moment matrix of [X y]
    DirectArgs a{};
    a.X = X; a.y = y; a.keys = from.keys; a.h = (uint32_t)perm_half_width(rows);
    a.subset = from.subset; a.limit = (uint32_t)from.limit; a.bad = from.bad;
    a.out = gram; a.tickets = tickets; a.L = L;
    a.rows = rows; a.n = n; a.M = M; a.dense_q = dense_q; a.n_items = M * gpass; a.perm = perm; a.perm_stride = perm_stride;
    const bool direct = direct_moments(p, M);
    const int S = direct ? direct_split(M, n) : rows_split(M);
    if (direct) {
        DirectFn fn = S == 2 ? direct_kernel<2>(NT) : direct_kernel<1>(NT);
        if (!fn || (S == 2 && !tickets)) return hipErrorInvalidValue;
        hipExtLaunchKernelGGL(fn, dim3((unsigned)(a.n_items * S)), dim3(64 * kDirectWaves), 0u, stream, start, stop, 0u, a);
        return hipGetLastError();
    }
    if (!perm) return hipErrorInvalidValue;
    if (rows_moments(p, M, n)) {
        int lds = 0;
        DirectFn fn = S == 2 ? rows_kernel<2>(NT, p % 4 == 0, &lds) : rows_kernel<1>(NT, p % 4 == 0, &lds);
        if (!fn || (S == 2 && !tickets)) return hipErrorInvalidValue;
        hipExtLaunchKernelGGL(fn, dim3((unsigned)((a.n_items + 7) / 8 * 8 * kTileGroups * S)), dim3(64 * kDirectWaves), (uint32_t)lds, stream, start, stop, 0u, a);
        return hipGetLastError();
    }
    GramTiles T{};
    T.ntiles = NT * (NT + 1) / 2;
    int tpw = 0;
    tile_split(T.ntiles, M * gpass, &T.tsplit, &tpw);
    if (T.tsplit == 0) return hipErrorInvalidValue;
    {
        int k = 0;
        for (int I = 0; I < NT; ++I)
            for (int J = I; J < NT; ++J) T.tile[k++] = (unsigned short)(I | (J << 8));
        for (; k < 48; ++k) T.tile[k] = 0;
    }
    int stride = NT * 16;
    if (stride % 32 == 0) stride += 16;                  // rows k and k + 1 of an operand read fall on different banks
    const size_t lds = sizeof(float) * (size_t)std::max(kGramWaves * kRowsPerChunk * stride, kGramWaves * tpw * 64 * 4);
    const int n_items = a.n_items;
    const dim3 grid((unsigned)((n_items + 7) / 8 * 8 * T.tsplit));
    const bool wide = p > 64;
    hipError_t e = hipErrorInvalidValue;
#define GRAM_CASE(N) case N: e = launch_gram_mfma<N>(wide, grid, lds, stream, X, y, perm, gram, rows, n, perm_stride, M, n_items, stride, L, T, dense_q, start, stop); break
    switch (tpw) {
        GRAM_CASE(1); GRAM_CASE(3); GRAM_CASE(5); GRAM_CASE(6); GRAM_CASE(7); GRAM_CASE(9); GRAM_CASE(10);
    }
#undef GRAM_CASE
    return e;
}

hipError_t gram_launch_chain(const float* gram, float* theta, int rows, int p, int n, int npass, int perm_stride, float alpha,
                             const float* lr_tab, int lr_base, int lr_len, const OptArgs& opt, hipStream_t stream,
                             hipEvent_t start, hipEvent_t stop)
{
    const int M = (rows + n - 1) / n;
    const int nsteps = M * npass, period = perm_stride == 0 ? M : nsteps;
    return gram_launch_chain_steps(gram, theta, p, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
}

hipError_t gram_launch_chain_steps(const float* gram, float* theta, int p, int nsteps, int period, float alpha, const float* lr_tab,
                                   int lr_base, int lr_len, const OptArgs& opt, hipStream_t stream, hipEvent_t start,
                                   hipEvent_t stop)
{
    if (p < 1 || p > kGramMaxP || nsteps < 1 || period < 1) return hipErrorInvalidValue;
    const GramLayout L = make_layout(p);
    if (L.tpr == 4) {
        switch (L.kq) {
        case 0: return launch_chain_ks<4, 0>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 1: return launch_chain_ks<4, 1>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 2: return launch_chain_ks<4, 2>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 3: return launch_chain_ks<4, 3>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 4: return launch_chain_ks<4, 4>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        }
    } else {
        switch (L.kq) {
        case 2: return launch_chain_ks<8, 2>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 3: return launch_chain_ks<8, 3>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        case 4: return launch_chain_ks<8, 4>(L, gram, theta, nsteps, period, alpha, lr_tab, lr_base, lr_len, opt, stream, start, stop);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace bmgd
