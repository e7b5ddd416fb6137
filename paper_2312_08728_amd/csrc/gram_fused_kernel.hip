// Least squares with few features and few, small mini-batches: the whole launch - partitions, moment matrices, chain of eq. (3.1) - in
// one kernel.
//
// What bounds such a launch is what surrounds its kernels: the partition, the moments and the chain of 40 steps on ten features take 20 us of
// the device, but three dispatches on two streams, their events and the waits between them 50 us.  So a workgroup takes a mini-batch:
// its wavefronts work out the entries of the partition they need, gather the rows straight into matrix operands, and leave the mini-batch's
// matrices in memory; the workgroup that finishes last runs the chain.  Nobody waits for anybody: the others have all been there (a ticket
// taken behind their stores tells), so no residency of the grid is needed.
//
// Per buffer, wall clock among others, before (three kernels) / now: 49 / 23 us at p = 10, n = 100, 2,000 rows x 2 passes (kernel 12 us: rows
// 4, to memory and the ticket 3, chain of 40 steps 5); 72 / 57 us at p = 37, n = 300, 20,011 rows x 2 passes with NAG and a table of rates
// (kernel 41 us, 25 of them the chain of 134 steps; what lies between kernels that carry events is 9 us).
#include "gram_chain.h"
#include "perm_device.h"

#include <hip/hip_ext.h>

#include <algorithm>

namespace bmgd {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kFusedWaves = 8;
constexpr int kFusedBlock = 64 * kFusedWaves;
constexpr int kFusedChain = 256;                     // threads of the chain at most: four per row
constexpr int kFusedMaxP = 63;                       // at most four tile rows, all tiles of a mini-batch in one wavefront's registers
constexpr int kFusedMaxBatch = 512;
constexpr int kFusedMaxSteps = 1008;                 // of a launch: their rates are in shared memory, zeros behind them
constexpr int kFusedRates = 1024;

struct FusedArgs {
    const float* X;
    const float* y;
    PermKeys keys;
    uint32_t h;
    const int32_t* subset;                           // (or NULL) the rows the run is restricted to, of a buffer of `limit` rows
    uint32_t limit;
    unsigned* bad;
    float* gram;
    float* theta;
    unsigned* ticket;                                // workgroups that have left their matrices; zero between launches
    GramLayout L;
    int rows, n, M, nsteps;
    float alpha;
    const float* lr_tab;
    int lr_base, lr_len;
    OptArgs opt;
};

// NT = KQ + 1 tile rows hold the p + 1 columns of [X y].  MFMA operand layout (v_mfma_f32_16x16x4_f32): a = A[lane % 16][lane / 16],
// b = B[lane / 16][lane % 16], c[v] = C[4 (lane / 16) + v][lane % 16]; with A = rows' and B = rows a lane's element of both is the same, so
// a row of a tile is one load per lane and serves every tile of its row and column.
template <int KQ, int KS, int RULE>
__global__ void __launch_bounds__(kFusedBlock) gram_fused_kernel(FusedArgs a)
{
    constexpr int NT = KQ + 1, TILES = NT * (NT + 1) / 2;
    constexpr int U = 8;                             // groups of four rows requested together
    // [wavefront][tile][lane] partial sums (of the upper four wavefronts, then of the lower four), later the rates of the steps; the
    // mini-batch's matrices in the chain's layout
    constexpr int RED = kFusedWaves / 2;
    __shared__ __align__(16) float lds[RED * TILES * 256];
    __shared__ __align__(16) float mat[(4 * KQ + KS) * kFusedChain + 64];
    __shared__ unsigned s_ticket;
    static_assert(RED * 256 >= kFusedRates && kFusedMaxSteps + 16 <= kFusedRates, "the rates of a launch's steps");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int item = blockIdx.x;                     // a mini-batch of a pass
    const int pass = item / a.M, m = item - pass * a.M;
    const int p = a.L.p;
    const int nb = min(a.n, a.rows - m * a.n);
    KeyRow key;
#pragma unroll
    for (int i = 0; i < kPermRounds; ++i) key.k[i] = a.keys.key[pass][i];

    for (int e = threadIdx.x; e < a.L.step_floats; e += kFusedBlock) mat[e] = 0.f;   // padding of the layout

    floatx4 acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int share = (nb + 4 * kFusedWaves - 1) / (4 * kFusedWaves) * 4;            // rows of a wavefront, whole groups of four
    const int r_end = min(nb, (wave + 1) * share);
    const int i16 = lane & 15;
    int col[NT];
#pragma unroll
    for (int f = 0; f < NT; ++f) col[f] = min(16 * f + i16, p - 1);                 // (beyond p: values that go into entries nobody reads)
    const bool is_y = 16 * (NT - 1) + i16 == p;
    for (int r0 = wave * share; r0 < r_end; r0 += 64) {
        const int cnt = min(64, r_end - r0);
        uint32_t idx = perm_entry((uint32_t)(m * a.n + r0 + min(lane, cnt - 1)), key, a.h, (uint32_t)a.rows);
        if (a.subset) {
            const uint32_t v = (uint32_t)a.subset[idx];
            if (v >= a.limit) __hip_atomic_store(a.bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            idx = v < a.limit ? v : 0u;
        }
        const float yv = a.y[idx];
        for (int g0 = 0; g0 < cnt; g0 += 4 * U) {
            float x[U][NT];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int src = min(g0 + 4 * u + (lane >> 4), 63);                  // the lane that holds the row's index
                const uint32_t r = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * src, (int)idx);
                const float* row = a.X + (size_t)r * (size_t)p;
#pragma unroll
                for (int f = 0; f < NT; ++f) x[u][f] = row[col[f]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int src = g0 + 4 * u + (lane >> 4);
                const float yy = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * min(src, 63), __builtin_bit_cast(int, yv)));
                x[u][NT - 1] = is_y ? yy : x[u][NT - 1];
                const bool there = src < cnt;                                       // rows beyond the wavefront's share count as zero
#pragma unroll
                for (int f = 0; f < NT; ++f) x[u][f] = there ? x[u][f] : 0.f;
                int t = 0;
#pragma unroll
                for (int I = 0; I < NT; ++I) {
#pragma unroll
                    for (int J = I; J < NT; ++J, ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][I], x[u][J], acc[t], 0, 0, 0);
                }
            }
        }
    }
    // the wavefronts' sums meet in shared memory, are divided by n_b and put in the chain's order
    floatx4* red = reinterpret_cast<floatx4*>(lds);
    if (wave >= RED) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) red[((wave - RED) * TILES + t) * 64 + lane] = acc[t];
    }
    __syncthreads();
    if (wave < RED) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            acc[t] += red[(wave * TILES + t) * 64 + lane];
            red[(wave * TILES + t) * 64 + lane] = acc[t];
        }
    }
    __syncthreads();
    const float inv = 1.f / (float)nb;
    auto pos = [&](int r, int c) {                   // gram_pos for four threads a row
        const int k = c >> 4, cc = c - 16 * KQ;
        return k < KQ ? ((k * a.L.nthr + r * 4 + ((c >> 2) & 3)) << 2) + (c & 3) : (4 * KQ + (cc >> 2)) * a.L.nthr + r * 4 + (cc & 3);
    };
    {
        int t = 0;
#pragma unroll
        for (int I = 0; I < NT; ++I) {
#pragma unroll
            for (int J = I; J < NT; ++J, ++t) {
                if (t % kFusedWaves != wave) continue;
                floatx4 s = red[t * 64 + lane];
#pragma unroll
                for (int w = 1; w < RED; ++w) s += red[(w * TILES + t) * 64 + lane];
                const int c = 16 * J + i16;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = 16 * I + 4 * (lane >> 4) + q;
                    const float val = s[q] * inv;
                    if (r < p && c < p) {
                        mat[pos(r, c)] = val;
                        if (I != J) mat[pos(c, r)] = val;
                    } else if (r < p && c == p) {
                        mat[a.L.b_off + r] = val;
                    }
                }
            }
        }
    }
    __syncthreads();
    // Out to memory, past this die's cache (agent scope), so that the workgroup that runs the chain finds them wherever it is; the ticket
    // is taken when they have arrived.
    float* out = a.gram + (size_t)item * a.L.step_floats;
    for (int e = threadIdx.x; e < a.L.step_floats; e += kFusedBlock)
        __hip_atomic_store(out + e, mat[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) s_ticket = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_ticket != gridDim.x - 1) return;

    // the last one: the chain
    if (threadIdx.x == 0) __hip_atomic_store(a.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    for (int s = threadIdx.x; s < a.nsteps; s += kFusedBlock) lds[s] = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
    for (int s = a.nsteps + threadIdx.x; s < kFusedRates; s += kFusedBlock) lds[s] = 0.f;
    __syncthreads();
    if ((int)threadIdx.x >= a.L.nthr) return;        // (whole wavefronts; a barrier counts those that are there)
    constexpr int per_step = 4 * KQ + KS + 1;
    constexpr int AHEAD = per_step <= 9 ? 8 : per_step <= 14 ? 6 : 4;
    gram_chain_steps<4, KQ, KS, AHEAD, kRateShared, RULE>(a.gram, a.theta, a.L, a.nsteps, a.nsteps, a.alpha, nullptr, 0, 0, lds, a.opt);
}

using FusedFn = void (*)(FusedArgs);

template <int KQ, int KS>
FusedFn pick_rule(int kind)
{
    if constexpr (4 * KQ + KS == 0) return nullptr;
    else
        return kind == kOptSgd ? gram_fused_kernel<KQ, KS, kRulePlain>
             : kind == kOptAdam ? gram_fused_kernel<KQ, KS, kRuleAdam> : gram_fused_kernel<KQ, KS, kRuleMomentum>;
}

template <int KQ>
FusedFn pick_ks(int ks, int kind)
{
    switch (ks) {
    case 0: return pick_rule<KQ, 0>(kind);
    case 1: return pick_rule<KQ, 1>(kind);
    case 2: return pick_rule<KQ, 2>(kind);
    case 3: return pick_rule<KQ, 3>(kind);
    case 4: return pick_rule<KQ, 4>(kind);
    }
    return nullptr;
}

FusedFn fused_kernel(const GramLayout& L, int kind)
{
    switch (L.kq) {
    case 0: return pick_ks<0>(L.ks, kind);
    case 1: return pick_ks<1>(L.ks, kind);
    case 2: return pick_ks<2>(L.ks, kind);
    case 3: return pick_ks<3>(L.ks, kind);
    }
    return nullptr;
}

}  // namespace

bool gram_fused_eligible(int64_t p, int64_t buffer_n, int64_t batch_n, int64_t passes, bool plain)
{
    const int64_t M = (buffer_n + batch_n - 1) / batch_n;
    // A launch of four passes at most.  A mini-batch is one workgroup's, so it must be short; and all rows together few enough that the
    // moments of a buffer need not overlap the chain of the one before.
    if (p > kFusedMaxP || batch_n > kFusedMaxBatch || kMaxPassesPerLaunch * M > kFusedMaxSteps ||
        kMaxPassesPerLaunch * buffer_n * p * 4 > (int64_t(1) << 24))
        return false;
    // Plain steps can be multiplied in pairs by separate kernels, which halves the chain; those kernels take 45 to 60 us a buffer however
    // few the steps (the host is the bound), this one 15 us and 0.1 to 0.25 us a step.  us per buffer of this one / of the others, 2 p
    // rows a mini-batch, where buffers follow one another (one that is waited for takes 30 us more here, 40 to 50 more there):
    //   steps      130       160       200       252       300       360       500       1000
    //   p = 10   27 / 50   30 / 50   34 / 56   42 / 53   47 / 52   53 / 50   69 / 48   125 / 71
    //   p = 31   35 / 46   38 / 48   43 / 48   52 / 48   64 / 49   71 / 50
    //   p = 47   42 / 49   48 / 47   59 / 48   68 / 50   80 / 50   91 / 56
    //   p = 63   50 / 59   59 / 59   69 / 58   81 / 58   95 / 59  108 / 63
    // With state the alternative is the chain step by step: as fast or up to a tenth faster from 250 steps on where buffers follow one
    // another (p = 5, 500 steps: 70 against 75 us), a fifth slower for a buffer that is waited for (129 against 107 us).
    const int64_t steps = std::min<int64_t>(kMaxPassesPerLaunch, passes) * M;
    return !plain || steps <= (p <= 32 ? 256 : p <= 48 ? 160 : 128);
}

hipError_t gram_launch_fused(const float* X, const float* y, const PermKeys& keys, const int32_t* subset, int64_t limit, unsigned* bad,
                             float* gram, float* theta, unsigned* ticket, int rows, int p, int n, int npass, float alpha,
                             const float* lr_tab, int lr_base, int lr_len, const OptArgs& opt, hipStream_t stream, hipEvent_t start,
                             hipEvent_t stop)
{
    const int M = (rows + n - 1) / n;
    if (p < 1 || p > kFusedMaxP || rows < 1 || n < 1 || npass < 1 || npass > kMaxPassesPerLaunch || M * npass > kFusedMaxSteps ||
        (subset && (!bad || limit < rows)))
        return hipErrorInvalidValue;
    FusedArgs a{};
    a.X = X; a.y = y; a.keys = keys; a.h = (uint32_t)perm_half_width(rows);
    a.subset = subset; a.limit = (uint32_t)limit; a.bad = bad;
    a.gram = gram; a.theta = theta; a.ticket = ticket;
    a.L = make_layout(p);
    a.rows = rows; a.n = n; a.M = M; a.nsteps = M * npass;
    a.alpha = alpha; a.lr_tab = lr_tab; a.lr_base = lr_base; a.lr_len = lr_len;
    a.opt = opt;
    FusedFn fn = fused_kernel(a.L, opt.kind);
    if (!fn || a.L.tpr != 4 || a.L.nthr > kFusedChain) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(fn, dim3((unsigned)a.nsteps), dim3(kFusedBlock), 0u, stream, start, stop, 0u, a);
    return hipGetLastError();
}

}  // namespace bmgd
