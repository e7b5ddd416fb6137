// Softmax regression on small mini-batches: all updates of a pass in one persistent kernel.
//
// Three launches per update (logits, residual, gradient + update; softmax_kernels.hip) cost 17-23 us whatever the size: each
// small kernel is a chain of dependent trips to memory, and the weights go out to memory and back between them.  Here the
// CLASSES are split over workgroups, 16 to each: a workgroup keeps its columns of W for the whole pass (fp32 master in
// registers, in the accumulator layout of its gradient tiles; bf16 copy in shared memory, where the logits read it), so
//     U = X_b W[:, mine]                    needs all features of a row, but nothing of other workgroups;
//     R = softmax_rows(U) - onehot(y)       needs two numbers per row from each of the others: the maximum of its classes and
//                                           their sum of e^(u - maximum);
//     W[:, mine] -= (alpha / n_b) X_b' R    is again the workgroup's own.
// Two numbers per row and workgroup are all that is exchanged (flagged words, glm_device.h: one trip over the fabric per update;
// none at all for up to 16 classes).  (Joined into one, the log of the sum on top of the maximum, they would cost a word less, but
// the probabilities would be off by the spacing of fp32 at the size of the logits.)  The mini-batch is read by every workgroup from its L2, twice per update (rows for the
// logits, transposed for the gradient), laid out once per pass in the order in which the matrix instructions take their
// operands (pack_kernel): one contiguous KiB per load instruction, requested ahead, the next update's first ones before
// this update's gradient.
//
// The exchange needs all workgroups of the launch resident at once, which work of other streams and processes can prevent.  So they
// meet before the first update (gather_workgroups): where they do not within a given time, one of them makes the whole pass by
// itself, class share by class share (pass_alone, the same sums in the same order), and the others leave.
//
// What bounds it: the trip over the fabric for small mini-batches, and one compute unit's load path (4 n p bytes per update)
// for larger ones (softmax_chain_eligible says where the line to the three launches lies).
#include "bmgd_internal.h"
#include "glm_device.h"

#include <float.h>

#include <algorithm>

namespace bmgd {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kClasses = 16;                       // classes per workgroup (two tiles of 16 that share the operands of X were slower nearly
                                                   // everywhere: twice the exponentials and registers; 25.1 against 17.6 us at 1000 x 256 x 200)
constexpr int NJ = kClasses / 16;
constexpr int kMaxTiles = 8;                       // row tiles and feature tiles of 16 per wavefront
constexpr int kMaxRows = 16 * kWaves * kMaxTiles;  // 1024: mini-batch rows, and features

// four values rounded to bf16 (to nearest, ties to even, by the conversion instruction)
__device__ __forceinline__ uint2 to_bf16x4(const float (&v)[4])
{
    typedef float f32x4_ __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x4_ __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint2, __builtin_convertvector((f32x4_{v[0], v[1], v[2], v[3]}), bf16x4_));
}

// e^x for x <= 0 or NaN: 2^n 2^f with n = x log2 e rounded to a whole number and f what is left (log2 e in two parts), in eight
// instructions.  As good as expf: over [-87, 0] a relative error of at most 8.5e-8 (2.7e-8 rms; expf 8.4e-8 and 2.6e-8), and the
// subnormal numbers below to their last unit.
__device__ __forceinline__ float exp_neg(float x)
{
    constexpr float kLog2e = 1.44269502f, kLog2eLo = 1.92596299e-8f, kRound = 12582912.f;   // 1.5 x 2^23: the sum's last bit is 1
    x = x < -200.f ? -200.f : x;                     // (keeps a NaN; e^-200 is 0)
    const float t = fmaf(x, kLog2e, kRound);
    const float f = fmaf(x, kLog2eLo, fmaf(x, kLog2e, kRound - t));
    return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), __builtin_bit_cast(int, t) - __builtin_bit_cast(int, kRound));
}

// The mini-batches of a pass in operand order, zeros beyond their rows and features:
//   XP  [m][row tile][feature step of 32][lane][8]    row = 16 tile + lane % 16, features 32 step + 8 (lane / 16) ..
//   XTP [m][feature tile][row step of 32][lane][8]    feature = 16 tile + lane % 16, rows 32 step + 8 (lane / 16) ..
//   YL  [m][n32] labels (-1 beyond the rows)
// 64 rows x 64 features per workgroup, 16 bytes per thread and access in both directions.
__global__ void __launch_bounds__(256) pack_kernel(const unsigned short* __restrict__ X, const int* __restrict__ y,
                                                   const int* __restrict__ perm, unsigned short* __restrict__ XP,
                                                   unsigned short* __restrict__ XTP, int* __restrict__ YL, int rows, int p, int n,
                                                   int n32, int p32, int jtiles, unsigned* __restrict__ meeting)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *meeting = 0;    // (of the launch that follows)
    constexpr int TS = 72;                           // tile row stride in elements: 16-byte aligned rows
    __shared__ __align__(16) unsigned short tile[64 * TS];
    const int m = blockIdx.x / jtiles, jt = blockIdx.x % jtiles;
    const int j0 = jt * 64, c0 = blockIdx.y * 64;
    const int nb = min(n, rows - m * n);
    const int seg = threadIdx.x & 7, rq = threadIdx.x >> 3;      // 8 chunks x 32
    const int KS = p32 / 32, NS = n32 / 32;
    const size_t batch = (size_t)m * n32 * p32;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = rq + 32 * h, j = j0 + r, c = c0 + 8 * seg;
        const size_t row = (size_t)perm[(size_t)m * n + min(j, nb - 1)];
        uint4 v = *reinterpret_cast<const uint4*>(X + row * p + min(c, p - 8));
        if (j >= nb || c >= p) v = make_uint4(0, 0, 0, 0);
        *reinterpret_cast<uint4*>(&tile[r * TS + 8 * seg]) = v;
        if (j < n32 && c < p32) {
            const int at = ((j >> 4) * KS + (c >> 5)) * 64 + (j & 15) + 16 * ((c >> 3) & 3);
            *reinterpret_cast<uint4*>(XP + batch + (size_t)at * 8) = v;
        }
    }
    if (blockIdx.y == 0 && threadIdx.x < 64 && j0 + (int)threadIdx.x < n32) {
        const int j = j0 + threadIdx.x;
        YL[(size_t)m * n32 + j] = j < nb ? y[perm[(size_t)m * n + j]] : -1;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int cl = rq + 32 * h, f = c0 + cl, j = j0 + 8 * seg;
        unsigned short e[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = tile[(8 * seg + q) * TS + cl];
        uint4 w;
        w.x = e[0] | ((unsigned)e[1] << 16);
        w.y = e[2] | ((unsigned)e[3] << 16);
        w.z = e[4] | ((unsigned)e[5] << 16);
        w.w = e[6] | ((unsigned)e[7] << 16);
        if (f < p32 && j < n32) {
            const int at = ((f >> 4) * NS + (j >> 5)) * 64 + (f & 15) + 16 * ((j >> 3) & 3);
            *reinterpret_cast<uint4*>(XTP + batch + (size_t)at * 8) = w;
        }
    }
}

__device__ __forceinline__ bf16x8 as_frag(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// maximum / sum over the 16 lanes that hold one row's classes; every lane of them receives it
__device__ __forceinline__ float max16(float v)
{
    v = fmaxf(v, dpp_mov<0xB1>(v));
    v = fmaxf(v, dpp_mov<0x4E>(v));
    v = fmaxf(v, dpp_mov<0x141>(v));
    return fmaxf(v, dpp_mov<0x140>(v));
}
__device__ __forceinline__ float sum16(float v) { return group_sum(v, 16); }

// lane l16 & 3 = v keeps value v (by value: selects between elements of an array in memory become loads from it)
__device__ __forceinline__ float quad_select(float x0, float x1, float x2, float x3, int l16)
{
    const float a = (l16 & 1) ? x1 : x0, b = (l16 & 1) ? x3 : x2;
    return (l16 & 2) ? b : a;
}

__device__ __forceinline__ float as_float(unsigned v) { return __builtin_bit_cast(float, v); }

// Pairs of flagged words (one row's two numbers each) requested back to back and awaited together (see ll_load4).
constexpr int kPolls = 4;
__device__ __forceinline__ void load_pairs(const unsigned long long* const (&src)[1][4], u32x4 (&w)[1][4])
{
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\t"
                 "global_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\t"
                 "global_load_dwordx4 %3, %7, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[0][3])
                 : "v"(src[0][0]), "v"(src[0][1]), "v"(src[0][2]), "v"(src[0][3])
                 : "memory");
}
__device__ __forceinline__ void load_pairs(const unsigned long long* const (&src)[2][4], u32x4 (&w)[2][4])
{
    asm volatile("global_load_dwordx4 %0, %8, off sc1\n\t"
                 "global_load_dwordx4 %1, %9, off sc1\n\t"
                 "global_load_dwordx4 %2, %10, off sc1\n\t"
                 "global_load_dwordx4 %3, %11, off sc1\n\t"
                 "global_load_dwordx4 %4, %12, off sc1\n\t"
                 "global_load_dwordx4 %5, %13, off sc1\n\t"
                 "global_load_dwordx4 %6, %14, off sc1\n\t"
                 "global_load_dwordx4 %7, %15, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[0][3]), "=&v"(w[1][0]), "=&v"(w[1][1]), "=&v"(w[1][2]), "=&v"(w[1][3])
                 : "v"(src[0][0]), "v"(src[0][1]), "v"(src[0][2]), "v"(src[0][3]), "v"(src[1][0]), "v"(src[1][1]), "v"(src[1][2]), "v"(src[1][3])
                 : "memory");
}

// Fragments a wavefront has in flight for a phase with T tiles per step (each is 1 KiB): deep enough for a trip to L2.
constexpr int ring_depth(int T) { return T == 1 ? 8 : T == 2 ? 4 : 2; }

// f(T) with the smallest compiled T that covers a wavefront's `mine` tiles of at most TMAX (the host picks TMAX so that every
// wavefront has at least TMAX / 2, or 0 or 1 of 1): what the others do not have is neither requested nor multiplied.
template <int N> struct Tiles { static constexpr int count = N; };
template <int TMAX, class F>
__device__ __forceinline__ void with_tiles(int mine, F f)
{
    if constexpr (TMAX == 1) {
        if (mine > 0) f(Tiles<1>{});
    } else if constexpr (TMAX == 2) {
        if (mine > 1) f(Tiles<2>{});
        else f(Tiles<1>{});
    } else {
        if (mine > TMAX * 3 / 4) f(Tiles<TMAX>{});
        else if (mine > TMAX / 2) f(Tiles<TMAX * 3 / 4>{});
        else f(Tiles<TMAX / 2>{});
    }
}

// steps 0 .. n - 1 of a phase over a ring of D slots whose first D requests have been made.  The main loop refills a slot
// right after its use, without any branch (a branch around a load makes the compiler wait for all of them); the last steps
// ask for nothing that is not used.
template <int D, class Fetch, class Use>
__device__ __forceinline__ void stream(int n, Fetch fetch, Use use)
{
    int k = 0;
    for (; k + 2 * D <= n; k += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            use(k + d, d);
            fetch(k + d + D, d);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (k + d < n) {
            use(k + d, d);
            if (k + d + D < n) fetch(k + d + D, d);
        }
#pragma unroll
    for (int d = 0; d + 1 < D; ++d)
        if (k + D + d < n) use(k + D + d, d);
}

// The workgroups of a launch meet: every one counts itself in `meeting`, and the first one may close the meeting for all if some
// have not come in time.  Called by one thread of each workgroup: enter first, then (after whatever can be done meanwhile) wait.
enum { kTogether, kAlone, kLeave };
constexpr unsigned kClosed = 1u << 31;
__device__ __forceinline__ unsigned enter_meeting(unsigned* meeting)
{
    return __hip_atomic_fetch_add(meeting, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int wait_for_meeting(unsigned* meeting, unsigned ticket, unsigned G, long long ticks, PollGuard& guard)
{
    if (ticket & kClosed) return kLeave;
    const long long t0 = wall_clock64();
    unsigned seen = ticket + 1;
    guard.arm();
    while (seen != G) {
        if (seen & kClosed) return kLeave;
        if (ticket == 0 && wall_clock64() - t0 > ticks) {
            // (a workgroup that comes in between makes the exchange fail, and the loop looks again)
            if (__hip_atomic_compare_exchange_strong(meeting, &seen, seen | kClosed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return kAlone;
            continue;
        }
        if (guard.expired()) return kLeave;          // (the first one always decides long before this)
        seen = __hip_atomic_load(meeting, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return kTogether;
}

// u <- exp(u - mx) (0 for padding classes) for a tile's four rows per lane; mx and sum of every row over a workgroup's classes.
// (What is kept per row sits in lane l16 & 3 = v of each quad for row 4 lq + v; the residual hands it round.)
__device__ __forceinline__ void row_sums(f32x4 (&u)[NJ], int l16, float& mx, float& own)
{
    float sm[4], sv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float m = -FLT_MAX;                          // (finite: a row of nothing but -infinity gets zeros here, not NaN)
#pragma unroll
        for (int j = 0; j < NJ; ++j) m = fmaxf(m, u[j][v]);
        m = max16(m);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            u[j][v] = exp_neg(u[j][v] - m);
            sum += u[j][v];
        }
        sm[v] = m;
        sv[v] = sum16(sum);
    }
    mx = quad_select(sm[0], sm[1], sm[2], sm[3], l16);
    own = quad_select(sv[0], sv[1], sv[2], sv[3], l16);
}

// lanes 0 .. 3 of each 16 hold the maxima of a tile's rows row0 .. row0 + 3, lanes 4 .. 7 publish their sums
__device__ __forceinline__ void publish_rows(unsigned long long* out, int row0, int nb, int l16, float mx, float own, unsigned tag)
{
    const int row = row0 + (l16 & 3);
    if (l16 < 8 && row < nb) ll_store(out + 2 * row + (l16 >> 2), l16 < 4 ? mx : own, tag);
}

// How the threads of a workgroup share the polling: a thread per row, J groups of R threads that share the workgroups; for
// more than 512 rows two rows a thread, 512 apart.
struct PollShape {
    int R, J, pj, pr;
    __device__ __forceinline__ PollShape(int n32, int G, int tid)
    {
        R = (n32 + 63) / 64 * 64;
        J = min(G, max(1, kThreads / R));
        pj = tid / R;
        pr = tid - pj * R;
    }
};

// Every row's maximum and sum over the workgroups of this thread's share, into rmax and rsum [J][R].  False: given up.
template <int ROWS>
__device__ __forceinline__ bool collect_rows(const unsigned long long* in, int word_stride, int G, int nb, unsigned tag, const PollShape& ps,
                                             PollGuard& guard, float* rmax, float* rsum)
{
    if (ps.pj >= ps.J || ps.pr >= nb) return true;
    bool gave_up = false;
    float m[ROWS], sum[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) { m[i] = -FLT_MAX; sum[i] = 0.f; }
    for (int q0 = ps.pj; q0 < G && !gave_up; q0 += kPolls * ps.J) {
        const unsigned long long* src[ROWS][kPolls];
        u32x4 word[ROWS][kPolls];
#pragma unroll
        for (int i = 0; i < ROWS; ++i)               // (a second row beyond the mini-batch: its last one again)
#pragma unroll
            for (int q = 0; q < kPolls; ++q) src[i][q] = in + (size_t)min(q0 + q * ps.J, G - 1) * word_stride + 2 * min(ps.pr + kThreads * i, nb - 1);
        guard.arm();
        while (true) {
            load_pairs(src, word);
            bool ok = true;
#pragma unroll
            for (int i = 0; i < ROWS; ++i)
#pragma unroll
                for (int q = 0; q < kPolls; ++q) ok = ok && word[i][q].y == tag && word[i][q].w == tag;
            if (ok) break;
            if (guard.expired()) { gave_up = true; break; }
        }
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            float v[kPolls], top = m[i];
#pragma unroll
            for (int q = 0; q < kPolls; ++q) {
                v[q] = q0 + q * ps.J < G ? as_float(word[i][q].x) : -INFINITY;
                top = fmaxf(top, v[q]);
            }
            sum[i] *= exp_neg(m[i] - top);
#pragma unroll
            for (int q = 0; q < kPolls; ++q) sum[i] = fmaf(as_float(word[i][q].z), exp_neg(v[q] - top), sum[i]);
            m[i] = top;
        }
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
        if (ps.pr + kThreads * i < nb) {
            rmax[ps.pj * ps.R + ps.pr + kThreads * i] = m[i];
            rsum[ps.pj * ps.R + ps.pr + kThreads * i] = sum[i];
        }
    return !gave_up;
}

// e^(mx - top) / sum with top and sum of row r over all workgroups, where mx is its maximum here
__device__ __forceinline__ float row_scale(const float* rmax, const float* rsum, const PollShape& ps, int r, int l16, float mx)
{
    float top, sum;
    if (ps.J == 1) {
        top = rmax[r];
        sum = rsum[r];
    } else {
        // the four lanes that keep the same row take every fourth share, then meet
        const int j0 = min(l16 >> 2, ps.J - 1) * ps.R + r, j1 = min((l16 >> 2) + 4, ps.J - 1) * ps.R + r;
        const float v0 = (l16 >> 2) < ps.J ? rmax[j0] : -INFINITY, v1 = (l16 >> 2) + 4 < ps.J ? rmax[j1] : -INFINITY;
        top = fmaxf(fmaxf(v0, v1), -FLT_MAX);
        top = fmaxf(top, dpp_mov<0x124>(top));
        top = fmaxf(top, dpp_mov<0x128>(top));
        sum = rsum[j0] * exp_neg(v0 - top) + rsum[j1] * exp_neg(v1 - top);
        sum += dpp_mov<0x124>(sum);
        sum += dpp_mov<0x128>(sum);
    }
    return exp_neg(mx - top) / sum;
}

// residual of a tile's rows r0 .. r0 + 3 per lane (scale and label as row_sums keeps them), transposed into shared memory
__device__ __forceinline__ void residual_tile(const f32x4 (&u)[NJ], float scale, int label, int r0, int c0, int nb, int C, int l16, unsigned short* Rt, int rs)
{
    const float f[4] = {dpp_mov<0x00>(scale), dpp_mov<0x55>(scale), dpp_mov<0xAA>(scale), dpp_mov<0xFF>(scale)};
    const float lq_ = __builtin_bit_cast(float, label);
    const int y[4] = {__builtin_bit_cast(int, dpp_mov<0x00>(lq_)), __builtin_bit_cast(int, dpp_mov<0x55>(lq_)),
                      __builtin_bit_cast(int, dpp_mov<0xAA>(lq_)), __builtin_bit_cast(int, dpp_mov<0xFF>(lq_))};
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        float r[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = c0 + 16 * j + l16;
            r[v] = u[j][v] * f[v] - (c == y[v] ? 1.f : 0.f);
            if (r0 + v >= nb || c >= C) r[v] = 0.f;
        }
        *reinterpret_cast<uint2*>(&Rt[(16 * j + l16) * rs + r0]) = to_bf16x4(r);
    }
}

// state of the update rule of features f0 .. f0 + 3 and class c, in memory laid out like W (loads from clamped addresses)
__device__ __forceinline__ void load_state(const SoftmaxChainArgs& a, int f0, int c, float (&m)[4], float (&sv)[4])
{
    const float* second = a.opt.kind == kOptAdam ? a.opt.s : a.opt.m;        // (no second array: the first again, not written)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const size_t at = (size_t)min(f0 + v, a.p - 1) * a.ldw + c;
        m[v] = a.opt.m[at];
        sv[v] = second[at];
    }
}
__device__ __forceinline__ void store_state(const SoftmaxChainArgs& a, int f0, int c, const float (&m)[4], const float (&sv)[4])
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (f0 + v < a.p && c < a.C) {
            const size_t at = (size_t)(f0 + v) * a.ldw + c;
            a.opt.m[at] = m[v];
            if (a.opt.kind == kOptAdam) a.opt.s[at] = sv[v];
        }
}

// The whole pass in one workgroup: every share of 16 classes in turn does what its workgroup would do, W and the state in memory, the
// bf16 copy in memory as well.  Only where the workgroups could not be resident together, so nothing here is done for speed but the
// sums are those of softmax_chain_kernel, in the same order.
template <bool OPT>
__device__ __forceinline__ void pass_alone(const SoftmaxChainArgs& a, int G, unsigned short* Wt, unsigned short* Rt, float* rmax, float* rsum)
{
    const int KS = a.p32 / 32, NS = a.n32 / 32, ws = a.p32 + 8, rs = a.n32 + 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const size_t batch = (size_t)a.n32 * a.p32, words_set = (size_t)G * a.word_stride;
    const PollShape ps(a.n32, G, tid);
    PollGuard guard{a.sync + 1, a.timeout_ticks, 0, 0};
    __shared__ int s_gave_up;
    if (tid == 0) s_gave_up = 0;
    __syncthreads();
    for (int s = 0; s < a.M; ++s) {
        const int nb = min(a.n, a.rows - s * a.n);
        const unsigned tag = a.tag_base + (unsigned)s + 1u;
        const float alpha = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        unsigned long long* words = a.words + (size_t)(s & 1) * words_set;
        auto load_w = [&](int c0) {                  // the bf16 copy of a share's columns
            const int chunks = a.p32 / 8;
            for (int e = tid; e < kClasses * chunks; e += kThreads) {
                const int c = e / chunks, f = 8 * (e - c * chunks);
                *reinterpret_cast<uint4*>(&Wt[c * ws + f]) = *reinterpret_cast<const uint4*>(a.WbT + (size_t)(c0 + c) * a.ldwt + f);
            }
            __syncthreads();
        };
        auto logits = [&](int rt, int c0, f32x4 (&u)[NJ]) {
            const unsigned short* x = a.XP + batch * s + (size_t)rt * KS * 512 + lane * 8;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float z = c0 + 16 * j + l16 < a.C ? 0.f : -INFINITY;
                u[j] = f32x4{z, z, z, z};
            }
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    u[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(*reinterpret_cast<const uint4*>(x + k * 512)),
                                                                   as_frag(*reinterpret_cast<const uint4*>(&Wt[(16 * j + l16) * ws + 32 * k + 8 * lq])), u[j], 0, 0, 0);
        };
        for (int g = 0; g < G; ++g) {
            load_w(g * kClasses);
            for (int rt = wave; rt < a.n32 / 16; rt += kWaves) {
                f32x4 u[NJ];
                float mx, own;
                logits(rt, g * kClasses, u);
                row_sums(u, l16, mx, own);
                publish_rows(words + (size_t)g * a.word_stride, 16 * rt + 4 * lq, nb, l16, mx, own, tag);
            }
            __syncthreads();
        }
        if (!collect_rows<2>(words, a.word_stride, G, nb, tag, ps, guard, rmax, rsum)) s_gave_up = 1;
        __syncthreads();
        if (s_gave_up) return;
        const float inv_nb = 1.f / (float)nb, scale = alpha * inv_nb;
        float oc1 = 1.f, oc2 = 1.f;
        if (OPT && a.opt.kind == kOptAdam) opt_corrections(a.opt, a.opt.k_base + s + 1, oc1, oc2);
        for (int g = 0; g < G; ++g) {
            const int c0 = g * kClasses;
            load_w(c0);
            for (int rt = wave; rt < a.n32 / 16; rt += kWaves) {
                f32x4 u[NJ];
                float mx, own;
                logits(rt, c0, u);
                row_sums(u, l16, mx, own);
                const int r0 = 16 * rt + 4 * lq;
                const int label = a.YL[(size_t)s * a.n32 + r0 + (l16 & 3)];
                residual_tile(u, row_scale(rmax, rsum, ps, min(r0 + (l16 & 3), nb - 1), l16, mx), label, r0, c0, nb, a.C, l16, Rt, rs);
            }
            __syncthreads();
            for (int ft = wave; ft < a.p32 / 16; ft += kWaves) {
                const unsigned short* x = a.XTP + batch * s + (size_t)ft * NS * 512 + lane * 8;
                const int f0 = 16 * ft + 4 * lq;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                    for (int k = 0; k < NS; ++k)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(*reinterpret_cast<const uint4*>(x + k * 512)),
                                                                      as_frag(*reinterpret_cast<const uint4*>(&Rt[(16 * j + l16) * rs + 32 * k + 8 * lq])), acc, 0, 0, 0);
                    const int c = c0 + 16 * j + l16;
                    float w[4], m[4], sv[4];
                    if constexpr (OPT) load_state(a, f0, c, m, sv);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        w[v] = 0.f;
                        if (f0 + v >= a.p || c >= a.C) continue;
                        w[v] = a.W[(size_t)(f0 + v) * a.ldw + c];
                        if constexpr (OPT) w[v] = opt_update(a.opt, w[v], acc[v] * inv_nb, alpha, m[v], sv[v], oc1, oc2);
                        else w[v] -= scale * acc[v];
                        a.W[(size_t)(f0 + v) * a.ldw + c] = w[v];
                    }
                    if constexpr (OPT) store_state(a, f0, c, m, sv);
                    *reinterpret_cast<uint2*>(a.WbT + (size_t)c * a.ldwt + f0) = to_bf16x4(w);
                }
            }
            __syncthreads();
        }
    }
}

// RT, FT: row tiles and feature tiles per wavefront (tile w, w + 8, ... belong to wavefront w); OPT: an update rule other
// than the plain step.
template <int RT, int FT, bool OPT>
__global__ void __launch_bounds__(kThreads, 2) softmax_chain_kernel(SoftmaxChainArgs a)
{
    constexpr int DL = ring_depth(RT), DG = ring_depth(FT);
    // when the first operands of a phase are asked for: as soon as the same phase of the update before has let go of the ring
    // (they come from memory the first time) if the registers allow, else later
    constexpr bool EARLY_L = RT <= 2 && FT <= 4, EARLY_G = FT <= 2;
    extern __shared__ __align__(16) unsigned short smem[];
    const int KS = a.p32 / 32, NS = a.n32 / 32;
    const int ws = a.p32 + 8, rs = a.n32 + 8;        // row strides: 16 bytes past a multiple of 64, so that eight rows fall on different banks
    unsigned short* Wt = smem;                       // [16][ws] bf16 copy of W, class-major
    unsigned short* Rt = Wt + kClasses * ws;         // [16][rs] residual, class-major
    float* rmax = reinterpret_cast<float*>(Rt + kClasses * rs);  // [J][R] a row's maximum over the classes of a share of the workgroups
    float* rsum = rmax + kMaxRows;                               // [J][R] ... and its sum of e^(u - that)
    __shared__ int s_abort, s_role;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int G = gridDim.x, g = blockIdx.x;
    const int c0 = g * kClasses;
    const int n_rt = a.n32 / 16, n_ft = a.p32 / 16;
    const size_t batch = (size_t)a.n32 * a.p32;      // elements of a mini-batch in XP and XTP

    unsigned ticket = 0;
    if (G > 1 && a.meeting_ticks == 0) {
        if (g == 0) pass_alone<OPT>(a, G, Wt, Rt, rmax, rsum);
        return;
    }
    if (tid == 0) {
        s_abort = 0;
        if (G > 1) ticket = enter_meeting(a.meeting);
    }
    // master weights: lane holds class c0 + 16 j + l16, features 16 tile + 4 lq + v.  Classes beyond C stay zero whatever their
    // gradient is (0 x Inf is NaN): their logits go through the same row sums as the others', as -infinity.
    float w[FT][NJ][4];
#pragma unroll
    for (int t = 0; t < FT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int f0 = 16 * (wave + kWaves * t) + 4 * lq, c = c0 + 16 * j + l16;
#pragma unroll
            for (int v = 0; v < 4; ++v) w[t][j][v] = f0 + v < a.p && c < a.C ? a.W[(size_t)(f0 + v) * a.ldw + c] : 0.f;
            if (wave + kWaves * t < n_ft) *reinterpret_cast<uint2*>(&Wt[(16 * j + l16) * ws + f0]) = to_bf16x4(w[t][j]);
        }

    unsigned real[NJ];                               // all bits for a class, none for one that fills up the workgroup
#pragma unroll
    for (int j = 0; j < NJ; ++j) real[j] = c0 + 16 * j + l16 < a.C ? ~0u : 0u;

    // state of the update rule, laid out like W: in registers beside W where there is room, else read and written in memory
    constexpr bool STATE = OPT && FT <= 2;
    float om[STATE ? FT : 1][NJ][4], os[STATE ? FT : 1][NJ][4];
    if constexpr (STATE) {
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j) load_state(a, 16 * (wave + kWaves * t) + 4 * lq, c0 + 16 * j + l16, om[t][j], os[t][j]);
    }

    // operand streams: wavefront w's tiles, clamped to the last one (what a clamped tile gives is dropped)
    unsigned lo[RT], go[FT];
#pragma unroll
    for (int t = 0; t < RT; ++t) lo[t] = (unsigned)(min(wave + kWaves * t, n_rt - 1) * KS * 512 + lane * 8);
#pragma unroll
    for (int t = 0; t < FT; ++t) go[t] = (unsigned)(min(wave + kWaves * t, n_ft - 1) * NS * 512 + lane * 8);
    uint4 la[DL][RT], ga[DG][FT];
    // tiles of this wavefront
    const int my_rt = max(0, (n_rt - wave + kWaves - 1) / kWaves), my_ft = max(0, (n_ft - wave + kWaves - 1) / kWaves);
    auto fetch_l = [&](auto T, const unsigned short* x, int k, int d) {
        const int kc = min(k, KS - 1) * 512;
#pragma unroll
        for (int t = 0; t < decltype(T)::count; ++t) la[d][t] = *reinterpret_cast<const uint4*>(x + lo[t] + kc);
    };
    auto fetch_g = [&](auto T, const unsigned short* x, int k, int d) {
        const int kc = min(k, NS - 1) * 512;
#pragma unroll
        for (int t = 0; t < decltype(T)::count; ++t) ga[d][t] = *reinterpret_cast<const uint4*>(x + go[t] + kc);
    };
    // the first requests of a phase over the mini-batch at x
    auto start_l = [&](const unsigned short* x) {
        with_tiles<RT>(my_rt, [&](auto T) {
#pragma unroll
            for (int d = 0; d < DL; ++d) fetch_l(T, x, d, d);
        });
    };
    auto start_g = [&](const unsigned short* x) {
        with_tiles<FT>(my_ft, [&](auto T) {
#pragma unroll
            for (int d = 0; d < DG; ++d) fetch_g(T, x, d, d);
        });
    };
    start_l(a.XP);
    if constexpr (EARLY_G) start_g(a.XTP);

    constexpr int ROWS = RT == kMaxTiles ? 2 : 1;
    const PollShape ps(a.n32, G, tid);
    const size_t words_set = (size_t)G * a.word_stride;
    PollGuard guard{a.sync + 1, a.timeout_ticks, 0, 0};
    if (G > 1 && tid == 0) s_role = wait_for_meeting(a.meeting, ticket, (unsigned)G, a.meeting_ticks, guard);
    __syncthreads();
    if (G > 1 && s_role != kTogether) {
        if (s_role == kAlone) pass_alone<OPT>(a, G, Wt, Rt, rmax, rsum);
        return;
    }

    for (int s = 0; s < a.M; ++s) {
        const int nb = min(a.n, a.rows - s * a.n);
        const unsigned tag = a.tag_base + (unsigned)s + 1u;
        const unsigned short* xt = a.XTP + batch * s;
        const float alpha = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        int label[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t)
            label[t] = a.YL[(size_t)s * a.n32 + 16 * min(wave + kWaves * t, n_rt - 1) + 4 * lq + (l16 & 3)];
        // logits of this workgroup's classes
        f32x4 u[RT][NJ];
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float z = c0 + 16 * j + l16 < a.C ? 0.f : -INFINITY;    // padding classes count as -infinity
                u[t][j] = f32x4{z, z, z, z};
            }
        with_tiles<RT>(my_rt, [&](auto T) {
            const unsigned short* x = a.XP + batch * s;
            stream<DL>(KS, [&](int k, int d) { fetch_l(T, x, k, d); }, [&](int k, int d) {
                bf16x8 b[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) b[j] = as_frag(*reinterpret_cast<const uint4*>(&Wt[(16 * j + l16) * ws + 32 * k + 8 * lq]));
#pragma unroll
                for (int t = 0; t < decltype(T)::count; ++t)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) u[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(la[d][t]), b[j], u[t][j], 0, 0, 0);
            });
        });
        const unsigned short* next = a.XP + batch * min(s + 1, a.M - 1);
        if constexpr (EARLY_L) start_l(next);
        if constexpr (!EARLY_G) start_g(xt);

        float mx[RT], own[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (t >= my_rt) break;
            row_sums(u[t], l16, mx[t], own[t]);
            __builtin_amdgcn_sched_barrier(0);           // (one tile's exponentials at a time: all of them together take too many registers)
        }
        if (G > 1) {
            unsigned long long* words = a.words + (size_t)(s & 1) * words_set;
#pragma unroll
            for (int t = 0; t < RT; ++t)
                if (t < my_rt) publish_rows(words + (size_t)g * a.word_stride, 16 * (wave + kWaves * t) + 4 * lq, nb, l16, mx[t], own[t], tag);
            __builtin_amdgcn_s_sleep(8);                 // (0.2 us: a poll sent at once comes back a moment before the words do)
            if (!collect_rows<ROWS>(words, a.word_stride, G, nb, tag, ps, guard, rmax, rsum)) s_abort = 1;
            __syncthreads();
            if (s_abort) return;                    // (every thread sees the same value: it is not written after this barrier)
        }
        // residual, transposed into shared memory
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (t >= my_rt) break;
            const int r0 = 16 * (wave + kWaves * t) + 4 * lq;
            const float scale = G > 1 ? row_scale(rmax, rsum, ps, min(r0 + (l16 & 3), nb - 1), l16, mx[t]) : 1.f / own[t];
            residual_tile(u[t], scale, label[t], r0, c0, nb, a.C, l16, Rt, rs);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();

        if constexpr (!EARLY_L && FT < 8) start_l(next);
        // gradient of this workgroup's columns
        f32x4 acc[FT][NJ];
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        with_tiles<FT>(my_ft, [&](auto T) {
            stream<DG>(NS, [&](int k, int d) { fetch_g(T, xt, k, d); }, [&](int k, int d) {
                bf16x8 b[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) b[j] = as_frag(*reinterpret_cast<const uint4*>(&Rt[(16 * j + l16) * rs + 32 * k + 8 * lq]));
#pragma unroll
                for (int t = 0; t < decltype(T)::count; ++t)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(ga[d][t]), b[j], acc[t][j], 0, 0, 0);
            });
        });
        if constexpr (EARLY_G) start_g(a.XTP + batch * min(s + 1, a.M - 1));
        if constexpr (!EARLY_L && FT == 8) start_l(next);
        // update, and the bf16 copy the next logits read
        const float inv_nb = 1.f / (float)nb, scale = alpha * inv_nb;
        float oc1 = 1.f, oc2 = 1.f;
        if (OPT && a.opt.kind == kOptAdam) opt_corrections(a.opt, a.opt.k_base + s + 1, oc1, oc2);
#pragma unroll
        for (int t = 0; t < FT; ++t) {
            if (t >= my_ft) break;
            const int f0 = 16 * (wave + kWaves * t) + 4 * lq;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int c = c0 + 16 * j + l16;
                if constexpr (!OPT) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[t][j][v] = as_float(__builtin_bit_cast(unsigned, w[t][j][v] - scale * acc[t][j][v]) & real[j]);
                } else {
                    float m[4], sv[4];
                    if constexpr (STATE) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) { m[v] = om[t][j][v]; sv[v] = os[t][j][v]; }
                    } else {
                        load_state(a, f0, c, m, sv);    // (all of a tile's at once, from clamped addresses)
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (f0 + v < a.p && c < a.C) w[t][j][v] = opt_update(a.opt, w[t][j][v], acc[t][j][v] * inv_nb, alpha, m[v], sv[v], oc1, oc2);
                    if constexpr (STATE) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) { om[t][j][v] = m[v]; os[t][j][v] = sv[v]; }
                    } else {
                        store_state(a, f0, c, m, sv);
                    }
                }
                *reinterpret_cast<uint2*>(&Wt[(16 * j + l16) * ws + f0]) = to_bf16x4(w[t][j]);
            }
        }
        __syncthreads();
    }

    // W and its bf16 copy (and the state) for whatever comes next
#pragma unroll
    for (int t = 0; t < FT; ++t) {
        const int f0 = 16 * (wave + kWaves * t) + 4 * lq;
        if constexpr (OPT && STATE) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) store_state(a, f0, c0 + 16 * j + l16, om[t][j], os[t][j]);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (f0 + v < a.p) a.W[(size_t)(f0 + v) * a.ldw + c0 + 16 * j + l16] = w[t][j][v];
    }
    const int chunks = a.p32 / 8;
    for (int e = tid; e < kClasses * chunks; e += kThreads) {
        const int c = e / chunks, f = 8 * (e - c * chunks);
        *reinterpret_cast<uint4*>(a.WbT + (size_t)(c0 + c) * a.ldwt + f) = *reinterpret_cast<const uint4*>(&Wt[c * ws + f]);
    }
}

int round32(int64_t v) { return (int)((v + 31) / 32 * 32); }

size_t chain_lds(int n32, int p32)
{
    return (size_t)kClasses * (size_t)(p32 + 8 + n32 + 8) * 2 + 2 * kMaxRows * 4;
}

// tiles per wavefront, rounded up to a compiled variant: index into {1, 2, 4, 8}
int tile_variant(int padded)
{
    const int t = (padded / 16 + kWaves - 1) / kWaves;
    return t <= 1 ? 0 : t <= 2 ? 1 : t <= 4 ? 2 : 3;
}

typedef void (*ChainKernel)(SoftmaxChainArgs);

template <bool OPT>
ChainKernel chain_kernel(int rt, int ft)
{
#define ROW(R) softmax_chain_kernel<R, 1, OPT>, softmax_chain_kernel<R, 2, OPT>, softmax_chain_kernel<R, 4, OPT>
    // (eight tiles both ways would be more than 512 rows of more than 512 features; the update rules with state take up to 512 features)
    static const ChainKernel table[4][3] = {{ROW(1)}, {ROW(2)}, {ROW(4)}, {ROW(8)}};
#undef ROW
    if (ft < 3) return table[rt][ft];
    if constexpr (!OPT) {
        static const ChainKernel wide[4] = {softmax_chain_kernel<1, 8, false>, softmax_chain_kernel<2, 8, false>, softmax_chain_kernel<4, 8, false>, nullptr};
        return wide[rt];
    }
    return nullptr;
}

ChainKernel chain_kernel(bool opt, int rt, int ft) { return opt ? chain_kernel<true>(rt, ft) : chain_kernel<false>(rt, ft); }

}  // namespace

// Where one kernel is the faster way (us per update, this kernel / three launches): 3.2 / 14.4 at n = 128, p = 64, C = 10;
// 6.3 / 16.9 at 100, 200, 130; 10.3 / 21.8 at 320, 320, 45; 11.1 / 22.0 at 256, 256, 1000; at n p = 2^18 what a workgroup reads
// per update has caught up: 13.4 / 22.2 at 512, 512, 10, but 17.9 / 21.1 at 256, 1000, 200 and 24.9 / 28.0 at 1000, 256, 300.
// With state (momentum, NAG, Adam) registers run out earlier: 16.2 / 31.3 at 320, 320, 45, 30.6 / 34.5 at 600, 320, 45 and
// 44.9 / 30.7 at 256, 1000, 10 (Adam).
bool softmax_chain_eligible(int64_t p, int64_t n, int64_t C, bool opt)
{
    if (p > kMaxRows || n > kMaxRows || C > 2048) return false;
    if (opt) return p <= kMaxRows / 2 && p * n <= (int64_t(1) << 17);
    return p * n <= (int64_t(1) << 18) && !(p > kMaxRows / 2 && n > kMaxRows / 2);
}

size_t softmax_chain_pack_bytes(int64_t p, int64_t n, int64_t batches)
{
    return (size_t)batches * ((size_t)round32(n) * round32(p) * 4 + (size_t)round32(n) * 4);
}

size_t softmax_chain_words_bytes(int64_t n, int64_t C)
{
    return (size_t)2 * ((C + kClasses - 1) / kClasses) * round32(n) * 16;
}

hipError_t softmax_chain_prepare(int64_t p, int64_t n, int64_t C, bool opt, int num_cus, bool* fits)
{
    *fits = false;
    const int G = (int)((C + kClasses - 1) / kClasses);
    const int ft = tile_variant(round32(p));
    // (a shorter last buffer has smaller mini-batches and may run a variant with fewer row tiles)
    for (int rt = tile_variant(round32(n)); rt >= 0; --rt) {
        if (!chain_kernel(opt, rt, ft)) return hipSuccess;
        const void* k = reinterpret_cast<const void*>(chain_kernel(opt, rt, ft));
        const size_t lds = chain_lds(round32(n), round32(p));
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kThreads, lds);
        if (e != hipSuccess) return e;
        if ((int64_t)per_cu * num_cus < G) return hipSuccess;
    }
    *fits = true;
    return hipSuccess;
}

hipError_t softmax_chain_pass(const void* X, const int32_t* y, const int32_t* perm, void* pack, SoftmaxChainArgs a, hipStream_t stream)
{
    a.n32 = round32(a.n);
    a.p32 = round32(a.p);
    a.M = (a.rows + a.n - 1) / a.n;
    a.word_stride = 2 * a.n32;
    if (a.n32 > kMaxRows || a.p32 > kMaxRows || a.C > a.ldw) return hipErrorInvalidValue;
    const size_t half = (size_t)a.M * a.n32 * a.p32;
    unsigned short* xp = static_cast<unsigned short*>(pack);
    unsigned short* xtp = xp + half;
    int* yl = reinterpret_cast<int*>(xtp + half);
    a.XP = xp; a.XTP = xtp; a.YL = yl;
    const int jtiles = (a.n32 + 63) / 64;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)(a.M * jtiles), (unsigned)((a.p32 + 63) / 64)), dim3(256), 0, stream,
                       static_cast<const unsigned short*>(X), y, perm, xp, xtp, yl, a.rows, a.p, a.n, a.n32, a.p32, jtiles, a.meeting);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int G = (a.C + kClasses - 1) / kClasses;
    const ChainKernel k = chain_kernel(a.opt.kind != kOptSgd, tile_variant(a.n32), tile_variant(a.p32));
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((unsigned)G), dim3(kThreads), chain_lds(a.n32, a.p32), stream, a);
    return hipGetLastError();
}

}  // namespace bmgd
