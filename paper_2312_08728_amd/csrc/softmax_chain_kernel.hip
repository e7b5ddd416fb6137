// Softmax regression on small mini-batches: all updates of a pass in one persistent kernel.
//
// Three launches per update (logits, residual, gradient + update; softmax_kernels.hip) cost 14 us even for 16 rows, and 35 us for 1,000 rows
// of 256 features and 2,000 classes: each small kernel is a chain of dependent trips to memory, and the weights go out to memory and
// back between them.  Here the CLASSES are split over workgroups, 16 to each: a workgroup keeps its columns of W for the whole pass (fp32
// master in registers, in the accumulator layout of its gradient tiles; bf16 copy in shared memory, where the logits read it), so
//     U = X_b W[:, mine]                    needs all features of a row, but nothing of other workgroups;
//     R = softmax_rows(U) - onehot(y)       needs one number per row from each of the others, its sum of e^u over their classes
//                                           (as 2^k f, see exp2_rest);
//     W[:, mine] -= (alpha / n_b) X_b' R    is again the workgroup's own.
// Those sums are all that is exchanged (a flagged word each, store_sum: one trip over the fabric per update; none at all for
// up to 16 classes).  The mini-batch is read by every workgroup from its L2, twice per update (rows for the
// logits, transposed for the gradient), laid out once per pass in the order in which the matrix instructions take their
// operands (pack_kernel): one contiguous KiB per load instruction, requested ahead, the next update's first ones before
// this update's gradient.
//
// The exchange needs all workgroups of the launch resident at once, which work of other streams and processes can prevent.  So they
// meet before the first update (wait_for_meeting): where they do not within a given time, one of them makes the whole pass by
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
                                                   // everywhere: twice the exponentials and registers)
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

constexpr float kLog2e = 1.44269502f, kLog2eLo = 1.92596299e-8f;   // log2 e in two parts
constexpr float kRound = 12582912.f;                // 1.5 x 2^23: the last bit of a sum with it is 1

// 2^n f for whole n <= 0; 0 for n = -infinity and, as between two sums that are NaN (store_sum), for n = NaN
__device__ __forceinline__ float scale_down(float f, float n)
{
    return __builtin_ldexpf(f, __builtin_bit_cast(int, fmaxf(n, -300.f) + kRound) - __builtin_bit_cast(int, kRound));
}

// e^x for x <= 0 or NaN: 2^n 2^f with n = x log2 e rounded to a whole number and f what is left, in eight
// instructions.  As good as expf: over [-87, 0] a relative error of at most 8.5e-8 (2.7e-8 rms; expf 8.4e-8 and 2.6e-8), and the
// subnormal numbers below to their last unit.
__device__ __forceinline__ float exp_neg(float x)
{
    x = x < -200.f ? -200.f : x;                     // (keeps a NaN; e^-200 is 0)
    const float t = fmaf(x, kLog2e, kRound);
    const float f = fmaf(x, kLog2eLo, fmaf(x, kLog2e, kRound - t));
    return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), __builtin_bit_cast(int, t) - __builtin_bit_cast(int, kRound));
}

// A row's sum of e^u over some classes is kept as 2^k f, k a whole number near their maximum times log2 e: exact to the last bits of
// f whatever the size of the logits (the log of the sum would be off by the spacing of fp32 there), and sums of several workgroups
// add up without an exponential.  e^m = 2^k * (what exp2_rest returns); from |k| = 2^23 on, where neighbouring numbers are further
// apart than that, the rest is left out.
__device__ __forceinline__ float exp2_rest(float m, float& k)
{
    k = fminf(fmaxf(rintf(m * kLog2e), -FLT_MAX), FLT_MAX);
    const float rest = fmaf(m, kLog2eLo, fmaf(m, kLog2e, -k));
    return __builtin_amdgcn_exp2f(fabsf(k) < 8388608.f ? rest : 0.f);
}

// The mini-batches of a pass in operand order, zeros beyond their rows and features:
//   XP  [m][row tile][feature step of 32][lane][8]    row = 16 tile + lane % 16, features 32 step + 8 (lane / 16) ..
//   XTP [m][feature tile][row step of 32][lane][8]    feature = 16 tile + lane % 16, rows 32 step + 8 (lane / 16) ..
//   YL  [m][n32] labels (-1 beyond the rows)
// 64 rows x 64 features per workgroup, 16 bytes per thread and access in both directions.
__global__ void __launch_bounds__(256) pack_kernel(const unsigned short* __restrict__ X, const int* __restrict__ y,
                                                   const int* __restrict__ perm, unsigned short* __restrict__ XP,
                                                   unsigned short* __restrict__ XTP, int* __restrict__ YL, int rows, int p, int n,
                                                   int n32, int p32, int jtiles, unsigned* __restrict__ meeting,
                                                   unsigned long long* __restrict__ words, int nwords)
{
    // for the launch that follows: nobody has come to the meeting, no word has been written
    const int64_t first = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
    if (first == 0) *meeting = 0;
    for (int64_t i = first; i < nwords; i += (int64_t)gridDim.x * gridDim.y * blockDim.x) words[i] = 0;
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

// What a workgroup tells the others about a row, in one 64-bit word that is written and read as a whole: its sum 2^k f as k (32 bits)
// and f (26), and a tag (6).  f lies between 0.7 and 23; f / 32 is positive, at least 2^-7 and below 2, so its fp32 pattern without
// the six leading bits, which are always the same, is all of it.  A sum of 0 (all classes at -infinity) is k = -infinity, NaN is
// k = +infinity: the first adds nothing, the second takes all there is from the others, and 0 / 0 is NaN.
// Words are cleared before a pass; every update writes all rows of its mini-batch, and only the last one can have fewer.  So a word
// of another update that a reader can find is that of two updates before, or none, and six bits tell it from the one awaited.
// (Two words a row with 32-bit tags took 28.2 against 22.4 us per update at n = 512, p = 256, C = 2000.)
constexpr unsigned kSumBits = 26, kSumMask = (1u << kSumBits) - 1u, kSumBase = 0x3C000000u;
constexpr float kSumScale = 1.f / 32.f;
__device__ __forceinline__ unsigned row_tag(int s) { return (unsigned)s % 63u + 1u; }
__device__ __forceinline__ void store_sum(unsigned long long* dst, float k, float f, unsigned tag)
{
    const unsigned low = (__builtin_bit_cast(unsigned, f * kSumScale) & kSumMask) | tag << kSumBits;
    __hip_atomic_store(dst, (unsigned long long)__builtin_bit_cast(unsigned, k) << 32 | low, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float sum_of(unsigned low) { return as_float((low & kSumMask) | kSumBase); }     // (of 2^5 sums)

// Pairs of words (two neighbouring rows each) requested back to back and awaited together (see ll_load4).
__device__ __forceinline__ void load_pairs(const unsigned long long* const (&src)[1], u32x4 (&w)[1])
{
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(w[0])
                 : "v"(src[0])
                 : "memory");
}
__device__ __forceinline__ void load_pairs(const unsigned long long* const (&src)[2], u32x4 (&w)[2])
{
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\t"
                 "global_load_dwordx4 %1, %3, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1])
                 : "v"(src[0]), "v"(src[1])
                 : "memory");
}
__device__ __forceinline__ void load_pairs(const unsigned long long* const (&src)[4], u32x4 (&w)[4])
{
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\t"
                 "global_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\t"
                 "global_load_dwordx4 %3, %7, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(src[0]), "v"(src[1]), "v"(src[2]), "v"(src[3])
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

// u <- exp(u - maximum) (0 for padding classes) for a tile's four rows per lane; each row's sum of e^u over a workgroup's classes is
// 2^k rest total.  (What is kept per row sits in lane l16 & 3 = v of each quad for row 4 lq + v; the residual hands it round.)
__device__ __forceinline__ void row_sums(f32x4 (&u)[NJ], int l16, float& k, float& rest, float& total)
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
    rest = exp2_rest(quad_select(sm[0], sm[1], sm[2], sm[3], l16), k);
    total = quad_select(sv[0], sv[1], sv[2], sv[3], l16);
    k = total > 0.f ? k : total == 0.f ? -INFINITY : INFINITY;
}

// lanes 0 .. 3 of each 16 publish a tile's rows row0 .. row0 + 3
__device__ __forceinline__ void publish_rows(unsigned long long* out, int row0, int nb, int l16, float k, float f, unsigned tag)
{
    const int row = row0 + (l16 & 3);
    if (l16 < 4 && row < nb) store_sum(out + row, k, f, tag);
}

// How the threads of a workgroup share the polling: a thread takes two neighbouring rows, J groups of R / 2 threads share the
// workgroups.
struct PollShape {
    int R, J, pj, pr;
    __device__ __forceinline__ PollShape(int n32, int G, int tid)
    {
        R = (n32 + 127) / 128 * 128;
        J = min(G, kThreads / (R / 2));
        pj = tid / (R / 2);
        pr = 2 * (tid - pj * (R / 2));
    }
};

// Every row's sum over the workgroups of this thread's share, into rk and rf [J][R], POLLS of them a trip.  False: given up.
template <int POLLS>
__device__ __forceinline__ bool collect_rows(const unsigned long long* in, int word_stride, int G, int nb, unsigned tag, const PollShape& ps,
                                             PollGuard& guard, float* rk, float* rf)
{
    if (ps.pj >= ps.J || ps.pr >= nb) return true;
    bool gave_up = false;
    const bool second = ps.pr + 1 < nb;              // a second row beyond the mini-batch is never published and not waited for
    float m[2] = {-FLT_MAX, -FLT_MAX}, sum[2] = {0.f, 0.f};
    for (int q0 = ps.pj; q0 < G && !gave_up; q0 += POLLS * ps.J) {
        const unsigned long long* src[POLLS];
        u32x4 word[POLLS];
#pragma unroll
        for (int q = 0; q < POLLS; ++q) src[q] = in + (size_t)min(q0 + q * ps.J, G - 1) * word_stride + ps.pr;
        guard.arm();
        while (true) {
            load_pairs(src, word);
            bool ok = true;
#pragma unroll
            for (int q = 0; q < POLLS; ++q) ok = ok && word[q].x >> kSumBits == tag && (word[q].z >> kSumBits == tag || !second);
            if (ok) break;
            if (guard.expired()) { gave_up = true; break; }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float k[POLLS], top = m[i];
#pragma unroll
            for (int q = 0; q < POLLS; ++q) {
                k[q] = q0 + q * ps.J < G ? as_float(i ? word[q].w : word[q].y) : -INFINITY;
                top = fmaxf(top, k[q]);
            }
            sum[i] = scale_down(sum[i], m[i] - top);
#pragma unroll
            for (int q = 0; q < POLLS; ++q) sum[i] += scale_down(sum_of(i ? word[q].z : word[q].x), k[q] - top);
            m[i] = top;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        rk[ps.pj * ps.R + ps.pr + i] = m[i];
        rf[ps.pj * ps.R + ps.pr + i] = sum[i];
    }
    return !gave_up;
}

// what e^(u - maximum) of row r is to be multiplied with: 2^k rest over the row's sum over all workgroups
__device__ __forceinline__ float row_scale(const float* rk, const float* rf, const PollShape& ps, int r, int l16, float k, float rest)
{
    float top, sum;
    if (ps.J == 1) {
        top = rk[r];
        sum = rf[r];
    } else {
        // the four lanes that keep the same row take every fourth share, then meet
        const int j0 = min(l16 >> 2, ps.J - 1) * ps.R + r, j1 = min((l16 >> 2) + 4, ps.J - 1) * ps.R + r;
        const float v0 = rk[j0], v1 = rk[j1];        // (one taken twice is the last one)
        top = fmaxf(v0, v1);
        top = fmaxf(top, dpp_mov<0x124>(top));
        top = fmaxf(top, dpp_mov<0x128>(top));
        sum = ((l16 >> 2) < ps.J ? scale_down(rf[j0], v0 - top) : 0.f) + ((l16 >> 2) + 4 < ps.J ? scale_down(rf[j1], v1 - top) : 0.f);
        sum += dpp_mov<0x124>(sum);
        sum += dpp_mov<0x128>(sum);
    }
    return scale_down(rest * kSumScale, k - top) / sum;
}

// residual of a tile's rows r0 .. r0 + 3 per lane (scale and label as row_sums keeps its results), transposed into shared memory
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
__device__ __attribute__((noinline)) void pass_alone(const SoftmaxChainArgs* args, int G, unsigned short* Wt, unsigned short* Rt, float* rk, float* rf, int* gave_up)
{
    const SoftmaxChainArgs a = *args;
    const int KS = a.p32 / 32, NS = a.n32 / 32, ws = a.p32 + 8, rs = a.n32 + 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const size_t batch = (size_t)a.n32 * a.p32, words_set = (size_t)G * a.word_stride;
    const PollShape ps(a.n32, G, tid);
    PollGuard guard{a.sync + 1, a.timeout_ticks, 0, 0};
    if (tid == 0) *gave_up = 0;
    __syncthreads();
    for (int s = 0; s < a.M; ++s) {
        const int nb = min(a.n, a.rows - s * a.n);
        const unsigned tag = row_tag(s);
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
                float k, rest, total;
                logits(rt, g * kClasses, u);
                row_sums(u, l16, k, rest, total);
                publish_rows(words + (size_t)g * a.word_stride, 16 * rt + 4 * lq, nb, l16, k, total * rest, tag);
            }
            __syncthreads();
        }
        if (!collect_rows<4>(words, a.word_stride, G, nb, tag, ps, guard, rk, rf)) *gave_up = 1;
        __syncthreads();
        if (*gave_up) return;
        const float inv_nb = 1.f / (float)nb, scale = alpha * inv_nb;
        float oc1 = 1.f, oc2 = 1.f;
        if (OPT && a.opt.kind == kOptAdam) opt_corrections(a.opt, a.opt.k_base + s + 1, oc1, oc2);
        for (int g = 0; g < G; ++g) {
            const int c0 = g * kClasses;
            load_w(c0);
            for (int rt = wave; rt < a.n32 / 16; rt += kWaves) {
                f32x4 u[NJ];
                float k, rest, total;
                logits(rt, c0, u);
                row_sums(u, l16, k, rest, total);
                const int r0 = 16 * rt + 4 * lq;
                const int label = a.YL[(size_t)s * a.n32 + r0 + (l16 & 3)];
                residual_tile(u, row_scale(rk, rf, ps, min(r0 + (l16 & 3), nb - 1), l16, k, rest), label, r0, c0, nb, a.C, l16, Rt, rs);
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
    float* rk = reinterpret_cast<float*>(Rt + kClasses * rs);  // [J][R] a row's sum over a share of the workgroups: k
    float* rf = rk + kMaxRows;                                 // [J][R] ... and f
    __shared__ int s_abort, s_role;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int G = gridDim.x, g = blockIdx.x;
    const int c0 = g * kClasses;
    const int n_rt = a.n32 / 16, n_ft = a.p32 / 16;
    const size_t batch = (size_t)a.n32 * a.p32;      // elements of a mini-batch in XP and XTP

    const SoftmaxChainArgs* args = (const SoftmaxChainArgs*)__builtin_amdgcn_kernarg_segment_ptr();   // (a itself, without a copy on the stack)
    unsigned ticket = 0;
    if (G > 1 && a.meeting_ticks == 0) {
        if (g == 0) pass_alone<OPT>(args, G, Wt, Rt, rk, rf, &s_abort);
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

    const PollShape ps(a.n32, G, tid);
    const size_t words_set = (size_t)G * a.word_stride;
    PollGuard guard{a.sync + 1, a.timeout_ticks, 0, 0};
    if (G > 1 && tid == 0) s_role = wait_for_meeting(a.meeting, ticket, (unsigned)G, a.meeting_ticks, guard);
    __syncthreads();
    if (G > 1 && s_role != kTogether) {
        if (s_role == kAlone) pass_alone<OPT>(args, G, Wt, Rt, rk, rf, &s_abort);
        return;
    }

    for (int s = 0; s < a.M; ++s) {
        const int nb = min(a.n, a.rows - s * a.n);
        const unsigned tag = row_tag(s);
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

        // k and rest of the rows' sums over this workgroup's classes; where it is alone, rest is the scale
        float k[RT], rest[RT];
        unsigned long long* words = a.words + (size_t)(s & 1) * words_set;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (t >= my_rt) break;
            float total;
            row_sums(u[t], l16, k[t], rest[t], total);
            if (G > 1) publish_rows(words + (size_t)g * a.word_stride, 16 * (wave + kWaves * t) + 4 * lq, nb, l16, k[t], total * rest[t], tag);
            else rest[t] = 1.f / total;
            __builtin_amdgcn_sched_barrier(0);           // (one tile's exponentials at a time: all of them together take too many registers)
        }
        if (G > 1) {
            __builtin_amdgcn_s_sleep(8);                 // (0.2 us: a poll sent at once comes back a moment before the words do)
            // (as many words a trip as a thread has: asking for four where there is one cost 0.6 us per update at G = 7)
            const bool got = G <= ps.J       ? collect_rows<1>(words, a.word_stride, G, nb, tag, ps, guard, rk, rf)
                             : G <= 2 * ps.J ? collect_rows<2>(words, a.word_stride, G, nb, tag, ps, guard, rk, rf)
                                             : collect_rows<4>(words, a.word_stride, G, nb, tag, ps, guard, rk, rf);
            if (!got) s_abort = 1;
            __syncthreads();
            if (s_abort) return;                    // (every thread sees the same value: it is not written after this barrier)
        }
        // residual, transposed into shared memory
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (t >= my_rt) break;
            const int r0 = 16 * (wave + kWaves * t) + 4 * lq;
            const float scale = G > 1 ? row_scale(rk, rf, ps, min(r0 + (l16 & 3), nb - 1), l16, k[t], rest[t]) : rest[t];
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

// Where one kernel is the faster way (us per update, this kernel / three launches; n, p, C).  What is left out here goes to the kernel of
// larger mini-batches, at 0.5 to 0.86 of the launches' time; the lines have not been drawn against it.  Small mini-batches gain most: 3.4 / 14.9
// at 100, 200, 10; 7.6 / 19.8 at 100, 200, 2000; 12.0 / 21.3 at 256, 512, 1000.  What a workgroup reads per update, 4 n p bytes, catches up
// around n p = 2^18: 13.6 / 20.6 at 512, 512, 10 and 26.3 / 31.1 with 2,000 classes, 20.3 / 23.7 at 256, 1000, 1000.
//   256 < n <= 512, p > 768 (eight feature tiles beside four row tiles: registers run out): 16.8 / 21.2 at 340, 760, 10, but 20.2 / 19.6
//     at 270, 968, 10 and 21.9 / 21.2 at 300, 872, 100.
//   n > 512: one group of threads collects the sums of all workgroups, four a trip of 0.7 us, so classes cost more, and less is left for them
//     the larger n p is.  As many classes as break even: 1140-1500 for n p up to 2^17 (950 at 600, 200), 710 at 1000, 192, 620 at 700, 280,
//     300 at 1000, 256, 250 at 800, 320; none at 560, 464, where with one workgroup and no exchange it is 20.9 / 24.1 (600, 432, 10).
//   State (momentum, NAG, Adam): registers run out earlier: 21.9 / 32.7 at 256, 512, 2000, 23.6 / 31.3 with Adam and 1,000 classes; n > 512 breaks even
//     at 1,000 to 1,600 classes (31.2 / 31.0 at 640, 200, 1000; 42.0 / 40.0 at 600, 216, 2000).
bool softmax_chain_eligible(int64_t p, int64_t n, int64_t C, bool opt)
{
    if (p > kMaxRows || n > kMaxRows || C > 2048) return false;
    if (opt) return p <= kMaxRows / 2 && p * n <= (int64_t(1) << 17) && (n <= kMaxRows / 2 || C <= 1000);
    if (p * n > (int64_t(1) << 18)) return false;
    if (n <= kMaxRows / 4) return true;
    if (n <= kMaxRows / 2) return p <= 768;
    if (p > 384) return p <= kMaxRows / 2 && C <= kClasses;
    return C <= std::min<int64_t>(1000, 1750 - 1500 * n * p / (int64_t(1) << 18));
}

size_t softmax_chain_pack_bytes(int64_t p, int64_t n, int64_t batches)
{
    return (size_t)batches * ((size_t)round32(n) * round32(p) * 4 + (size_t)round32(n) * 4);
}

size_t softmax_chain_words_bytes(int64_t n, int64_t C)
{
    return (size_t)2 * ((C + kClasses - 1) / kClasses) * round32(n) * 8;
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
    a.word_stride = a.n32;
    if (a.n32 > kMaxRows || a.p32 > kMaxRows || a.C > a.ldw) return hipErrorInvalidValue;
    const size_t half = (size_t)a.M * a.n32 * a.p32;
    unsigned short* xp = static_cast<unsigned short*>(pack);
    unsigned short* xtp = xp + half;
    int* yl = reinterpret_cast<int*>(xtp + half);
    a.XP = xp; a.XTP = xtp; a.YL = yl;
    const int jtiles = (a.n32 + 63) / 64;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)(a.M * jtiles), (unsigned)((a.p32 + 63) / 64)), dim3(256), 0, stream,
                       static_cast<const unsigned short*>(X), y, perm, xp, xtp, yl, a.rows, a.p, a.n, a.n32, a.p32, jtiles, a.meeting, a.words,
                       2 * ((a.C + kClasses - 1) / kClasses) * a.word_stride);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int G = (a.C + kClasses - 1) / kClasses;
    const ChainKernel k = chain_kernel(a.opt.kind != kOptSgd, tile_variant(a.n32), tile_variant(a.p32));
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((unsigned)G), dim3(kThreads), chain_lds(a.n32, a.p32), stream, a);
    return hipGetLastError();
}

}  // namespace bmgd
