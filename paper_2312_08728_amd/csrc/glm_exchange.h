// The exchange wavefronts of the persistent GLM kernels, and what they share around them.
//
// A workgroup of these kernels is a set of "row" wavefronts, which read rows and accumulate the gradient sums of a
// step of eq. (2.1), and three or four exchange wavefronts, which carry those sums to the other workgroups and bring the
// new theta back.  The two kinds meet only through flags in shared memory:
//   s_published      counts publications of row wavefronts over all steps (each stores its sums to shared memory first);
//   s_theta_version  versions of theta the exchange wavefronts have delivered to shared memory (version v = theta
//                    after v steps of the launch, kept in the copy v & 1), each of them counted;
//   s_abort          set by an exchange wavefront when a wait ran out: everybody leaves.
// A row wavefront must not poll global memory itself: loads return to a wavefront in the order it issued them, so
// its poll would come back behind the newest rows it has in flight.
//
// Three forms.  exchange_wavefront: two trips over the fabric per step, asking for everything a trip needs at once:
//   0. the workgroup's sums leave as flagged words {value : tag};
//   1. workgroup g adds up, for the g-th slice of the columns (whole 128-byte lines of words), the words of all G
//      workgroups in a fixed order, applies the update to its slice of theta and publishes the new values in
//      kThetaCopies copies of theta (a workgroup later reads copy g mod kThetaCopies, so no set of words is polled
//      by the whole grid);
//   2. it collects the whole new theta from its copy into shared memory and raises the version.
// exchange_by_die: the same with the sums added up on each die first, three shorter trips.
// exchange_one_trip: every workgroup adds up all words itself and makes the whole update.
// Polls are bounded by the wall clock.
//
// What bounds a step of short rows is latency: each trip is the time until the slowest workgroup has stored its words, the way there and back, and the
// instructions between them, 1.0 us and more over the fabric, 0.4 to 0.6 within a die; and all that a compute unit asks for passes through one memory
// pipeline in turn, so rows are requested when the exchange has nothing to send or to ask for (s_sent).
#pragma once

#include "bmgd_internal.h"
#include "glm_device.h"

#include <type_traits>

namespace bmgd {
namespace {

constexpr int kRowWaves = 8;                          // (glm_split_kernel.hip)

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// (pointers into shared memory carry its address space, so that accesses through them are shared-memory
// instructions and are counted apart from the row loads)
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) unsigned lds_u32;
typedef __attribute__((address_space(3))) int lds_i32;

constexpr int kAgentScope = 0x10;                    // cache policy of a buffer instruction: sc1

__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const void* base, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// (A function, so that its argument is a scalar copy: bit-casting an element of a vector in place reads element 0.)
__device__ __forceinline__ float as_float(unsigned v) { return __builtin_bit_cast(float, v); }

// two flagged words next to each other: {value, tag, value, tag}
__device__ __forceinline__ u32x4 word_pair(float v0, float v1, unsigned tag)
{
    u32x4 w;
    w.x = __builtin_bit_cast(unsigned, v0); w.y = tag;
    w.z = __builtin_bit_cast(unsigned, v1); w.w = tag;
    return w;
}

// A wait of a row wavefront, written as one block of assembly.  The compiler must see no loop and no branch out of
// the row loop at such a place: it keeps count of the row loads in flight per path through the control-flow graph,
// and every extra path (a poll loop, an early exit, which the structuriser routes through the loop's latch) makes
// it wait for rows that the path actually taken does not need.
// Wait until the word at shared-memory address `addr` is >= want, or the word at `abort_addr` is non-zero.  (Both are read in one trip, and
// nothing sleeps: with two trips and a sleep in between 0.03 to 0.1 us more per update.)
__device__ __forceinline__ void lds_wait_ge(unsigned addr, unsigned want, unsigned abort_addr)
{
    unsigned t, stop;
    asm volatile("1:\n\t"
                 "ds_read_b32 %0, %2\n\t"
                 "ds_read_b32 %1, %4\n\t"
                 "s_waitcnt lgkmcnt(0)\n\t"
                 "v_cmp_ge_u32_e32 vcc, %0, %3\n\t"
                 "s_cbranch_vccnz 2f\n\t"
                 "v_cmp_ne_u32_e32 vcc, 0, %1\n\t"
                 "s_cbranch_vccz 1b\n"
                 "2:"
                 : "=&v"(t), "=&v"(stop) : "v"(addr), "v"(want), "v"(abort_addr) : "vcc", "memory");
}

// The same for an exchange wavefront, which must not go on with the step if a wait ran out anywhere in the workgroup: until every
// lane's word (one address per lane) is >= want, or the word at `abort_addr` is non-zero; that word is returned.  It looks at both in
// one trip to shared memory.  No limit of its own is needed: the row wavefronts wait on shared memory only, and of the exchange
// wavefronts each either goes on or ends its poll with the abort word set.
template <bool SLEEP>
__device__ __forceinline__ unsigned lds_wait_all_ge(unsigned addr, unsigned want, unsigned abort_addr)
{
    unsigned t, stop;
    if constexpr (SLEEP)                             // a wait as long as a step's rows
        asm volatile("s_branch 3f\n"
                     "1:\n\t"
                     "s_sleep 1\n"
                     "3:\n\t"
                     "ds_read_b32 %0, %2\n\t"
                     "ds_read_b32 %1, %4\n\t"
                     "s_waitcnt lgkmcnt(0)\n\t"
                     "v_cmp_lt_u32_e32 vcc, %0, %3\n\t"
                     "s_cbranch_vccz 2f\n\t"
                     "v_cmp_ne_u32_e32 vcc, 0, %1\n\t"
                     "s_cbranch_vccz 1b\n"
                     "2:"
                     : "=&v"(t), "=&v"(stop) : "v"(addr), "v"(want), "v"(abort_addr) : "vcc", "memory");
    else
        asm volatile("1:\n\t"
                     "ds_read_b32 %0, %2\n\t"
                     "ds_read_b32 %1, %4\n\t"
                     "s_waitcnt lgkmcnt(0)\n\t"
                     "v_cmp_lt_u32_e32 vcc, %0, %3\n\t"
                     "s_cbranch_vccz 2f\n\t"
                     "v_cmp_ne_u32_e32 vcc, 0, %1\n\t"
                     "s_cbranch_vccz 1b\n"
                     "2:"
                     : "=&v"(t), "=&v"(stop) : "v"(addr), "v"(want), "v"(abort_addr) : "vcc", "memory");
    return (unsigned)__builtin_amdgcn_readfirstlane((int)stop);
}

// One is added to the word at shared-memory address `addr`, behind everything this wavefront has asked of shared memory.  For one lane.
// (An atomic add of the language counts the active lanes first.)
__device__ __forceinline__ void lds_add_one(unsigned addr)
{
    asm volatile("ds_add_u32 %0, %1" :: "v"(addr), "v"(1u) : "memory");
}

template <class T>
__device__ __forceinline__ unsigned lds_address(const T* word) { return (unsigned)(uintptr_t)word; }

// Mini-batches of the steps of a launch: step s is mini-batch m = s mod M of pass t = s / M.
struct StepGeometry {
    int M, n, n_tail, perm_stride;
    float rcpM;
    __device__ __forceinline__ explicit StepGeometry(const ExchangeArgs& a)
    {
        M = (a.rows + a.n - 1) / a.n;
        n = a.n;
        n_tail = a.rows - (M - 1) * a.n;
        perm_stride = a.perm_stride;
        rcpM = 1.0f / (float)M;
    }
    // s = t M + m, from a float reciprocal plus a correction: exact for s < 2^23, which the host guarantees
    __device__ __forceinline__ void split(int s, int& t, int& m) const
    {
        t = (int)((float)s * rcpM);
        m = s - t * M;
        if (m >= M) { m -= M; ++t; }
        if (m < 0) { m += M; --t; }
    }
    __device__ __forceinline__ int batch_rows(int s) const { int t, m; split(s, t, m); return m == M - 1 ? n_tail : n; }
    // where the mini-batch of step s starts in the array of partitions
    __device__ __forceinline__ size_t batch_base(int s) const
    {
        int t, m;
        split(s, t, m);
        return (size_t)t * (size_t)perm_stride + (size_t)m * (size_t)n;
    }
};

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f32x2 lds_f32x2;

// A row is taken as whole vectors of four floats whatever its length: its last vector starts four columns before its end, so that it may repeat
// up to three columns of the one before.  Theta, sums, words and the state of an update rule are laid out the same way, by position: width of
// them (an even number), the first `shift` of the last four standing for no column.  These hold 0 in theta; what is added up there is
// not looked at.  (Rows of fewer than eight floats that are no multiple of four keep to smaller vectors, and have no such positions.)
// The hardware loads vectors from any multiple of four bytes; rows loaded float by float or in pairs took 5.5 instead of 3.3 us per update at
// p = 301, n = 1000, 9.5 instead of 5.6 at 1502, 1000, 3.5 instead of 2.9 at 201, 1500: these then did not fit the registers, or took as many
// times the loads.
__device__ __forceinline__ int position_of(const ExchangeArgs& a, int c) { return c + (c >= a.width - 4 ? a.shift : 0); }
// the column of a position (below `width`), or one below 0 where there is none
__device__ __forceinline__ int column_of(const ExchangeArgs& a, int pos)
{
    const int k = pos - (a.width - 4);
    return k < 0 ? pos : k < a.shift ? -1 : pos - a.shift;
}
// where the vector of a row that starts at a position is loaded from; beyond the row (theta is 0 there) its start
__device__ __forceinline__ int vector_from(const ExchangeArgs& a, int pos) { return pos >= a.width ? 0 : pos - (pos >= a.width - 4 ? a.shift : 0); }

// Theta into the first `stride` floats of `th`, by position (0 where there is no column), and zeros into the others up to `total`.  (Multiples of
// 16; MAX: the largest stride.)  All that a thread loads is asked for at once and comes while the zeros go out: with a load and its position to
// work out in each turn of one loop over everything, a launch of one update took 10.1 us instead of 9.1 at p = 1000, n = 200, 19.0 instead of 17.0 at
// 4096, 200.
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
template <int BLOCK, int MAX>
__device__ __forceinline__ void load_theta(const ExchangeArgs& a, lds_f32* th, int stride, int total, int tid)
{
    constexpr int K = (MAX + BLOCK - 1) / BLOCK;
    float v[K];
    int col[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int c = tid + BLOCK * k;
        col[k] = c < a.width ? column_of(a, c) : -1;
        v[k] = a.theta[max(0, min(col[k], a.p - 1))];
    }
    for (int c = stride + 4 * tid; c < total; c += 4 * BLOCK) *(lds_u32x4*)(th + c) = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int c = tid + BLOCK * k;
        if (c < stride) th[c] = col[k] >= 0 && col[k] < a.p ? v[k] : 0.f;
    }
}

// The sum over the lanes with the same lane % PPc (8 <= PPc <= 64, uniform), in all of them.
__device__ __forceinline__ f32x2 pair_slot_sum(f32x2 v, int PPc)
{
    if (PPc == 8) {                                  // the usual case as one straight line
        v.x += dpp_mov<0x128>(v.x); v.y += dpp_mov<0x128>(v.y);
        v.x = swap16_sum(v.x); v.y = swap16_sum(v.y);
        v.x = swap32_sum(v.x); v.y = swap32_sum(v.y);
    } else if (PPc < 64) {
        if (PPc == 16) { v.x = swap16_sum(v.x); v.y = swap16_sum(v.y); }
        v.x = swap32_sum(v.x); v.y = swap32_sum(v.y);
    }
    return v;
}
// The same for PW (2 .. 64) known when compiled.
template <int PW>
__device__ __forceinline__ f32x2 lane_groups_sum(f32x2 v)
{
    if constexpr (PW == 2) { v.x += dpp_mov<0x122>(v.x); v.y += dpp_mov<0x122>(v.y); }
    if constexpr (PW <= 4) { v.x += dpp_mov<0x124>(v.x); v.y += dpp_mov<0x124>(v.y); }
    return pair_slot_sum(v, PW <= 8 ? 8 : PW);
}

// The exchange wavefronts' view of the workgroup's shared memory.
struct ExchangeLds {
    lds_f32* th;                  // [2][th_stride]: theta by version parity (th_stride even, >= the positions of a row)
    int th_stride;
    lds_f32* state;               // [NX][3][64][2]: for each exchange wavefront Adam's bias corrections of the coming steps, and the state
                                  //   of the pairs of columns it updates
    lds_f32* red;                 // [2][NX][64][2]: the exchange wavefronts' partial sums, by parity
    const lds_f32* sums;          // [NSUM][sums_stride]: the workgroup's gradient sums of a step; column c is the sum over
    int sums_stride;              //   the NSUM arrays (even)
    unsigned publishers;          // publications of row wavefronts that complete a step
    lds_u32* s_published;
    lds_u32* s_theta_version;     // raised by every exchange wavefront once per step: NX v when version v is complete
    lds_i32* s_abort;
    lds_u32* s_sent;              // raised by every exchange wavefront once per step, where rows wait for it: those of a later step may be requested
    lds_u32* s_xarrived;          // [NX] sets of partial sums each exchange wavefront has left in `red`
    lds_u32* s_xconsumed;         //         sets that the first one has added up (two-trip form)
};
constexpr int kExchangeState = 3 * 128, kExchangeRed = 2 * 128;     // floats of `state` and `red` per exchange wavefront

// What the exchange wavefronts of all forms do the same way.  NSUM: arrays of sums in shared memory.
//
// All of this stands on the critical path of a step, between the last row and the first of the next step, where one wavefront
// on its SIMD issues an instruction in four clocks at best and a branch taken costs more: 100 instructions are 0.2 us.  So it is written
// for few instructions: loops have one exit at the bottom and constant bounds (all reads of shared memory in one go; as run-time
// loops each turn waited for its own read, 8 x 130 clocks), a wait that ran out is a flag that is looked at once per step, lanes
// are summed with DPP, and shared memory's order (a wavefront's requests are served in the order they were made) stands where fences
// would wait for stores to global memory as well.
template <bool OPT, int NX, int NSUM>
struct ExchangeCommon {
    const ExchangeArgs& a;
    const ExchangeLds& x;
    const int lane, xw;
    const int G, g;
    const int p;                                     // positions of a row, for columns (as everywhere in the exchange)
    const int pp;
    const StepGeometry geo;
    const unsigned words_bytes;
    const unsigned abort_addr;
    long long poll_start = 0;                        // when the words of a trip were first asked for

    __device__ __forceinline__ ExchangeCommon(const ExchangeArgs& a_, const ExchangeLds& x_, int lane_, int xw_)
        : a(a_), x(x_), lane(lane_), xw(xw_), G(gridDim.x), g(blockIdx.x), p(a_.width), pp((a_.p + 15) & ~15), geo(a_),
          words_bytes((unsigned)((size_t)gridDim.x * (size_t)((a_.p + 15) & ~15) * 8)), abort_addr(lds_address(x_.s_abort))
    {
    }

    // until the word of every lane is >= want; non-zero: a wait ran out
    template <bool SLEEP>
    __device__ __forceinline__ unsigned wait_ge(const lds_u32* word, unsigned want) const
    {
        return lds_wait_all_ge<SLEEP>(lds_address(word), want, abort_addr);
    }

    // After a failed poll whose requests were sent at time `sent`: go on polling?  (The abort flag in global memory is looked at now and
    // then: a load from it costs a trip over the fabric, as much as the poll itself.)
    __device__ __forceinline__ bool go_on(unsigned& misses, long long sent)
    {
        if (misses == 0u) poll_start = sent;
        ++misses;
        if (sent - poll_start > a.timeout_ticks) return false;
        return (misses & 31u) != 0u || __hip_atomic_load(a.sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    }

    // U pairs of words per lane (`ask(u)` loads the u-th), asked for all together until all that the lane needs carry the tag
    // (`tags(w, u)`: the smaller of the u-th pair's tags, or `tag` where the lane does not need it).  Non-zero: the wait ran out.  (No tag
    // beyond the one waited for can be there yet, so all are equal to it if the smallest is.)  Measured against it and not kept: two or
    // three sets of requests under way one behind the other (0.4 us more per update at p = 200, n = 4096: the polls slow the stores they wait
    // for), and asking again only for what has not come (0.4 us more: a branch around each request).
    template <int U, class Ask, class Tags>
    __device__ __forceinline__ unsigned poll(unsigned tag, u32x4 (&w)[U], Ask&& ask, Tags&& tags)
    {
        unsigned misses = 0u;
        bool miss;
        long long sent;
        do {
            sent = wall_clock64();   // (looked at only if the poll fails, when it has long come)
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = ask(u);
            asm volatile("" ::: "memory");
            unsigned least = tag;
#pragma unroll
            for (int u = 0; u < U; ++u) least = min(least, tags(w[u], u));
            miss = __builtin_amdgcn_ballot_w64(least != tag) != 0ull;
        } while (miss && go_on(misses, sent));
        return miss ? 1u : 0u;
    }

    // a wait of this wavefront ran out: the others of the workgroup and the other workgroups are told
    __device__ __forceinline__ void give_up() const
    {
        if (lane == 0) {
            __hip_atomic_store(a.sync + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(x.s_abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }

    // the workgroup's sums of columns c and c + 1, added up as a fixed tree
    __device__ __forceinline__ f32x2 sum_of(int c) const
    {
        f32x2 v[NSUM];
#pragma unroll
        for (int k = 0; k < NSUM; ++k) v[k] = *(const lds_f32x2*)(x.sums + k * x.sums_stride + c);
#pragma unroll
        for (int w = 1; w < NSUM; w *= 2) {
#pragma unroll
            for (int k = 0; k + w < NSUM; k += 2 * w) { v[k].x += v[k + w].x; v[k].y += v[k + w].y; }
        }
        return v[0];
    }

    // The same of the pairs of columns PW xw + (0 .. PW - 1) where PW < 64: 64 / PW groups of lanes share the arrays, and their sums meet over
    // the lanes.  c: the first column of this lane's pair, or where there is none any other's.
    template <int PW>
    __device__ __forceinline__ f32x2 shared_sum_of(int c) const
    {
        constexpr int SG = 64 / PW, J = (NSUM + SG - 1) / SG;
        const int sg = lane / PW;
        f32x2 v[J];
#pragma unroll
        for (int j = 0; j < J; ++j) v[j] = *(const lds_f32x2*)(x.sums + min(sg + SG * j, NSUM - 1) * x.sums_stride + c);
        if constexpr (NSUM % SG != 0) {
            if (sg + SG * (J - 1) >= NSUM) v[J - 1] = f32x2{0.f, 0.f};
        }
#pragma unroll
        for (int w = 1; w < J; w *= 2) {
#pragma unroll
            for (int k = 0; k + w < J; k += 2 * w) { v[k].x += v[k + w].x; v[k].y += v[k + w].y; }
        }
        return lane_groups_sum<PW>(v[0]);
    }

    // this wavefront's share of the workgroup's sums of the columns below `cover`, as flagged words: what the others wait for.  U: pairs a lane sends
    // of sums that are one array, all read at once; stores beyond `cover` go to an address that the buffer's range check drops.  (As a loop over the
    // columns that there are, unrolled in eights, the compiler waited for the stores of the odd turns before the others': 0.2 us per update at p = 4096.)
    template <int SCOPE, int U>
    __device__ __forceinline__ void send_sums(__amdgpu_buffer_rsrc_t part, unsigned tag, int cover) const
    {
        auto send = [&](int c, f32x2 v) {
            __builtin_amdgcn_raw_buffer_store_b128(word_pair(v.x, v.y, tag), part, (unsigned)(((size_t)g * pp + c) * 8), 0, SCOPE);
        };
        asm volatile("" ::: "memory");
        if constexpr (NSUM == 1) {
            f32x2 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *(const lds_f32x2*)(x.sums + min(2 * lane + 128 * (xw + NX * u), pp - 2));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = 2 * lane + 128 * (xw + NX * u);
                __builtin_amdgcn_raw_buffer_store_b128(word_pair(v[u].x, v[u].y, tag), part, c < cover ? (unsigned)(((size_t)g * pp + c) * 8) : 0x7ffffff0u, 0, SCOPE);
            }
        } else {
            auto share = [&](auto pw) {
                constexpr int PW = decltype(pw)::value;
                const int c = 2 * (PW * xw + (lane & (PW - 1)));
                const f32x2 v = shared_sum_of<PW>(min(c, pp - 2));
                if (c < cover && lane < PW) send(c, v);
            };
            if (cover <= 16 * NX) share(std::integral_constant<int, 8>{});
            else if (cover <= 32 * NX) share(std::integral_constant<int, 16>{});
            else if (cover <= 64 * NX) share(std::integral_constant<int, 32>{});
            else {
#pragma unroll 1
                for (int c0 = 128 * xw; c0 < cover; c0 += 128 * NX) {
                    const int c = c0 + 2 * lane;
                    if (c < cover) send(c, sum_of(c));
                }
            }
        }
    }

    // What an update rule with state needs waits in shared memory, where reading it costs the update next to nothing (two powers a
    // step and state in global memory stood on its critical path: logistic regression with Adam, p = 512, n = 1000: 5.3 us per
    // update): Adam's bias corrections, which depend on the update's number alone, of 64 steps at a time, formed by 64 lanes
    // at once; and the state of the pair of columns that this wavefront's lane (or slot) `k` updates.
    __device__ __forceinline__ void corrections(int done)
    {
        if constexpr (OPT) {
            if (a.opt.kind == kOptAdam && (done & 63) == 0) {
                float f1, f2;
                opt_corrections(a.opt, a.opt.k_base + done + lane + 1, f1, f2);
                ((lds_f32x2*)(x.state + xw * 384))[lane] = f32x2{f1, f2};
            }
        }
    }
    __device__ __forceinline__ void load_state(int k, const float* m, const float* s) const
    {
        lds_f32x2* keep = (lds_f32x2*)(x.state + xw * 384 + 128) + k;
        keep[0] = f32x2{m[0], m[1]};
        if (a.opt.kind == kOptAdam) keep[64] = f32x2{s[0], s[1]};
    }
    __device__ __forceinline__ void store_state(int k, float* m, float* s) const
    {
        const lds_f32x2* keep = (const lds_f32x2*)(x.state + xw * 384 + 128) + k;
        const f32x2 v = keep[0], w = keep[64];
        m[0] = v.x; m[1] = v.y;
        if (a.opt.kind == kOptAdam) { s[0] = w.x; s[1] = w.y; }
    }
    // The update of the pair of columns c, c + 1: new values from the old ones and the pair's sums.  k: where its state is kept (`writes`: by
    // this lane; lanes that hold the same pair make the same update).  HALVES: lanes 32 apart hold the same pair, so each of them works out
    // one column (Adam's square root and divisions: 0.15 us of a step for a pair).
    template <bool HALVES>
    __device__ __forceinline__ f32x2 update(f32x2 old, f32x2 sum, float nb, float scale, float alpha, int done, int k, bool writes, int c) const
    {
        f32x2 now;
        if constexpr (!OPT) {
            now = f32x2{old.x - scale * sum.x, old.y - scale * sum.y};
        } else {
            asm volatile("" ::: "memory");
            const f32x2 f = ((const lds_f32x2*)(x.state + xw * 384))[done & 63];   // (not looked at but by Adam)
            if constexpr (HALVES) {
                const bool second = lane >= 32;
                lds_f32* keep = x.state + xw * 384 + 128 + 2 * k + (second ? 1 : 0);
                float m = keep[0], s = keep[128];
                now.x = opt_update(a.opt, second ? old.y : old.x, (second ? sum.y : sum.x) / nb, alpha, m, s, f.x, f.y);
                if (writes) {
                    keep[0] = m;
                    if (a.opt.kind == kOptAdam) keep[128] = s;
                }
                now.y = now.x;
                asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(now.x), "+v"(now.y));
            } else {
                lds_f32x2* keep = (lds_f32x2*)(x.state + xw * 384 + 128) + k;
                const f32x2 m = keep[0], s = keep[64];
                float m0 = m.x, m1 = m.y, s0 = s.x, s1 = s.y;
                now.x = opt_update(a.opt, old.x, sum.x / nb, alpha, m0, s0, f.x, f.y);
                now.y = opt_update(a.opt, old.y, sum.y / nb, alpha, m1, s1, f.x, f.y);
                if (writes) {
                    keep[0] = f32x2{m0, m1};
                    if (a.opt.kind == kOptAdam) keep[64] = f32x2{s0, s1};
                }
            }
        }
        const int hole = c - (p - 4);
        return f32x2{(unsigned)hole < (unsigned)a.shift ? 0.f : now.x, (unsigned)(hole + 1) < (unsigned)a.shift ? 0.f : now.y};
    }

    // (everything this wavefront has stored to shared memory stays in front of the count)
    __device__ __forceinline__ void raise_version() const
    {
        asm volatile("" ::: "memory");
        if (lane == 0) lds_add_one(lds_address(x.s_theta_version));
    }
    __device__ __forceinline__ void mark_sent() const
    {
        asm volatile("" ::: "memory");
        if (lane == 0) lds_add_one(lds_address(x.s_sent));
    }
    __device__ __forceinline__ void mark_arrived(unsigned count) const
    {
        asm volatile("" ::: "memory");
        if (lane == 0) __hip_atomic_store(x.s_xarrived + xw, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    // the end of a launch: theta to global memory
    __device__ __forceinline__ void finish(int steps) const
    {
        if (g == 0 && xw == 0) {
            if (wait_ge<true>(x.s_theta_version, NX * (unsigned)steps)) return;
            asm volatile("" ::: "memory");
            const lds_f32* fin = x.th + ((unsigned)steps & 1u) * x.th_stride;
            for (int c = lane; c < a.p; c += 64) a.theta[c] = fin[position_of(a, c)];
        }
    }
};

// All steps [a.s_begin, a.s_end) of a launch in two trips over the fabric each, by exchange wavefront xw of NX of workgroup
// blockIdx.x of gridDim.x (a multiple of 8).  Returns when the last version of theta has been delivered (workgroup 0 also writes it
// to a.theta), or with s_abort and the global abort flag set when a wait ran out.
// The wavefronts share every phase: each sends a part of the workgroup's sums, adds up a part of the
// workgroups for the slice (the first one then adds the NX partial sums in their order and applies the update) and
// collects a part of theta.  A wavefront pulls freshly written lines at a fraction of what a compute unit can take, so several on as
// many SIMDs finish a trip sooner, beside row traffic too (glm_split_kernel.hip has both figures).
// GATED: the row wavefronts wait for s_sent.  U1, U2: pairs of words a lane requests per trip when it sums the slice / collects theta (sums that are one array: all of them).
template <bool OPT, int NX, int NSUM, bool GATED, int U1, int U2>
__device__ __forceinline__ void exchange_wavefront(const ExchangeArgs& a, const ExchangeLds& x, int lane, int xw)
{
    ExchangeCommon<OPT, NX, NSUM> ex(a, x, lane, xw);
    const int G = ex.G, g = ex.g, p = ex.p, pp = ex.pp;
    const int first = a.s_begin, last = a.s_end;
    const unsigned copies_bytes = (unsigned)((size_t)kThetaCopies * pp * 8);
    // Workgroup g owns the columns [c_lo, c_hi) of theta (whole 128-byte lines of words, so no line has two writers).
    const int cw = (((p + G - 1) / G) + 15) & ~15;
    const int c_lo = min(p, g * cw), c_hi = min(p, c_lo + cw);
    const int npair = cw / 2;                        // column pairs of a slice (a multiple of 8)
    int PPc = 8;                                     // pairs taken side by side by the lanes (a power of two) ...
    while (PPc < npair && PPc < 64) PPc *= 2;
    const int SG = 64 / PPc;                         // ... by SG groups of lanes, each group taking every SG-th workgroup
    const int my_pair = lane & (PPc - 1), my_sg = lane / PPc;
    // State of an update rule: a slice of one chunk keeps it in shared memory from step to step (a wider one, chunk by chunk, does not)
    const bool one_chunk = npair <= PPc;
    auto load_state = [&](int c) {                   // (the arrays reach to p rounded up to 16)
        if constexpr (OPT) {
            if (xw == 0 && my_sg == 0 && c < c_hi) ex.load_state(my_pair, a.opt.m + c, a.opt.s + c);
        }
    };
    auto store_state = [&](int c) {
        if constexpr (OPT) {
            asm volatile("" ::: "memory");
            if (xw == 0 && my_sg == 0 && c < c_hi) ex.store_state(my_pair, a.opt.m + c, a.opt.s + c);
        }
    };
    if (one_chunk) load_state(c_lo + 2 * my_pair);
    // Rows wait until the first trip's words have come in, where these are many (us per update at p = 2500, n = 1500: 9.10 not at all, 8.94 until this
    // workgroup's sums are out, 8.29 so; but 4.22, 4.18 and 4.35 on 64 workgroups at p = 1028, n = 200)
    const bool early = G * p <= (1 << 18);
    unsigned dead = 0u;
    unsigned phase = 0u;                             // chunks of slices summed so far (the same in all NX wavefronts)
    int s = first;
#pragma clang loop unroll(disable)
    do {
        const unsigned tag = a.tag_base + (unsigned)(s - first) + 1u;
        const float alpha_s = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        const float nb = (float)ex.geo.batch_rows(s);
        const float scale = alpha_s / nb;
        const unsigned ver = (unsigned)(s - first);
        const lds_f32* th_old = x.th + (ver & 1u) * x.th_stride;
        lds_f32* th_new = x.th + ((ver + 1u) & 1u) * x.th_stride;
        ex.corrections(s - first);
        const __amdgpu_buffer_rsrc_t part = words_rsrc(a.ll_part + (size_t)(s & 1) * G * pp, ex.words_bytes);
        const __amdgpu_buffer_rsrc_t thw = words_rsrc(a.ll_theta + (size_t)(s & 1) * kThetaCopies * pp, copies_bytes);
        // (the buffer of the copy this workgroup reads is that copy alone, so loads beyond its row of words are answered with
        // zeros by the range check without going to memory, and are not looked at)
        const __amdgpu_buffer_rsrc_t mine = words_rsrc(a.ll_theta + ((size_t)(s & 1) * kThetaCopies + (size_t)(g % kThetaCopies)) * pp, (unsigned)(pp * 8));
        // This workgroup's own rows first: until they have been summed nothing can be complete, and polling the
        // fabric meanwhile would only take bandwidth from the rows.  (The rows were multiplied by a complete theta, so
        // every exchange wavefront has delivered its part of the version that this step's update starts from.)
        dead |= ex.template wait_ge<false>(x.s_published, (ver + 1u) * x.publishers);
        // 0. this workgroup's sums out of shared memory
        ex.template send_sums<kAgentScope, U2>(part, tag, p);
        if (GATED && early) ex.mark_sent();

        // 1. this workgroup's slice, if it has one: sum over all workgroups, in a fixed order; the update; the new
        //    values into every copy of theta
        if (c_lo < c_hi) {
            int pb = 0;
#pragma clang loop unroll(disable)
            do {
                const int c = c_lo + 2 * (pb + my_pair);
                const bool own = c < c_hi;                       // (a slice ends on a multiple of 16 or at p)
                if (!one_chunk) {
                    load_state(c);
                    // two sets of partial sums alternate: a wavefront does not overwrite a set before the first one has added
                    // it up (a slice of one chunk cannot come to that: its theta has been collected since)
                    if (phase >= 2u) dead |= ex.template wait_ge<false>(x.s_xconsumed, phase - 1u);
                }
                // One address register per lane (its pair of columns in the row of words of workgroup my_sg); what differs
                // between a lane's loads is uniform and goes into the scalar offset.  Load u of wavefront xw takes the
                // workgroups SG (xw + NX u) + my_sg.  G is a multiple of SG, so whether a load is beyond the last
                // workgroup is uniform too (such loads repeat the last group and are not added).
                const unsigned voff = (unsigned)min(c, pp - 2) * 8u + (unsigned)my_sg * (unsigned)(pp * 8);
                f32x2 t = {0.f, 0.f};
                int i0 = SG * xw;
#pragma clang loop unroll(disable)
                do {
                    u32x4 w[U1];
                    dead |= ex.poll(tag, w,
                        [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(part, voff, (unsigned)min(i0 + SG * NX * u, G - SG) * (unsigned)(pp * 8), kAgentScope); },
                        [&](const u32x4& v, int) { return own ? min(v.y, v.w) : tag; });
#pragma unroll
                    for (int u = 0; u < U1; ++u) {
                        const bool there = i0 + SG * NX * u < G;
                        t.x += there ? as_float(w[u].x) : 0.f;
                        t.y += there ? as_float(w[u].z) : 0.f;
                    }
                    i0 += SG * NX * U1;
                } while (i0 - SG * xw < G && dead == 0u);
                t = pair_slot_sum(t, PPc);           // the SG groups' sums meet over the lanes: every lane has its pair's
                // the NX wavefronts' sums meet in the first one
                lds_f32x2* set = (lds_f32x2*)(x.red + (phase & 1u) * NX * 128);
                if (xw != 0) {
                    if (lane < PPc) set[xw * 64 + lane] = t;
                    ex.mark_arrived(phase + 1u);
                } else {
                    dead |= ex.template wait_ge<false>(x.s_xarrived + 1 + min(lane, NX - 2), phase + 1u);
                    asm volatile("" ::: "memory");
                    f32x2 v[NX - 1];
#pragma unroll
                    for (int k = 1; k < NX; ++k) v[k - 1] = set[k * 64 + my_pair];
#pragma unroll
                    for (int k = 1; k < NX; ++k) { t.x += v[k - 1].x; t.y += v[k - 1].y; }
                }
                if (own && xw == 0) {
                    const f32x2 old = *(const lds_f32x2*)(th_old + c);
                    const f32x2 now = ex.template update<false>(old, t, nb, scale, alpha_s, s - first, my_pair, my_sg == 0, c);
                    const u32x4 nw = word_pair(now.x, now.y, tag);
                    // the groups of lanes share the copies between them
                    const unsigned to = (unsigned)c * 8u + (unsigned)(my_sg * pp * 8);
                    static_assert(kThetaCopies == 8, "as many copies as groups of lanes at most");
                    __builtin_amdgcn_raw_buffer_store_b128(nw, thw, to, 0u, kAgentScope);
                    for (int r = SG; r < kThetaCopies; r += SG)
                        __builtin_amdgcn_raw_buffer_store_b128(nw, thw, to, (unsigned)(r * pp * 8), kAgentScope);
                }
                if (!one_chunk) {
                    store_state(c);
                    asm volatile("" ::: "memory");
                    if (xw == 0 && lane == 0) __hip_atomic_store(x.s_xconsumed, phase + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                ++phase;
                pb += PPc;
            } while (pb < npair && dead == 0u);
        }
        if (GATED && !early) ex.mark_sent();
        // 2. the whole new theta, from this workgroup's copy
        if (128 * xw < p && dead == 0u) {
            const unsigned copy_off = (unsigned)lane * 16u;
            auto collect = [&](auto count, int c0) {
                constexpr int U = decltype(count)::value;
                u32x4 w[U];
                dead |= ex.poll(tag, w,
                    [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(mine, copy_off, (unsigned)(c0 + 128 * NX * u) * 8u, kAgentScope); },
                    [&](const u32x4& v, int u) { return c0 + 2 * (lane + 64 * NX * u) < p ? min(v.y, v.w) : tag; });
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int c = c0 + 2 * (lane + 64 * NX * u);
                    if (c < p) *(lds_f32x2*)(th_new + c) = f32x2{as_float(w[u].x), as_float(w[u].z)};
                }
            };
            if (p <= 128 * NX) {
                collect(std::integral_constant<int, 1>{}, 128 * xw);
            } else {
                int c0 = 128 * xw;
#pragma clang loop unroll(disable)
                do {
                    collect(std::integral_constant<int, U2>{}, c0);
                    c0 += 128 * NX * U2;
                } while (c0 < p && dead == 0u);
            }
        }
        if (dead != 0u) ex.give_up();
        ex.raise_version();
        ++s;
    } while (s < last && dead == 0u);
    if (dead != 0u) return;
    if (one_chunk) store_state(c_lo + 2 * my_pair);
    ex.finish(last - first);
}

// Columns dealt out to the NX exchange wavefronts of a workgroup as pairs: wavefront xw holds the pairs PW xw + (0 .. PW - 1), PW a power of
// two, in SG = 64 / PW groups of lanes, which share what there is to add up for a pair; their sums meet over the lanes, and nothing is handed
// from wavefront to wavefront.  For the exchange in which every workgroup makes the whole update.
// us per update with chunks of 64 pairs, whose workgroups the wavefronts shared and whose partial sums met in shared memory (a hand-over, with
// twelve arrays of sums read by one wavefront, was 0.6 of the 2.9 us) / now: 3.40 / 2.89 at p = 123, n = 777 with momentum, 2.93 / 2.49 at
// p = 128, n = 1024, 2.88 / 2.22 at p = 30, n = 3000, 2.84 / 2.12 at p = 512, n = 90 on 8 workgroups; one workgroup 1.43 / 1.30 at p = 128, n = 96.
template <bool OPT, int NX, int NSUM, int PW>
struct PairExchange : ExchangeCommon<OPT, NX, NSUM> {
    static constexpr int SG = 64 / PW;
    const int pair, sg;                              // this lane's
    const int c;                                     // first column of its pair,
    const int cc;                                    //   or where there is none the last one
    const bool own;
    __device__ __forceinline__ PairExchange(const ExchangeArgs& a, const ExchangeLds& x, int lane, int xw)
        : ExchangeCommon<OPT, NX, NSUM>(a, x, lane, xw), pair(lane & (PW - 1)), sg(lane / PW), c(2 * (PW * xw + pair)), cc(min(c, this->pp - 2)), own(c < this->p)
    {
    }

    // the workgroup's sums of this lane's pair, in all groups of lanes
    __device__ __forceinline__ f32x2 own_sum() const
    {
        asm volatile("" ::: "memory");
        return this->template shared_sum_of<PW>(cc);
    }
    __device__ __forceinline__ void send(f32x2 v, __amdgpu_buffer_rsrc_t part, unsigned tag) const
    {
        if (own && sg == 0)
            __builtin_amdgcn_raw_buffer_store_b128(word_pair(v.x, v.y, tag), part, (unsigned)(((size_t)this->g * this->pp + c) * 8), 0, kAgentScope);
    }
    // the new values of this lane's pair to shared memory
    __device__ __forceinline__ void apply(const lds_f32* th_old, lds_f32* th_new, f32x2 sum, float nb, float scale, float alpha, int done)
    {
        const f32x2 old = *(const lds_f32x2*)(th_old + cc);
        const f32x2 now = this->template update<(PW <= 32)>(old, sum, nb, scale, alpha, done, pair, own && (this->lane & 31) < PW, c);
        if (own && sg == 0) *(lds_f32x2*)(th_new + c) = now;
    }
};

// The same steps in ONE trip over the fabric: every workgroup adds up all sums of all workgroups itself, in the same order, and keeps
// its own copy of theta and of an update rule's state (at m + g pp).  For few words (G p of them come in per step and workgroup).
template <bool OPT, int NX, int NSUM, bool GATED, int PW>
__device__ __forceinline__ void exchange_one_trip(const ExchangeArgs& a, const ExchangeLds& x, int lane, int xw)
{
    PairExchange<OPT, NX, NSUM, PW> ex(a, x, lane, xw);
    constexpr int SG = 64 / PW;
    const int G = ex.G, g = ex.g, pp = ex.pp;
    const int first = a.s_begin, last = a.s_end;
    const bool mine = ex.own && ex.sg < G;
    const unsigned voff = (unsigned)ex.cc * 8u + (unsigned)min(ex.sg, G - 1) * (unsigned)(pp * 8);
    const int loads = (G + SG - 1) / SG;             // pairs of words a lane asks for per step (as one, two, four, or eight at a time)
    if constexpr (OPT) {
        if (ex.own && ex.sg == 0) ex.load_state(ex.pair, a.opt.m + (size_t)g * pp + ex.c, a.opt.s + (size_t)g * pp + ex.c);   // (the arrays reach to p rounded up to 16, per workgroup)
    }
    unsigned dead = 0u;
    int s = first;
#pragma clang loop unroll(disable)
    do {
        const unsigned tag = a.tag_base + (unsigned)(s - first) + 1u;
        const float alpha_s = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        const float nb = (float)ex.geo.batch_rows(s);
        const float scale = alpha_s / nb;
        const unsigned ver = (unsigned)(s - first);
        const lds_f32* th_old = x.th + (ver & 1u) * x.th_stride;
        lds_f32* th_new = x.th + ((ver + 1u) & 1u) * x.th_stride;
        ex.corrections(s - first);
        const __amdgpu_buffer_rsrc_t part = words_rsrc(a.ll_part + (size_t)(s & 1) * G * pp, ex.words_bytes);
        dead |= ex.template wait_ge<false>(x.s_published, (ver + 1u) * x.publishers);
        f32x2 t = ex.own_sum();
        if (G > 1) {
            ex.send(t, part, tag);
            if constexpr (GATED) ex.mark_sent();
            // Words of many workgroups take a wavefront long to fetch: asked for at once they would be fetched twice, none of the others'
            // having come yet (0.27 us per update with 32 workgroups at p = 128, n = 1024; nothing with few)
            if (loads > 2) __builtin_amdgcn_s_sleep(15);
            // Load u of a lane takes the workgroup i + sg, i = i0 + SG u.  The last loads start at G - SG at most;
            // what they bring a second time (workgroups below i) is not added.
            f32x2 r = {0.f, 0.f};
            // A wavefront without columns asks for nothing where the words are many.  (Where they are few it is better kept busy: it would look at shared
            // memory all the time that the others' words take, 0.15 us more per update at p = 16 on 3 to 16 workgroups.)
            const bool columns = PW >= 8 || 2 * PW * xw < ex.p;
            auto trips = [&](auto count) {
                constexpr int U = decltype(count)::value;
                int i0 = 0;
#pragma clang loop unroll(disable)
                do {
                    u32x4 w[U];
                    dead |= ex.poll(tag, w,
                        [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(part, voff, (unsigned)max(0, min(i0 + SG * u, G - SG)) * (unsigned)(pp * 8), kAgentScope); },
                        [&](const u32x4& v, int) { return mine ? min(v.y, v.w) : tag; });
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = i0 + SG * u;
                        const bool add = mine && i < G && max(0, min(i, G - SG)) + ex.sg >= i;
                        r.x += add ? as_float(w[u].x) : 0.f;
                        r.y += add ? as_float(w[u].z) : 0.f;
                    }
                    i0 += SG * U;
                } while (i0 < G && dead == 0u);
            };
            if (!columns) {}
            else if (loads <= 1) trips(std::integral_constant<int, 1>{});
            else if (loads <= 2) trips(std::integral_constant<int, 2>{});
            else if (loads <= 4) trips(std::integral_constant<int, 4>{});
            else trips(std::integral_constant<int, 8>{});
            t = lane_groups_sum<PW>(r);
        }
        ex.apply(th_old, th_new, t, nb, scale, alpha_s, s - first);
        if (dead != 0u) ex.give_up();
        ex.raise_version();
        ++s;
    } while (s < last && dead == 0u);
    if (dead != 0u) return;
    if constexpr (OPT) {
        asm volatile("" ::: "memory");
        if (ex.own && ex.sg == 0) ex.store_state(ex.pair, a.opt.m + (size_t)g * pp + ex.c, a.opt.s + (size_t)g * pp + ex.c);
    }
    ex.finish(last - first);
}

// The same steps over two levels: the workgroups g with the same g mod 8 first add up their sums among themselves, line by line (16 columns);
// the eight sums of a line meet in the eight wavefronts that made them, each of which makes the line's update and hands the new values to
// its own workgroups.  The hardware deals the workgroups of a launch out to its eight dies in turn, so the first and the last of these
// three trips stay on a die, and their words in the die's L2: they are stored without a scope, which leaves them there, and read at device
// scope, which passes the unit's own cache by.  Whether the workgroups are where they should be is looked at in every launch (`near`).
//
// What it is for: a trip between workgroups of one die takes 0.4 to 0.6 us, one over the fabric 1.0 and more, and a slice of 16 columns is 256 words
// a column there, which four wavefronts fetch and hand over to one (0.7 us); here a wavefront asks for 4 of them a lane and then for one.  us per
// update, two trips / this: 3.48 / 2.86 at p = 200, n = 4096 (256 workgroups), 3.64 / 3.27 at p = 512, n = 1000 with Adam (160), 3.19 / 2.83 at 128, 900 (40),
// 3.91 / 3.61 at 1000, 500 (160), 5.06 / 4.70 at 1024, 2000 (256); rows of more than 1024 floats 5.54 / 5.01 at 1500, 1000, 5.57 / 4.67 at 2048, 300.
// The eight sums of a line go to every die separately: a line that all dies ask for took 1.45 us instead of 1.18, one that four wavefronts
// write a quarter of 2.6.  Every workgroup making the whole update from the dies' sums costs a trip less and more for its words: 3.5 us at p = 200.
// It is the faster way as long as a wavefront has one line (up to 1024 floats), two or three: each line more is two trips one behind the other (4.20
// against 3.32 at p = 200 on 24 workgroups, 16.3 against 3.7 at p = 1000 on 16; both lines in the same trips: 3.60 against 3.23 at p = 400 on 32,
// 4.26 against 3.76 at p = 1000 on 64), which the callers' rule sees to (glm_by_die).
// LW: lines a wavefront takes at a time.  U2: pairs of words a lane requests at a time when it collects theta (sums that are one array: all of them).
template <bool OPT, int NX, int NSUM, int LW, int U2>
__device__ __forceinline__ void exchange_by_die(const ExchangeArgs& a, const ExchangeLds& x, int lane, int xw)
{
    ExchangeCommon<OPT, NX, NSUM> ex(a, x, lane, xw);
    const int G = ex.G, g = ex.g, p = ex.p, pp = ex.pp;
    const int first = a.s_begin, last = a.s_end;
    const int die = g & 7, i_die = g >> 3, G_die = G >> 3;
    // line l: wavefront l / G_die of workgroup l mod G_die of each die; eight pairs by eight groups of lanes, each taking every eighth
    // workgroup in the first trip and one die's sum in the second
    const int lines = pp / 16;
    const int lpair = lane & 7, lsg = lane >> 3;
    const int l0 = i_die + G_die * xw, dl = G_die * NX;
    const unsigned lrow = (unsigned)(8 * min(lsg, G_die - 1) + die) * (unsigned)(pp * 8);
    const unsigned drow = (unsigned)(8 * die + lsg) * (unsigned)(pp * 8);
    const unsigned dies_bytes = (unsigned)(64u * (unsigned)pp * 8u);
    unsigned dead = 0u;
    // Which die is this workgroup on, and are the others of its first level there as well?  (In the row of words that the second step uses.)
    bool near;
    {
        const unsigned tag = a.tag_base + 1u;
        const unsigned xcc = (unsigned)__builtin_amdgcn_s_getreg(6164);          // XCC_ID, bits 0 .. 3
        unsigned long long* row0 = a.ll_part + (size_t)((first + 1) & 1) * G * pp;
        if (xw == 0 && lane == 0) ll_store(row0 + (size_t)g * pp, as_float(xcc), tag);
        // The state of all lines comes while the others' answers do (launches of one update with Adam: 9.5 us instead of 11.3 with the two one after the
        // other, at p = 1000, n = 2000; 14.7 and 16.3 at 2048, 2048).  What a wavefront reads here is written back behind sums that it has contributed to.
        if constexpr (OPT) {
            float m[LW][2], v[LW][2];
#pragma unroll
            for (int k = 0; k < LW; ++k) {
                const int c = 16 * min(l0 + dl * k, lines - 1) + 2 * lpair;
                m[k][0] = a.opt.m[c]; m[k][1] = a.opt.m[c + 1];
                if (a.opt.kind == kOptAdam) { v[k][0] = a.opt.s[c]; v[k][1] = a.opt.s[c + 1]; }
            }
#pragma unroll
            for (int k = 0; k < LW; ++k)
                if (lane < 8) ex.load_state(8 * k + lane, m[k], v[k]);
        }
        const __amdgpu_buffer_rsrc_t rows = words_rsrc(row0, ex.words_bytes);
        u32x4 w[1];
        const unsigned from = (unsigned)(8 * min(lane, G_die - 1) + die) * (unsigned)(pp * 8);
        dead |= ex.poll(tag, w, [&](int) { return __builtin_amdgcn_raw_buffer_load_b128(rows, from, 0u, kAgentScope); }, [&](const u32x4& v, int) { return v.y; });
        near = a.far == 0 && __builtin_amdgcn_ballot_w64(w[0].x != xcc) == 0ull;
    }
    int s = first;
#pragma clang loop unroll(disable)
    do {
        const unsigned tag = a.tag_base + (unsigned)(s - first) + 1u;
        const float alpha_s = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        const float nb = (float)ex.geo.batch_rows(s);
        const float scale = alpha_s / nb;
        const unsigned ver = (unsigned)(s - first);
        const lds_f32* th_old = x.th + (ver & 1u) * x.th_stride;
        lds_f32* th_new = x.th + ((ver + 1u) & 1u) * x.th_stride;
        ex.corrections(s - first);
        const __amdgpu_buffer_rsrc_t part = words_rsrc(a.ll_part + (size_t)(s & 1) * G * pp, ex.words_bytes);
        const __amdgpu_buffer_rsrc_t dies = words_rsrc(a.ll_dies + (size_t)(s & 1) * 64 * pp, dies_bytes);
        const __amdgpu_buffer_rsrc_t mine = words_rsrc(a.ll_theta + ((size_t)(s & 1) * kThetaCopies + (size_t)die) * pp, (unsigned)(pp * 8));
        dead |= ex.template wait_ge<false>(x.s_published, (ver + 1u) * x.publishers);
        if (near) ex.template send_sums<0, U2>(part, tag, pp);
        else ex.template send_sums<kAgentScope, U2>(part, tag, pp);
        if (l0 >= lines) ex.mark_sent();
        for (int l = l0, k0 = 0; l < lines && dead == 0u; l += LW * dl, k0 += 8 * LW) {
            f32x2 r[LW];
            {
                u32x4 w[4 * LW];
                dead |= ex.poll(tag, w,
                    [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(part, lrow + (unsigned)lpair * 16u, (unsigned)(8 * max(0, min(8 * (u & 3), G_die - 8))) * (unsigned)(pp * 8) + (unsigned)min(l + dl * (u >> 2), lines - 1) * 128u, kAgentScope); },
                    [&](const u32x4& v, int) { return min(v.y, v.w); });
#pragma unroll
                for (int j = 0; j < LW; ++j) {
                    r[j] = f32x2{0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool add = 8 * u < G_die && lsg < G_die && max(0, min(8 * u, G_die - 8)) + lsg >= 8 * u;
                        r[j].x += add ? as_float(w[4 * j + u].x) : 0.f;
                        r[j].y += add ? as_float(w[4 * j + u].z) : 0.f;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < LW; ++j) {
                r[j] = pair_slot_sum(r[j], 8);
                if (j == 0 || l + dl * j < lines)    // (to the eight dies)
                    __builtin_amdgcn_raw_buffer_store_b128(word_pair(r[j].x, r[j].y, tag), dies, (unsigned)((8 * lsg + die) * pp + 2 * lpair) * 8u, (unsigned)(l + dl * j) * 128u, kAgentScope);
            }
            if (l == l0) ex.mark_sent();
            {
                u32x4 w[LW];
                dead |= ex.poll(tag, w,
                    [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(dies, drow + (unsigned)lpair * 16u, (unsigned)min(l + dl * u, (l + dl * u < lines ? lines - 1 : l)) * 128u, kAgentScope); },
                    [&](const u32x4& v, int) { return min(v.y, v.w); });
#pragma unroll
                for (int j = 0; j < LW; ++j) r[j] = pair_slot_sum(f32x2{as_float(w[j].x), as_float(w[j].z)}, 8);
            }
#pragma unroll
            for (int j = 0; j < LW; ++j)
                if (j == 0 || l + dl * j < lines) {
                    const int c = 16 * (l + dl * j) + 2 * lpair;
                    const f32x2 old = *(const lds_f32x2*)(th_old + c);
                    const f32x2 now = ex.template update<true>(old, r[j], nb, scale, alpha_s, s - first, k0 + 8 * j + lpair, (lane & 31) < 8, c);
                    if (lane < 8) {
                        if (near) __builtin_amdgcn_raw_buffer_store_b128(word_pair(now.x, now.y, tag), mine, (unsigned)c * 8u, 0u, 0);
                        else __builtin_amdgcn_raw_buffer_store_b128(word_pair(now.x, now.y, tag), mine, (unsigned)c * 8u, 0u, kAgentScope);
                    }
                }
        }
        // the whole new theta, from this die's copy
        if (128 * xw < p && dead == 0u) {
            const unsigned copy_off = (unsigned)lane * 16u;
            auto collect = [&](auto count, int c0) {
                constexpr int U = decltype(count)::value;
                u32x4 w[U];
                dead |= ex.poll(tag, w,
                    [&](int u) { return __builtin_amdgcn_raw_buffer_load_b128(mine, copy_off, (unsigned)(c0 + 128 * NX * u) * 8u, kAgentScope); },
                    [&](const u32x4& v, int u) { return c0 + 2 * (lane + 64 * NX * u) < p ? min(v.y, v.w) : tag; });
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int c = c0 + 2 * (lane + 64 * NX * u);
                    if (c < p) *(lds_f32x2*)(th_new + c) = f32x2{as_float(w[u].x), as_float(w[u].z)};
                }
            };
            if (p <= 128 * NX) {
                collect(std::integral_constant<int, 1>{}, 128 * xw);
            } else {
                int c0 = 128 * xw;
#pragma clang loop unroll(disable)
                do {
                    collect(std::integral_constant<int, U2>{}, c0);
                    c0 += 128 * NX * U2;
                } while (c0 < p && dead == 0u);
            }
        }
        if (dead != 0u) ex.give_up();
        ex.raise_version();
        ++s;
    } while (s < last && dead == 0u);
    if (dead != 0u) return;
    if constexpr (OPT) {
        asm volatile("" ::: "memory");
        if (die == 0) {
            int k = 0;
            for (int l = l0; l < lines; l += dl, ++k)
                if (lane < 8) ex.store_state(8 * k + lane, a.opt.m + 16 * l + 2 * lane, a.opt.s + 16 * l + 2 * lane);
        }
    }
    ex.finish(last - first);
}

}  // namespace
}  // namespace bmgd
