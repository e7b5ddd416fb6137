// Softmax regression on large mini-batches: the updates of up to four passes in persistent kernels of many updates each.
//
// One update of eq. (2.1) has three phases, each of which needs what all workgroups did in the one before:
//   logits     U = X_b W               128 rows x 128 classes x a share of the features per workgroup; partial sums to memory
//   residual   R = softmax_rows(U) - onehot(y)   four rows per workgroup, partial sums added up in a fixed order, R as bf16
//   update     W <- W - (alpha / n_b) X_b' R     FT features x 128 classes per workgroup, all rows; master in fp32, bf16 copy
// Three launches (softmax_kernels.hip) spend as much on their edges as on their contractions: the launch, the first operands from
// memory, the last results to it, three times per update.  Here a phase begins when counters in memory say that what it reads is
// complete, and its rows of X, which depend on nothing, are requested before that.
//
// Counters (arrive / await): a workgroup that has written its part waits for its stores, then adds one to the counter of the part;
// readers poll.  What one workgroup writes and another reads (U, R, the bf16 copy of W) is stored and loaded at device scope, so it
// is never found in a compute unit's own cache.  A die's L2 serves such a load as fast as others if nobody has written the line since the die
// last had it (0.30 against 0.29 us per 32 KB and compute unit; 90 ns for a load that depends on the one before); the first load of a line
// freshly written at device scope goes beyond the die, whichever die wrote it (220 ns; words stored without a scope stay in the die's L2).  Invalidating caches between phases costs 2 us and more.  A phase's parts are counted in every update by
// every workgroup, also where a short last mini-batch leaves nothing to do, and nothing is awaited less often than in every update:
// so a count can only be reached by arrivals of the update that is waited for.
//   (an arrival for update s + 1 follows, through the waits in front of it, all arrivals for update s at the same counter)
//
// The rows of a mini-batch are gathered from X for both contractions: for the update the contraction runs over rows, and the operands
// (features or classes by rows) are read from the row-major tiles in shared memory with the transposing read, so nothing is ever
// stored transposed but the copy of W.
//
// All workgroups that take part must be running.  They meet before the first update; if some have not come in time, those that are
// there share the work among themselves (parts of a phase are dealt round): the same sums in the same order, down to one workgroup.
// A workgroup keeps its compute unit to itself from the meeting to the end of the launch, and another persistent kernel that waits for
// that unit gives up after its limit.  So a launch makes only as many updates as those that have come make in about an eighth of the limit;
// the next one goes on from there, with the counters as they are, and meets again.  All workgroups make everything in the first launch, or nearly
// so, and leave the others nothing to do.  (Launches that end often even where all have come were tried: with runs of several contexts in
// turn their workgroups stand on the device half and half most of the time, and a device that changes its queues at such a moment
// puts them back in an order that keeps a third kernel waiting past its limit.)
#include "bmgd_internal.h"
#include "glm_device.h"
#include "lds_load.h"

#include <algorithm>

namespace bmgd {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int TR = 128, TC = 128, TK = 64;          // rows and classes of a tile, and the depth of an operand tile
constexpr int kRowsPerItem = 4;                     // rows of a residual item: two wavefronts each
constexpr int kStages = 4;
constexpr int kStageBytes = (TR + TC) * TK * 2;
constexpr int kMaxRows = 2048;                      // of a mini-batch: its row numbers are kept in shared memory, twice
constexpr int kTsAt = 3 * kStageBytes;              // the update's transposed tile: behind the stages that are requested ahead
constexpr int kIdxAt = kTsAt + TC * (128 + 8) * 2;
constexpr int kRedAt = kIdxAt + 2 * kMaxRows * 4;
constexpr int kLds = kRedAt + 128;
constexpr int kAgentScope = 16;                     // sc1
constexpr int kLine = 32;                           // counters stand in lines of their own
constexpr long long kMeeting = 10000;               // ticks: 0.1 ms
constexpr int kSubs = 4, kRSubs = 32;               // counters a part's arrivals are spread over (one address takes 0.04 us per arrival)

template <int N> struct IntC { static constexpr int value = N; };

__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory"); }

// Until the first two tiles of nt have landed for this wavefront.  Of the first three the rows of X were requested first and the other operand
// (2 load instructions each) behind them; the fourth, and every further one, was requested whole (LT load instructions).
template <int LT>
__device__ __forceinline__ void wait_first(int nt)
{
    if (nt >= 4) wait_loads<2 + LT>();
    else if (nt == 3) wait_loads<2>();
    else wait_loads<0>();
}

// The operand tiles 0 .. nt - 1 (nt >= 1, the first kStages of them requested) in turn.  While the matrix instructions of a tile run the
// operands of the next one are read from shared memory (request: the tile that takes the place of this one; read: the operands that stand
// in two sets of registers; multiply: the products, each followed by the read of what takes the place of its other operand, if there is a
// next tile).  Everything that would be decided tile by tile is known to the compiler: an iteration's 12 or 16 matrix instructions are
// 200 cycles, those of two wavefronts to a SIMD 400, and twenty scalar instructions with their branches half of that.
template <int LT, class Set, class Request, class Read, class Begin, class Multiply>
struct Walk {
    int nt;
    Request& request;
    Read& read;
    Begin& begin;
    Multiply& multiply;

    // LEFT: tiles from t on (any number beyond kStages + 1 is like that)
    template <int LEFT>
    __device__ __forceinline__ void step(int t, Set& now, Set& next)
    {
        if constexpr (LEFT > 1) {
            wait_loads<(LEFT - 2 < 2 ? LEFT - 2 : 2) * LT>();
            __builtin_amdgcn_s_barrier();            // (the wait is for this wavefront's reads of tile t as well)
            asm volatile("" ::: "memory");
            if constexpr (LEFT > kStages) request(t + kStages);
            read(next, t + 1);
        }
        multiply(now, t, IntC<(LEFT > 1)>{});
    }
    template <int LEFT>
    __device__ __forceinline__ void rest(int t, Set& now, Set& next)
    {
        step<LEFT>(t, now, next);
        if constexpr (LEFT > 1) rest<LEFT - 1>(t + 1, next, now);
    }
    __device__ __forceinline__ void all()
    {
        Set even, odd;
        wait_first<LT>(nt);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read(even, 0);
        begin();
        int t = 0;
        for (; t + kStages + 1 < nt; t += 2) {
            step<kStages + 2>(t, even, odd);
            step<kStages + 2>(t + 1, odd, even);
        }
        switch (nt - t) {
        case 5: rest<5>(t, even, odd); break;
        case 4: rest<4>(t, even, odd); break;
        case 3: rest<3>(t, even, odd); break;
        case 2: rest<2>(t, even, odd); break;
        default: rest<1>(t, even, odd); break;
        }
    }
};

template <int LT, class Set, class Request, class Read, class Begin, class Multiply>
__device__ __forceinline__ void walk_tiles(int nt, Request& request, Read& read, Begin& begin, Multiply& multiply)
{
    Walk<LT, Set, Request, Read, Begin, Multiply>{nt, request, read, begin, multiply}.all();
}

// The same value, but what is worked out from it stays where it is used: left to itself the compiler keeps every address of every phase in
// registers for the whole kernel, and then has none left
__device__ __forceinline__ int here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ u32x2 to_bf16x4(const float (&v)[4])
{
    typedef __bf16 bf16x4_ __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(u32x2, __builtin_convertvector((f32x4{v[0], v[1], v[2], v[3]}), bf16x4_));
}

__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_mov<0xB1>(v));
    v = fmaxf(v, dpp_mov<0x4E>(v));
    v = fmaxf(v, dpp_mov<0x141>(v));
    v = fmaxf(v, dpp_mov<0x140>(v));
    v = fmaxf(v, __shfl_xor(v, 16));
    return fmaxf(v, __shfl_xor(v, 32));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t area(void* base, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);
}

// Work items of a phase: part k of those dealt round to the workgroups (workgroup b takes k = b, b + nwg, ...).  Consecutive workgroups
// go to the eight dies in turn; die x gets the x-th contiguous eighth of the items.
struct Deal {
    int items, per;
    __device__ __forceinline__ explicit Deal(int n) : items(n), per((n + 7) / 8) {}
    __device__ __forceinline__ int rounds() const { return 8 * per; }
    __device__ __forceinline__ int item(int k) const      // -1: none
    {
        const int i = (k & 7) * per + (k >> 3);
        return i < items ? i : -1;
    }
};

// KB groups of 512 classes: the sum of the partial sums of row j, in their order.  Every load is issued up front, or as many as leave the
// registers to what the whole kernel keeps in them.
template <int KB, int SP>
__device__ __forceinline__ void residual_sums(const SoftmaxPassArgs& a, __amdgpu_buffer_rsrc_t U, int j, int half, int lane, f32x4 (&sum)[KB])
{
    constexpr int G = SP * KB > 16 ? 16 / KB : SP;
#pragma unroll
    for (int s0 = 0; s0 < SP; s0 += G) {
        f32x4 q[G][KB];
#pragma unroll
        for (int sp = 0; sp < G; ++sp)
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const int c = min(4 * (lane + 64 * (half + 2 * k)), a.ldw - 4);
                q[sp][k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(U, (unsigned)c * 4u, (unsigned)(((size_t)(s0 + sp) * a.m_pad + j) * a.ldw * 4), kAgentScope));
            }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            sum[k] = s0 == 0 ? q[0][k] : sum[k] + q[0][k];
#pragma unroll
            for (int sp = 1; sp < G; ++sp) sum[k] += q[sp][k];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// (One piece of code behind the sums, whatever their number: twelve copies were half of the kernel.)
template <int KB>
__device__ __forceinline__ void residual_rows(const SoftmaxPassArgs& a, __amdgpu_buffer_rsrc_t U, __amdgpu_buffer_rsrc_t R, const int* idx, int nb, int j0,
                                              float* red, int wave, int lane_)
{
    const int lane = here(lane_);
    const int rr = wave >> 1, half = wave & 1, j = j0 + rr;
    const bool real = j < nb;
    f32x4 sum_q[KB];
    int label = -1;
    if (real) {
        label = a.y[idx[j]];
        if (a.splits == 1) residual_sums<KB, 1>(a, U, j, half, lane, sum_q);
        else if (a.splits == 2) residual_sums<KB, 2>(a, U, j, half, lane, sum_q);
        else if (a.splits == 4) residual_sums<KB, 4>(a, U, j, half, lane, sum_q);
        else residual_sums<KB, 8>(a, U, j, half, lane, sum_q);
    }
    float u[KB][4], mx = -INFINITY;
    if (real) {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const f32x4 t = sum_q[k];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                u[k][v] = 4 * (lane + 64 * (half + 2 * k)) + v < a.C ? t[v] : -INFINITY;      // padding classes (and clamped reads)
                mx = fmaxf(mx, u[k][v]);
            }
        }
        mx = wave_max(mx);
    }
    if (lane == 0) red[wave] = mx;
    wg_barrier();
    float sum = 0.f;
    if (real) {
        mx = fmaxf(red[wave & ~1], red[wave | 1]);
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                u[k][v] = expf(u[k][v] - mx);
                sum += u[k][v];
            }
        sum = group_sum(sum, 64);
    }
    if (lane == 0) red[8 + wave] = sum;
    wg_barrier();
    if (j >= (nb + TK - 1) / TK * TK) return;        // (rows that no operand tile of the update reaches)
    const float inv = real ? 1.f / (red[8 + (wave & ~1)] + red[8 + (wave | 1)]) : 0.f;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const int c = 4 * (lane + 64 * (half + 2 * k));
        float r[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) r[v] = real && c + v < a.C ? u[k][v] * inv - (c + v == label ? 1.f : 0.f) : 0.f;
        if (c < a.ldw) __builtin_amdgcn_raw_buffer_store_b64(to_bf16x4(r), R, (unsigned)c * 2u, (unsigned)((size_t)j * a.ldw * 2), kAgentScope);
    }
}

// FT: features of an update tile; OPT: an update rule other than the plain step.
// Eight wavefronts, two per SIMD: each pair w, w + 4 owns a quarter of the workgroup's tile (64 classes by 64 rows or FT / 2 features),
// and its two wavefronts take half of every operand tile's depth each: an operand is read from shared memory twice, not four times, per
// tile (64 + 32 KB per tile at 128 bytes a clock; 96 + 32 KB took 0.50 against 0.39 us).  Those reads run behind the matrix instructions of the tile
// before (Walk): a tile of the update takes 0.45 us with that, 0.67 without; one of the logits 0.70 and 0.73, most of it the wait for rows of X from
// memory (0.55 where they come from a die's L2).  All 256 registers are in use; FT = 128 spills 16 more (with state 19), FT = 64 and 96 with
// state 3 each: reloads in the first requests and the last tiles of a walk, and for FT = 128 with state in every tile of the update.
template <int FT, bool OPT>
__global__ void __launch_bounds__(kThreads, 2) softmax_pass_kernel(SoftmaxPassArgs a)
{
    extern __shared__ __align__(1024) unsigned char smem[];
    __shared__ int s_abort, s_rank, s_nwg;
    constexpr int FW = FT / 2, NF = FW / 16;         // features of a wavefront, in tiles of 16
    constexpr int NCX = FT / 8;                      // 16-byte chunks of a row's features; load instructions of an operand tile
    constexpr int LX = (NCX + kWaves - 1) / kWaves, LXLess = NCX / kWaves, kMoreLoads = NCX % kWaves ? NCX % kWaves : kWaves;   // wavefronts with LX of them; the others have LXLess
    constexpr unsigned kRAt = TK * FT * 2;           // the residual's part of a stage
    constexpr bool kEarlyWeights = FT < 128;         // master weights requested ahead of the products (for wider tiles the registers do not suffice)

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int kh = wave >> 2, wm = wave & 1, wn = (wave >> 1) & 1;
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    lds_byte* const lds = (lds_byte*)smem;
    const unsigned lds0 = (unsigned)(size_t)lds;
    int* const idx_all = reinterpret_cast<int*>(smem + kIdxAt);
    float* const red = reinterpret_cast<float*>(smem + kRedAt);

    // (what a launch leaves for the next one is another word than what it reads: its wavefronts read at any time)
    const int s_begin = *a.progress;
    if (s_begin >= a.updates) {
        if (blockIdx.x == 0 && tid == 0) *a.progress_next = s_begin;
        return;
    }
    // the meeting: word = closed (bit 31), workgroups that came in time (bits 16-30, once closed), tickets drawn (bits 0-15)
    PollGuard guard{a.sync + 1, a.timeout_ticks, 0, 0};
    if (a.meeting_ticks == 0) {                      // no time to meet: one workgroup alone
        if (blockIdx.x != 0) return;
        if (tid == 0) { s_rank = 0; s_nwg = 1; s_abort = 0; }
    } else if (tid == 0) {
        const unsigned G = gridDim.x;
        const unsigned got = __hip_atomic_fetch_add(a.meeting, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned ticket = got & 0xFFFFu;
        unsigned seen = got + 1;
        int nwg = 0;
        const long long t0 = wall_clock64();
        guard.arm();
        while (true) {
            if (seen >> 31) { nwg = (int)((seen >> 16) & 0x7FFFu); break; }
            if (seen == G) { nwg = (int)G; break; }
            // The first one waits for the others as long as those that have come would take for the launch: no more than is lost by going on with
            // them, and two kernels that have half of the units each do not keep each other waiting.  (All come to an idle device in kMeeting.)
            const long long waited = wall_clock64() - t0;
            if (ticket == 0 && waited >= kMeeting && waited * (seen & 0xFFFFu) >= a.meeting_ticks) {
                // (a workgroup that comes in between makes the exchange fail, and the loop looks again)
                const unsigned closed = seen | seen << 16 | 1u << 31;
                if (__hip_atomic_compare_exchange_strong(a.meeting, &seen, closed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) seen = closed;
                continue;
            }
            if (guard.expired()) { nwg = 0; break; } // (the first one always decides long before this)
            seen = __hip_atomic_load(a.meeting, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_rank = nwg == (int)G ? (int)blockIdx.x : (int)ticket;
        s_nwg = nwg;
        s_abort = 0;
    }
    wg_barrier();
    const int rank = __builtin_amdgcn_readfirstlane(s_rank), nwg = __builtin_amdgcn_readfirstlane(s_nwg);
    if (rank >= nwg) return;                         // came too late

    const int S = a.splits, tiles_c = a.ldw / TC, tiles_r = a.m_pad / TR, tiles_f = (a.p + FT - 1) / FT;
    const Deal dl(S * tiles_r * tiles_c), dr(a.n_pad / kRowsPerItem), dg(tiles_f * tiles_c);
    const int CG = tiles_c % 2 ? tiles_c : tiles_c / 2, ncg = tiles_c / CG;      // groups of class tiles, and of feature tiles,
    const int FG = tiles_f % S ? tiles_f : tiles_f / S;                          // that one die's items have in common
    unsigned* const cnt_u = a.counters;                                          // [tiles_r][kSubs]
    unsigned* const cnt_r = cnt_u + (size_t)tiles_r * kSubs * kLine;             // [kRSubs]
    unsigned* const cnt_w = cnt_r + (size_t)kRSubs * kLine;                      // [tiles_c][kSubs]
    const __amdgpu_buffer_rsrc_t U = area(a.U, (size_t)S * a.m_pad * a.ldw * 4), R = area(a.R, (size_t)a.n_pad * a.ldw * 2);

    // until the NSUB counters at `first` have seen `updates` times `items` arrivals; false: given up
    auto await = [&](auto NSUB, const unsigned* first, int items, unsigned updates) -> bool {
        constexpr int n = decltype(NSUB)::value;
        if (wave == 0) {
            const int q = min(here(lane), n - 1);
            const unsigned target = (unsigned)((items - q + n - 1) / n) * updates;
            guard.arm();
            while (true) {
                const unsigned v = __hip_atomic_load(first + q * kLine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__all((int)(v - target) >= 0)) break;
                if (guard.expired()) { s_abort = 1; break; }
            }
        }
        wg_barrier();
        return __builtin_amdgcn_readfirstlane(s_abort) == 0;
    };
    // all stores of the workgroup have reached memory, and its reads of shared memory have returned
    auto arrive = [&](unsigned* counter) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (tid == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // ---- logits -------------------------------------------------------------------------------------
    struct Logits { int split, rt, ct, kb, nt; } L{0, 0, 0, 0, 0};
    const unsigned short* lx[2];                     // a lane's rows of X: position lane % 8 of row 8 (wave + 8 h) + lane / 8
    const int kc = ((lane & 7) ^ (lane >> 3)) * 8;   // (chunk c of row r stands at c ^ (r mod 8))
    const unsigned short* const zeros = a.WbT + a.p; // (padding of the copy's first row: there is some if p is not a multiple of TK)
    auto l_at = [&](int item) {
        const int cc = item % CG, rest = item / CG, rt = rest % tiles_r, sg = rest / tiles_r;
        L.split = sg / ncg;
        L.ct = (sg % ncg) * CG + cc;
        L.rt = rt;
        L.kb = L.split * a.k_per_split;
        L.nt = max(0, (min(a.p, L.kb + a.k_per_split) - L.kb + TK - 1) / TK);
    };
    auto l_request_x = [&](int t) {
        const int k0 = L.kb + t * TK;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const unsigned short* p = lx[h] + t * TK;
            if (k0 + TK > a.p) p = k0 + here(kc) < a.p ? p : zeros;
            load_to_lds(p, lds0 + (unsigned)(t % kStages) * kStageBytes + (unsigned)(wave + kWaves * h) * 1024);
        }
    };
    // the first tiles' rows of X, which wait for nothing
    auto l_begin = [&](const int* idx, int nb) {
        if (L.rt * TR >= nb) return;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            lx[h] = a.X + (size_t)idx[min(L.rt * TR + 8 * (wave + kWaves * h) + (here(lane) >> 3), nb - 1)] * a.p + L.kb + here(kc);
        for (int t = 0; t < kStages - 1; ++t)
            if (t < L.nt) l_request_x(t);
    };
    // The rows of X that the next update's logits read here, into this die's L2 (a word from every line of 128 bytes, but for the first tiles,
    // which come straight behind): each of the CG workgroups that have the rows in common takes its share, as far as kAhead loads go.
    // us per update without and with: 32.0 / 30.8 (3072 features, 1024 rows, 1000 classes: products of the logits 8.4 / 5.6), 103 / 95 (4096, 2048,
    // 2000); with seven tiles 22.6 / 23.3 (800, 1024, 1000, Adam).
    constexpr int kAhead = 2, kAheadTiles = 8;       // loads of a thread; tiles of the logits' depth from which it pays
    struct Ahead {
        unsigned v[kAhead];
    };
    auto l_ahead = [&](Ahead& w, const int* idx, int nb, int cc) {
        const int lines = TR * (L.nt - (kStages - 1)), tid_ = here(tid);
#pragma unroll
        for (int h = 0; h < kAhead; ++h) {
            const int e = (cc + CG * h) * kThreads + tid_, r = e % TR, t = kStages - 1 + e / TR;
            w.v[h] = 0;
            if (e < lines) w.v[h] = *reinterpret_cast<const unsigned*>(a.X + (size_t)idx[min(L.rt * TR + r, nb - 1)] * a.p + L.kb + t * TK);
        }
    };
    // the sums of the two wavefronts of a pair over the halves of the depth: each adds up and keeps two of its four rows of tiles
    // (classes); acc[0], acc[1] hold them afterwards
    auto meet_halves = [&](auto& acc) {
        constexpr int N = sizeof(acc[0]) / sizeof(f32x4);
        const int lane = here(tid) & 63;
        unsigned char* const mine = smem + wave * 8192 + lane * 16;
        const unsigned char* const other = smem + (wave ^ 4) * 8192 + lane * 16;
        wg_barrier();                                // all operands read: the stages are free
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) *reinterpret_cast<f32x4*>(mine + (i * N + j) * 1024) = kh ? acc[i][j] : acc[2 + i][j];
        wg_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const f32x4 o = *reinterpret_cast<const f32x4*>(other + (i * N + j) * 1024);
                const f32x4 s = kh ? acc[2 + i][j] : acc[i][j];
                acc[i][j] = kh ? o + s : s + o;      // (first half of the depth + second half)
            }
    };
    auto l_rest = [&]() {
        const int lane = here(tid) & 63, l16 = lane & 15, lq = lane >> 4, kc = ((lane & 7) ^ (lane >> 3)) * 8;
        const unsigned short* ws[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) ws[h] = a.WbT + (size_t)(L.ct * TC + 8 * (wave + kWaves * h) + (lane >> 3)) * a.ldwt + L.kb + kc;
        auto request_w = [&](int t) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                load_to_lds_agent(ws[h] + t * TK, lds0 + (unsigned)(t % kStages) * kStageBytes + TR * TK * 2 + (unsigned)(wave + kWaves * h) * 1024);
        };
        for (int t = 0; t < kStages - 1; ++t)
            if (t < L.nt) request_w(t);
        if (kStages - 1 < L.nt) {
            l_request_x(kStages - 1);
            request_w(kStages - 1);
        }
        f32x4 acc[4][4];                             // classes 16 i + 4 lq .., row 16 j + l16 of the wavefront's quarter
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int c = ((4 * kh + lq) ^ (l16 & 7)) * 16;
        struct Rows {
            bf16x8 f[4];
        };
        auto at = [&](int t) -> const unsigned char* { return smem + (t % kStages) * kStageBytes + c; };
        auto request = [&](int t) {
            l_request_x(t);
            request_w(t);
        };
        auto read = [&](Rows& x, int t) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x.f[i] = *reinterpret_cast<const bf16x8*>(at(t) + (wm * 64 + 16 * i + l16) * (TK * 2));
        };
        bf16x8 fw[4];                                // of the copy of W
        auto read_w = [&](int t, int i) { fw[i] = *reinterpret_cast<const bf16x8*>(at(t) + TR * TK * 2 + (wn * 64 + 16 * i + l16) * (TK * 2)); };
        auto multiply = [&](const Rows& x, int t, auto MORE) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i], x.f[j], acc[i][j], 0, 0, 0);
                if constexpr (decltype(MORE)::value) read_w(t + 1, i);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto begin = [&]() {
#pragma unroll
            for (int i = 0; i < 4; ++i) read_w(0, i);
        };
        if (L.nt > 0) walk_tiles<4, Rows>(L.nt, request, read, begin, multiply);
        meet_halves(acc);
        const unsigned lane_at = (unsigned)(l16 * a.ldw + 4 * lq) * 4u;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const size_t row = (size_t)L.split * a.m_pad + L.rt * TR + wm * 64 + 16 * j;
                const int cls = L.ct * TC + wn * 64 + 16 * (2 * kh + i);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), U, lane_at, (unsigned)((row * a.ldw + cls) * 4), kAgentScope);
            }
    };

    // ---- update -------------------------------------------------------------------------------------
    int g_ft = 0, g_ct = 0;
    auto g_at = [&](int item) {
        const int cc = item % CG, rest = item / CG, f = rest % FG, fg = rest / FG;
        g_ct = (fg % ncg) * CG + cc;
        g_ft = (fg / ncg) * FG + f;
    };
    // rows of X for the update: row i of an operand tile stands with its 16-byte chunks in place c ^ swizzle(i), so that the four rows of a
    // transposing read fall on different banks (rows of 192 and 64 bytes do by themselves)
    constexpr int kSwz = FT == 128 ? 7 : FT == 64 ? 3 : 0;
    int gx_row[LX], gx_col[LX];
#pragma unroll
    for (int h = 0; h < LX; ++h) {
        const int q = (wave + kWaves * h) * 64 + lane, r = q / NCX;
        gx_row[h] = r;
        gx_col[h] = ((q % NCX) ^ (2 * (r & kSwz))) * 8;
    }
    auto g_put = [&](const unsigned short* src, int t, int h) {
        load_to_lds(src, lds0 + (unsigned)(t % kStages) * kStageBytes + (unsigned)(wave + kWaves * h) * 1024);
    };
    auto g_src = [&](int row, int col) { return a.X + (size_t)row * a.p + min(g_ft * FT + col, a.p - 8); };
    auto g_request_x = [&](int t, const int* idx, int nb) {
#pragma unroll
        for (int h = 0; h < LX; ++h) {
            if (wave + kWaves * h >= NCX) continue;
            g_put(g_src(idx[min(t * TK + here(gx_row[h]), nb - 1)], here(gx_col[h])), t, h);
        }
    };
    // (the residual of rows beyond the mini-batch is zero)
    auto g_begin = [&](const int* idx, int nb) {
        const int nt = (nb + TK - 1) / TK;
        for (int t = 0; t < kStages - 1; ++t)
            if (t < nt) g_request_x(t, idx, nb);
    };
    // transposing reads: lane l points at four elements of row 8 lq + 4 q + l16 / 4, and receives one column of four rows
    unsigned rd_r[2][4], rd_x[2][NF];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int row = kh * 32 + 8 * lq + 4 * q + (l16 >> 2), half = (l16 & 3) >> 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) rd_r[q][i] = kRAt + (unsigned)(row * TC * 2 + ((2 * (4 * wn + i) + half) ^ (2 * (row & 7))) * 16 + (l16 & 1) * 8);
#pragma unroll
        for (int j = 0; j < NF; ++j) rd_x[q][j] = (unsigned)(row * FT * 2 + ((2 * (NF * wm + j) + half) ^ (2 * (row & kSwz))) * 16 + (l16 & 1) * 8);
    }
    // master weights: this lane's four classes of each of its features
    struct Block {
        f32x4 v[2][NF];
    };
    auto g_load = [&](Block& b, const float* from) { // (from clamped addresses)
        const int lane = here(tid) & 63, l16 = lane & 15, lq = lane >> 4;
        const int f0 = g_ft * FT + wm * FW + l16, c0 = g_ct * TC + wn * 64 + 32 * kh + 4 * lq;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) b.v[i][j] = *reinterpret_cast<const f32x4*>(from + (size_t)min(f0 + 16 * j, a.p - 1) * a.ldw + c0 + 16 * i);
    };
    auto g_store = [&](const Block& b, float* to) {
        const int lane = here(tid) & 63, l16 = lane & 15, lq = lane >> 4;
        const int f0 = g_ft * FT + wm * FW + l16, c0 = g_ct * TC + wn * 64 + 32 * kh + 4 * lq;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
                if (f0 + 16 * j < a.p) *reinterpret_cast<f32x4*>(to + (size_t)(f0 + 16 * j) * a.ldw + c0 + 16 * i) = b.v[i][j];
    };
    auto g_rest = [&](int s, const int* idx, int nb, Block& w) {
        const int nt = (nb + TK - 1) / TK;
        const int lane = here(tid) & 63, rrow = 4 * wave + (lane >> 4);
        const unsigned short* const rs = a.R + (size_t)rrow * a.ldw + g_ct * TC + ((lane & 15) ^ (2 * (rrow & 7))) * 8;
        auto request_r = [&](int t) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                load_to_lds_agent(rs + (size_t)(t * TK + 32 * h) * a.ldw, lds0 + (unsigned)(t % kStages) * kStageBytes + kRAt + (unsigned)(wave + kWaves * h) * 1024);
        };
        for (int t = 0; t < kStages - 1; ++t)
            if (t < nt) request_r(t);
        if (kStages - 1 < nt) {
            g_request_x(kStages - 1, idx, nb);
            request_r(kStages - 1);
        }
        f32x4 acc[4][NF];                            // classes 16 i + 4 lq .., feature 16 j + l16 of the wavefront's quarter
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        int ahead[LX];                               // row numbers of the tile that is requested next
        auto look_up = [&](int t) {
#pragma unroll
            for (int h = 0; h < LX; ++h) ahead[h] = idx[min(t * TK + gx_row[h], nb - 1)];
        };
        look_up(kStages);
        auto request = [&](int t) {
#pragma unroll
            for (int h = 0; h < LX; ++h) {
                if (wave + kWaves * h >= NCX) continue;
                g_put(g_src(ahead[h], gx_col[h]), t, h);
            }
            request_r(t);
            look_up(t + 1);
        };
        struct Rows {
            bf16x8 f[NF];
        };
        bf16x8 fr[4];                                // of the residual
        auto read_tr = [&](int t, unsigned at0, unsigned at1) {
            lds_byte* st = lds + (t % kStages) * kStageBytes;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(st + at0));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(st + at1));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto read = [&](Rows& x, int t) {
#pragma unroll
            for (int j = 0; j < NF; ++j) x.f[j] = read_tr(t, rd_x[0][j], rd_x[1][j]);
        };
        auto begin = [&]() {
#pragma unroll
            for (int i = 0; i < 4; ++i) fr[i] = read_tr(0, rd_r[0][i], rd_r[1][i]);
        };
        auto multiply = [&](const Rows& x, int t, auto MORE) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < NF; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[i], x.f[j], acc[i][j], 0, 0, 0);
                if constexpr (decltype(MORE)::value) fr[i] = read_tr(t + 1, rd_r[0][i], rd_r[1][i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (LX == LXLess || wave < kMoreLoads) walk_tiles<LX + 2, Rows>(nt, request, read, begin, multiply);
        else walk_tiles<LXLess + 2, Rows>(nt, request, read, begin, multiply);
        if constexpr (!kEarlyWeights) g_load(w, a.W);
        meet_halves(acc);
        const int tid_ = here(tid), l16 = tid_ & 15, lq = (tid_ & 63) >> 4;
        const int f0 = g_ft * FT + wm * FW + l16, c0 = g_ct * TC + wn * 64 + 32 * kh + 4 * lq;
        const float alpha = a.lr_tab ? a.lr_tab[min(a.lr_base + s, a.lr_len - 1)] : a.alpha;
        const float inv_nb = 1.f / (float)nb, scale = alpha * inv_nb;
        float oc1 = 1.f, oc2 = 1.f;
        if (OPT && a.opt.kind == kOptAdam) opt_corrections(a.opt, a.opt.k_base + s + 1, oc1, oc2);
        unsigned short* const Ts = reinterpret_cast<unsigned short*>(smem + kTsAt);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const int f = f0 + 16 * j, c = c0 + 16 * i;
                float nw[4];
                if constexpr (!OPT) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) nw[v] = w.v[i][j][v] - scale * acc[i][j][v];
                } else {
                    const size_t at = (size_t)min(f, a.p - 1) * a.ldw + c;
                    f32x4 m = *reinterpret_cast<const f32x4*>(a.opt.m + at), sv = {0.f, 0.f, 0.f, 0.f};
                    if (a.opt.kind == kOptAdam) sv = *reinterpret_cast<const f32x4*>(a.opt.s + at);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float mv = m[v], s2 = sv[v];
                        nw[v] = opt_update(a.opt, w.v[i][j][v], acc[i][j][v] * inv_nb, alpha, mv, s2, oc1, oc2);
                        m[v] = c + v < a.C ? mv : 0.f;
                        sv[v] = c + v < a.C ? s2 : 0.f;
                    }
                    if (f < a.p) {
                        *reinterpret_cast<f32x4*>(a.opt.m + at) = m;
                        if (a.opt.kind == kOptAdam) *reinterpret_cast<f32x4*>(a.opt.s + at) = sv;
                    }
                }
                // (classes beyond C stay zero whatever the rows hold)
#pragma unroll
                for (int v = 0; v < 4; ++v) nw[v] = c + v < a.C ? nw[v] : 0.f;
                w.v[i][j] = f32x4{nw[0], nw[1], nw[2], nw[3]};
                const u32x2 b = to_bf16x4(nw);
                const int cl = wn * 64 + 32 * kh + 16 * i + 4 * lq, fl = wm * FW + 16 * j + l16;
                Ts[(cl + 0) * (FT + 8) + fl] = (unsigned short)b.x;
                Ts[(cl + 1) * (FT + 8) + fl] = (unsigned short)(b.x >> 16);
                Ts[(cl + 2) * (FT + 8) + fl] = (unsigned short)b.y;
                Ts[(cl + 3) * (FT + 8) + fl] = (unsigned short)(b.y >> 16);
            }
        wg_barrier();
        const __amdgpu_buffer_rsrc_t copy = area(a.WbT, (size_t)a.ldw * a.ldwt * 2);
#pragma unroll
        for (int e0 = 0; e0 < TC * NCX; e0 += kThreads) {
            const int e = e0 + tid_, cl = e / NCX, fc = e - cl * NCX;
            const u32x4 v = *reinterpret_cast<const u32x4*>(&Ts[cl * (FT + 8) + 8 * fc]);
            if (g_ft * FT + 8 * fc < a.p)
                __builtin_amdgcn_raw_buffer_store_b128(v, copy, (unsigned)(((size_t)(g_ct * TC + cl) * a.ldwt + g_ft * FT + 8 * fc) * 2), 0, kAgentScope);
        }
    };

    // row numbers of mini-batch m of pass t (repeated beyond its end), in order of the loads of this wavefront
    auto request_idx = [&](int t, int m, int nb, int which) {
        const int* src = a.perm + (size_t)t * a.perm_stride + (size_t)m * a.n;
        for (int c = wave; c * 64 < nb; c += kWaves)
            load_word_to_lds(src + min(c * 64 + lane, nb - 1), lds0 + kIdxAt + (unsigned)which * (kMaxRows * 4) + (unsigned)c * 256);
    };

    const int M = a.M, updates = s_begin + min(a.updates - s_begin, max(a.updates_alone, (int)(a.updates_each * (float)nwg)));
    if (rank == 0 && tid == 0) {
        *a.progress_next = updates;
        *a.next_meeting = 0;                         // (the word of the launch before, which has ended, is that of the next one)
    }
    const int t_begin = s_begin / M, m_begin = s_begin - t_begin * M, nb_begin = min(a.n, a.rows - m_begin * a.n);
    const int* const idx_begin = idx_all + (s_begin & 1) * kMaxRows;
    request_idx(t_begin, m_begin, nb_begin, s_begin & 1);
    wait_loads<0>();
    wg_barrier();
    const int l_first = rank < dl.rounds() ? dl.item(rank) : -1, r_first = rank < dr.rounds() ? dr.item(rank) : -1, g_first = rank < dg.rounds() ? dg.item(rank) : -1;
    // (where the first items of each update stand is worked out once: a division is 0.1 us)
    if (l_first >= 0) l_at(l_first);
    const Logits L_first = L;
    if (g_first >= 0) g_at(g_first);
    const int g_ft_first = g_ft, g_ct_first = g_ct, cc_first = max(l_first, 0) % CG;
    if (l_first >= 0) l_begin(idx_begin, nb_begin);
    for (int s = s_begin, t = t_begin, m = m_begin; s < updates; ++s) {
        const int nb = min(a.n, a.rows - m * a.n);
        const int* const idx = idx_all + (s & 1) * kMaxRows;
        for (int k = rank; k < dl.rounds(); k += nwg) {
            const int item = dl.item(k);
            if (item < 0) continue;
            if (k != rank) { l_at(item); l_begin(idx, nb); }
            if (!await(IntC<kSubs>{}, cnt_w + (size_t)L.ct * kSubs * kLine, tiles_f, (unsigned)s)) return;
            if (L.rt * TR < nb) l_rest();
            arrive(cnt_u + (size_t)(L.rt * kSubs + (L.split * tiles_c + L.ct) % kSubs) * kLine);
        }
        // the next update's row numbers, and the first rows of X for this one's update
        const int m1 = m + 1 < M ? m + 1 : 0, t1 = m + 1 < M ? t : t + 1, nb1 = min(a.n, a.rows - m1 * a.n);
        if (s + 1 < updates) request_idx(t1, m1, nb1, (s + 1) & 1);
        if (g_first >= 0) { g_ft = g_ft_first; g_ct = g_ct_first; g_begin(idx, nb); }
        for (int k = rank; k < dr.rounds(); k += nwg) {
            const int item = dr.item(k);
            if (item < 0) continue;
            const int j0 = item * kRowsPerItem;
            if (!await(IntC<kSubs>{}, cnt_u + (size_t)(j0 / TR) * kSubs * kLine, S * tiles_c, (unsigned)s + 1)) return;
            if (a.ldw <= 512) residual_rows<1>(a, U, R, idx, nb, j0, red, wave, lane);
            else if (a.ldw <= 1024) residual_rows<2>(a, U, R, idx, nb, j0, red, wave, lane);
            else residual_rows<4>(a, U, R, idx, nb, j0, red, wave, lane);
            arrive(cnt_r + (size_t)(item % kRSubs) * kLine);
        }
        Ahead ahead{};
        if (r_first >= 0 && l_first >= 0 && L_first.nt >= kAheadTiles && s + 1 < updates && L_first.rt * TR < nb1) {
            L = L_first;
            l_ahead(ahead, idx_all + ((s + 1) & 1) * kMaxRows, nb1, cc_first);
        }
        for (int k = rank; k < dg.rounds(); k += nwg) {
            const int item = dg.item(k);
            if (item < 0) continue;
            if (k != rank) { g_at(item); g_begin(idx, nb); }
            Block w;
            if constexpr (kEarlyWeights) g_load(w, a.W);
            if (!await(IntC<kRSubs>{}, cnt_r, dr.items, (unsigned)s + 1)) return;
            g_rest(s, idx, nb, w);
            arrive(cnt_w + (size_t)(g_ct * kSubs + g_ft % kSubs) * kLine);
            g_store(w, a.W);                         // what only this workgroup reads again leaves behind what the others wait for
        }
        asm volatile("" :: "v"(ahead.v[0]), "v"(ahead.v[1]));
        t = t1;
        m = m1;
        if (s + 1 < updates) {
            // (behind an arrival the row numbers have landed for the whole workgroup)
            if (g_first < 0) {
                wait_loads<0>();
                wg_barrier();
            }
            if (l_first >= 0) { L = L_first; l_begin(idx_all + ((s + 1) & 1) * kMaxRows, nb1); }
        }
    }
}

typedef void (*PassKernel)(SoftmaxPassArgs);

PassKernel pass_kernel(int ft, bool opt)
{
    switch (ft) {
    case 32: return opt ? softmax_pass_kernel<32, true> : softmax_pass_kernel<32, false>;
    case 64: return opt ? softmax_pass_kernel<64, true> : softmax_pass_kernel<64, false>;
    case 96: return opt ? softmax_pass_kernel<96, true> : softmax_pass_kernel<96, false>;
    default: return opt ? softmax_pass_kernel<128, true> : softmax_pass_kernel<128, false>;
    }
}

// Features of an update tile: the width with which the last round of tiles is least in vain
int pass_features(int p, int tiles_c, int num_cus)
{
    int best = 32;
    long long cost = -1;
    for (int ft = 32; ft <= 128; ft += 32) {
        const long long rounds = ((long long)((p + ft - 1) / ft) * tiles_c + num_cus - 1) / num_cus;
        const long long c = rounds * (ft + TC);
        if (cost < 0 || c < cost) { cost = c; best = ft; }
    }
    return best;
}

// Ticks of the device's clock (100 MHz) that one workgroup takes for an update alone: its tiles of both contractions, 64 deep or 64 rows long,
// and what an item costs besides.  ms, measured / as here: 6.0 / 6.8 (3072 features, 1024 rows, 1000 classes; Adam 7.9 / 10.3), 20.4 / 24.0 (4096,
// 2048, 2000; Adam 29.7 / 33.2), 30.9 / 29.2 (16384, 512, 2000), 3.7 / 2.9 (4096, 250, 1000), 1.15 / 1.47 (1160, 651, 247), 1.2 / 1.4 (8, 2048, 2).
long long pass_alone_ticks(const SoftmaxDims& d, int p, int ft, bool opt)
{
    const long long tiles_c = d.c_pad / TC, tiles_r = d.m_pad / TR, tiles_f = (p + ft - 1) / ft;
    const long long logits = d.splits * tiles_r * tiles_c, depth = tiles_r * tiles_c * ((p + TK - 1) / TK);
    const long long residual = d.n_pad / kRowsPerItem, update = tiles_f * tiles_c;
    return 400 * logits + 75 * depth + 250 * residual + update * (400 + 45 * (d.n_pad / TK) + (opt ? 14 * ft : 0));
}

int pass_groups(const SoftmaxDims& d, int p, int num_cus, int ft)
{
    const int tiles_c = d.c_pad / TC;
    const int items = std::max({d.splits * (d.m_pad / TR) * tiles_c, d.n_pad / kRowsPerItem, (p + ft - 1) / ft * tiles_c});
    return std::min(num_cus, (items + 7) / 8 * 8);
}

}  // namespace

size_t softmax_pass_counter_bytes(const SoftmaxDims& d)
{
    return (size_t)(3 + d.m_pad / TR * kSubs + kRSubs + d.c_pad / TC * kSubs) * kLine * 4;
}

// Against the three launches, us per update, this kernel / launches: few features beside many rows 16.3 / 23.4 (8 features, 1100 rows, 10
// classes), 20.2 / 32.2 (40, 2048, 10), 20.3 / 26.0 (136, 1100, 2; Adam 22.9 / 35.5), 26.7 / 45.1 (264, 2048, 1000); few rows 12.2 / 14.8 (1032, 8, 2);
// 0.48 to 0.86 of them over 8 to 16384 features, 8 to 2048 rows and 2 to 2000 classes, and at most 0.96 for a run of one update.  More rows
// than kMaxRows take the launches because their numbers, of this mini-batch and the next, would no longer fit shared memory.
bool softmax_pass_eligible(int64_t p, int64_t n, int64_t C)
{
    return n <= kMaxRows && p <= 16384 && C <= 2048;
}

hipError_t softmax_pass_prepare(int64_t p, int64_t n, int64_t C, bool opt, int num_cus, bool* fits)
{
    *fits = false;
    const SoftmaxDims d = softmax_dims(p, n, C);
    const void* k = reinterpret_cast<const void*>(pass_kernel(pass_features((int)p, d.c_pad / TC, num_cus), opt));
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kThreads, kLds);
    if (e != hipSuccess) return e;
    *fits = per_cu >= 1;
    return hipSuccess;
}

hipError_t softmax_pass(SoftmaxPassArgs a, const SoftmaxDims& d, void* counters, int num_cus, long long hold_ticks, hipStream_t stream)
{
    if (a.n > kMaxRows || d.c_pad != a.ldw || d.m_pad / TR * TR != d.m_pad) return hipErrorInvalidValue;
    a.M = (a.rows + a.n - 1) / a.n;
    a.m_pad = d.m_pad;
    a.n_pad = d.n_pad;
    a.splits = d.splits;
    a.k_per_split = d.k_per_split;
    unsigned* const meetings = static_cast<unsigned*>(counters);
    int* const progress = static_cast<int*>(counters) + 2 * kLine;
    a.counters = meetings + 3 * kLine;
    hipError_t e = launch_fill_zero(counters, softmax_pass_counter_bytes(d), stream);
    if (e != hipSuccess) return e;
    const int ft = pass_features(a.p, d.c_pad / TC, num_cus);
    const bool opt = a.opt.kind != kOptSgd;
    const dim3 grid((unsigned)pass_groups(d, a.p, num_cus, ft));
    const long long alone = pass_alone_ticks(d, a.p, ft, opt);
    a.updates = a.npass * a.M;
    a.updates_alone = (int)std::min<long long>(std::max(1LL, hold_ticks / alone), a.updates);
    // (an update of all workgroups takes 1.2 to 4 times what one alone takes divided by their number, the more the less of it there is)
    a.updates_each = (float)hold_ticks / (4.f * (float)alone);
    a.meeting_ticks = hold_ticks < 125 ? 0 : std::min(hold_ticks, alone * a.updates_alone);
    for (int s = 0, launch = 0; s < a.updates; s += a.updates_alone, ++launch) {
        a.meeting = meetings + (launch & 1) * kLine;
        a.next_meeting = meetings + (~launch & 1) * kLine;
        a.progress = progress + (launch & 1);
        a.progress_next = progress + (~launch & 1);
        hipLaunchKernelGGL(pass_kernel(ft, opt), grid, dim3(kThreads), kLds, stream, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace bmgd
