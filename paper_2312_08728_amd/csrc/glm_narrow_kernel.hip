// Fused mini-batch gradient + update for rows of up to 1024 floats (least squares, logistic) when the rows a
// workgroup takes per step fit its registers; persistent over all steps of up to four passes, on G workgroups, one per
// compute unit.
//
// A step of eq. (2.1) on such rows moves little data (a few KB per workgroup), so the chain of steps is bound by the
// exchange of the gradient sums between the workgroups, and the kernel's job is to put nothing else on that path:
//
//   * A row is held by L cooperating lanes of a row wavefront (L a power of two, 64 / L rows side by side, PF rows
//     one after the other per lane; lane l owns the columns V (l + L k) .. + V - 1, k < CPL).  RW row wavefronts
//     per workgroup.
//   * Each row wavefront holds TWO groups of rows in registers and alternates between them: the group used in step
//     s is refilled, as soon as it has been used, with the rows of step s + 2 (rows do not depend on theta).  Rows
//     therefore have a whole step to arrive and are never copied between registers while in flight.  The loop over
//     steps is straight-line code (two steps per trip, one exit at the bottom, steps past the end run empty), so
//     that the compiler's count of loads in flight is exact and a step waits only for its own rows.
//   * The row wavefronts never touch global memory except for rows: their sums go to shared memory, and four
//     exchange wavefronts (glm_exchange.h), one per SIMD, carry them to the other workgroups and bring the new theta
//     back.  Row wavefronts wait for theta on a flag in shared memory.
//
// Two forms.  Eight row wavefronts, sums added up slice by slice, over two levels or in two trips over the fabric per step (G a multiple of 8): where G p
// is large.  Twelve row wavefronts (the workgroup's sixteen fill the unit), one trip per step, any G, p <= 512: where every workgroup
// can add up the few sums itself; they hold fewer floats of a row each (registers), but fewer workgroups are what is wanted there.
// Odd rows of up to 256 floats in the first form take twelve as well where these hold them (2.96 us per update at p = 201, n = 1500, 2.81 at 202 with
// eight; callers read the number of threads in the statistics).
#include "glm_exchange.h"

#include <hip/hip_ext.h>

#include <algorithm>

namespace bmgd {

namespace {

// Registers: two groups of PF rows of CPL * V floats per lane.  Loads: a group is PF * (CPL + 2) of them (chunks,
// response, next index), and the two groups' loads together must stay below the 63 that a wavefront's count of
// loads in flight can hold.
constexpr bool narrow_shape_ok(int v, int cpl, int pf, int rw)
{
    return (v == 4 || (rw > kRowWaves && cpl == 1)) && cpl <= 4 && pf <= 8 && v * cpl * pf <= (rw > kRowWaves ? 24 : 32) && pf * (cpl + 2) <= 24;
}

// Wavefronts 0 .. 3 are the exchange wavefronts (the hardware deals the wavefronts of a workgroup out to the four
// SIMDs in turn, so each SIMD gets one), the others the RW row wavefronts.
constexpr int kXWaves = 4;
constexpr int narrow_block(int rw) { return 64 * (kXWaves + rw); }

// The k-th of two or four values.  (Arguments by value: a choice between elements of an array that the compiler has not yet taken apart
// becomes an indexed load from scratch.)
__device__ __forceinline__ float pick2(int k, float v0, float v1) { return k == 1 ? v1 : v0; }
__device__ __forceinline__ float pick4(int k, float v0, float v1, float v2, float v3) { return (k & 2) != 0 ? pick2(k & 1, v2, v3) : pick2(k & 1, v0, v1); }

// EX: how the sums are exchanged: in one trip, with so many pairs of columns to an exchange wavefront (2, 4, 8, ... 64), over two levels or in two
// trips.  (A kernel each: the code of several in one needs more scalar registers than there are, and reads them back in the middle of
// a step.)
constexpr int kTwoTrips = 0, kByDie = 1;
template <int V, int CPL, int PF, int RW, int EX, bool OPT>
__global__ void __launch_bounds__(narrow_block(RW)) glm_narrow_kernel(ExchangeArgs a)
{
    extern __shared__ __align__(16) float smem[];
    __shared__ int s_abort;                          // set by the exchange wavefront when a wait ran out
    __shared__ unsigned s_theta_version;             // versions of theta delivered to shared memory so far
    __shared__ unsigned s_sent;                      // raised by the exchange wavefronts: a step's sums are on their way
    __shared__ unsigned s_published;                 // publications of row wavefronts, counted over all steps
    __shared__ unsigned s_xarrived[kXWaves], s_xconsumed;   // hand-over of partial sums between the exchange wavefronts

    constexpr bool ONE = EX >= 2, kGated = ONE ? EX > 8 : EX == kByDie;   // (whether rows wait for s_sent)
    constexpr int E = CPL * V;                       // floats of a row held per lane
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = gridDim.x;
    const int g = blockIdx.x;
    const int p = a.p;
    const int L = a.L;
    const int width = a.width;                       // positions of a row (glm_exchange.h)
    const int stride = max((p + 15) & ~15, V * L * CPL);          // of theta and of the sums in shared memory (rows of up to 7 floats: 16)
    lds_f32* th = (lds_f32*)smem;                    // [2][stride]: theta, by version parity
    lds_f32* sums = th + 2 * stride;                 // [RW][stride]: each row wavefront's gradient sums of a step
    lds_f32* xstate = sums + RW * stride;            // scratch of the exchange wavefronts
    const int first = a.s_begin, last = a.s_end;

    // theta (version 0 in copy 0) and the sums; positions beyond the row stay zero for good (rows are read at column 0 there)
    load_theta<narrow_block(RW), V == 4 ? 256 * CPL : 16>(a, th, stride, (2 + RW) * stride, tid);
    if (tid == 0) { s_abort = 0; s_theta_version = 0u; s_published = 0u; s_sent = 0u; s_xconsumed = 0u; }
    if (tid < kXWaves) s_xarrived[tid] = 0u;
    __syncthreads();                                 // the only barrier: from here on the wavefronts meet through flags

    const int rw = wave - kXWaves;
    if (rw >= 0) {
        // ------------------------------------------------------------------------------------ row wavefronts
        const StepGeometry geo(a);
        const int lsub = lane & (L - 1);
        const int slot = lane >> a.logL;
        const int rpw = 64 >> a.logL;                // rows side by side in a wavefront
        const int S_total = G * RW * rpw;    // row slots of the grid: row j of a mini-batch goes to slot j mod S_total
        const int myslot = (g * RW + rw) * rpw + slot;
        int col[CPL], from[CPL];                     // positions of this lane's vectors, and where in a row they are loaded from
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            col[k] = V * (lsub + L * k);
            from[k] = V == 4 ? vector_from(a, col[k]) : col[k] < p ? col[k] : 0;
        }

        // A group: the rows of one step.  Besides the rows it carries their responses and the indices of the rows
        // that take their place at the group's next request; both are loaded right behind the rows, so they have
        // arrived when the rows have (loads return in order) and waiting for them waits for nothing else.
        struct Group {
            float x[PF][E];
            float y[PF];
            int idx_next[PF];
            unsigned ok, ok_next;                    // bit q: row q exists
            int sq;                                  // the step whose row indices are loaded next
        };
        auto load_idx = [&](Group& S) {
            const bool live = S.sq < last;
            const int sc = live ? S.sq : first;      // beyond the end: the first step's rows again (valid addresses, not used)
            const int nb = geo.batch_rows(sc);
            const size_t base = geo.batch_base(sc);
            S.ok_next = 0u;
#pragma unroll
            for (int q = 0; q < PF; ++q) {
                const int j = q * S_total + myslot;
                const bool ok = live && j < nb;
                S.idx_next[q] = a.perm[base + (size_t)(ok ? j : 0)];
                S.ok_next |= ok ? (1u << q) : 0u;
            }
            S.sq += 2;
        };
        auto request = [&](Group& S) {
#pragma unroll
            for (int q = 0; q < PF; ++q) {
                const float* row = a.X + (size_t)S.idx_next[q] * (size_t)p;
#pragma unroll
                for (int k = 0; k < CPL; ++k) load_vec_unaligned<V>(row + from[k], &S.x[q][k * V]);
            }
#pragma unroll
            for (int q = 0; q < PF; ++q) S.y[q] = a.y[S.idx_next[q]];
            S.ok = S.ok_next;
            load_idx(S);
        };
        auto keep = [&](const Group& S) {
#pragma unroll
            for (int q = 0; q < PF; ++q) {
#pragma unroll
                for (int e = 0; e < E; ++e) asm volatile("" :: "v"(S.x[q][e]));
                asm volatile("" :: "v"(S.y[q]), "v"(S.idx_next[q]));
            }
        };
        Group A, B;
        A.sq = first; B.sq = first + 1;
        load_idx(A); load_idx(B);
        request(A); request(B);

        const unsigned abort_addr = (unsigned)(uintptr_t)(lds_u32*)&s_abort;
        const unsigned version_addr = (unsigned)(uintptr_t)(lds_u32*)&s_theta_version;
        const bool gated = kGated && (!ONE || G > 1);
        const unsigned sent_addr = (unsigned)(uintptr_t)(lds_u32*)&s_sent;
        lds_f32* my_sums = sums + rw * stride;
        // Step s on the rows in S, then S is refilled.  Straight-line code with one conditional (the publication).  A
        // step past the end uses rows requested beyond the end, publishes nothing and waits for the last version only.
        auto process = [&](Group& S, int s) {
            const bool live = s < last;
            const unsigned want = (unsigned)(min(s, last) - first);
            lds_wait_ge(version_addr, want * kXWaves, abort_addr);   // (every exchange wavefront raises it once per version)
            const lds_f32* src = th + (want & 1u) * stride;
            float thr[E], acc[E], dot[PF], r[PF];
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
#pragma unroll
                for (int v = 0; v < V; ++v) thr[k * V + v] = src[col[k] + v];
            }
#pragma unroll
            for (int q = 0; q < PF; ++q) {
                dot[q] = S.x[q][0] * thr[0];
#pragma unroll
                for (int e = 1; e < E; ++e) dot[q] = fmaf(S.x[q][e], thr[e], dot[q]);
            }
            // (no loads inside: the branches do not disturb their count)
            if (CPL > 1 || L == 64) {
#pragma unroll
                for (int q = 0; q < PF; ++q) dot[q] = group_sum(dot[q], 64);
            } else if (L == 32) {
#pragma unroll
                for (int q = 0; q < PF; ++q) dot[q] = group_sum(dot[q], 32);
            } else {
#pragma unroll
                for (int q = 0; q < PF; ++q) dot[q] = row_group_sum(dot[q], L);
            }
            // Residuals: lane l of four works out those of the rows q = l mod 4 and hands them to the others (exp and a division cost
            // more than the products of a row, and every lane of the group would make the same).
            constexpr int Q = PF < 3 ? PF : 4;
            auto residuals_from = [&](auto from) {
                constexpr int q0 = decltype(from)::value;
                const int mine = lane & (Q - 1);
                const float u = Q == 1 ? dot[q0] : Q == 2 ? pick2(mine, dot[q0], dot[q0 + Q - 1]) : pick4(mine, dot[q0], dot[q0 + Q / 4], dot[q0 + Q / 2], dot[PF == 3 ? 2 : q0 + Q - 1]);
                const float yq = Q == 1 ? S.y[q0] : Q == 2 ? pick2(mine, S.y[q0], S.y[q0 + Q - 1]) : pick4(mine, S.y[q0], S.y[q0 + Q / 4], S.y[q0 + Q / 2], S.y[PF == 3 ? 2 : q0 + Q - 1]);
                const float res = ((S.ok >> (q0 + mine)) & 1u) != 0u ? residual(a.model, u, yq) : 0.f;
                if constexpr (Q == 1) r[q0] = res;
                if constexpr (Q >= 2) { r[q0] = dpp_mov<0x00>(res); r[q0 + 1] = dpp_mov<0x55>(res); }
                if constexpr (Q == 4) r[q0 + 2] = dpp_mov<0xAA>(res);
                if constexpr (Q == 4 && PF != 3) r[q0 + 3] = dpp_mov<0xFF>(res);
            };
            residuals_from(std::integral_constant<int, 0>{});
            if constexpr (PF == 8) residuals_from(std::integral_constant<int, 4>{});
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = r[0] * S.x[0][e];
#pragma unroll
            for (int q = 1; q < PF; ++q) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = fmaf(r[q], S.x[q][e], acc[e]);
            }
            if (CPL == 1 && L == 32) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = swap32_sum(acc[e]);
            } else if (CPL == 1 && L < 32) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = slot_sum_flat(acc[e], L);
            }                                        // lanes < L: the wavefront's sums
            if (live) {
                if (lane < L) {
#pragma unroll
                    for (int k = 0; k < CPL; ++k)
                        if (col[k] < (V == 4 ? width : p)) {
#pragma unroll
                            for (int v = 0; v < V; ++v) my_sums[col[k] + v] = acc[k * V + v];
                        }
                }
                // (shared memory serves a wavefront's requests in order: the count is raised after the sums are in place;
                // a release here would wait for the rows in flight as well)
                asm volatile("" ::: "memory");
                if (lane == 0) lds_add_one(lds_address((lds_u32*)&s_published));
            }
            // What the exchange sends and asks for first would stand behind these requests in the unit's memory pipeline; they go out while
            // its words are under way.
            if constexpr (kGated) lds_wait_ge(sent_addr, gated ? (unsigned)(min(s + 1, last) - first) * kXWaves : 0u, abort_addr);
            request(S);
        };
        int su = first;
#pragma clang loop unroll(disable)
        do {
            process(A, su);
            process(B, su + 1);
            su += 2;
        } while (su < last && __hip_atomic_load(&s_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0);
        // What was requested beyond the last step is still in flight.  It is named here as if it were needed, so that
        // the last requests stay where they are in the loop: moved behind the loop's exit test (they are dead when
        // the loop ends), their results would reach the registers of the next trip through copies, and a copy waits
        // for its load.
        keep(A); keep(B);
        return;
    }

    // ------------------------------------------------------------------------------------ exchange wavefronts
    __builtin_amdgcn_s_setprio(3);                   // (they share their SIMDs with row wavefronts that are requesting rows)
    const ExchangeLds x{th, stride, xstate, xstate + kExchangeState * kXWaves, sums, stride, (unsigned)RW,
                        (lds_u32*)&s_published, (lds_u32*)&s_theta_version, (lds_i32*)&s_abort, (lds_u32*)&s_sent,
                        (lds_u32*)s_xarrived, (lds_u32*)&s_xconsumed};
    if constexpr (ONE) exchange_one_trip<OPT, kXWaves, RW, kGated, EX>(a, x, lane, wave);
    else if constexpr (EX == kByDie) exchange_by_die<OPT, kXWaves, RW, 1, 2>(a, x, lane, wave);   // (p <= 1024: two loads per lane collect theta ...
    else exchange_wavefront<OPT, kXWaves, RW, kGated, 8, 2>(a, x, lane, wave);   // ... and eight cover the slice for up to 256 workgroups)
}

using KernelFn = void (*)(ExchangeArgs);

template <bool OPT, int RW, int EX, int V, int CPL, int PF>
KernelFn pick()
{
    // (one trip: up to 8 EX columns; rows of fewer than eight floats have two or eight pairs)
    constexpr bool fits = EX < 2 ? V == 4 : RW > kRowWaves && (EX == 64 ? V == 4 && CPL == 2 : CPL == 1 && (EX == 2 || EX == 8 || V == 4));
    if constexpr (!narrow_shape_ok(V, CPL, PF, RW) || !fits) return nullptr;
    else return glm_narrow_kernel<V, CPL, PF, RW, EX, OPT>;
}

template <bool OPT, int RW, int EX, int V, int CPL>
KernelFn pick_pf(int pf)
{
    switch (pf) {
    case 1: return pick<OPT, RW, EX, V, CPL, 1>();
    case 2: return pick<OPT, RW, EX, V, CPL, 2>();
    case 3: return pick<OPT, RW, EX, V, CPL, 3>();
    case 4: return pick<OPT, RW, EX, V, CPL, 4>();
    case 8: return pick<OPT, RW, EX, V, CPL, 8>();
    }
    return nullptr;
}

template <bool OPT, int RW, int EX>
KernelFn pick_row(int v, int cpl, int pf)
{
    if (v == 4) return cpl == 1 ? pick_pf<OPT, RW, EX, 4, 1>(pf) : cpl == 2 ? pick_pf<OPT, RW, EX, 4, 2>(pf) : pick_pf<OPT, RW, EX, 4, 4>(pf);
    if (v == 2) return pick_pf<OPT, RW, EX, 2, 1>(pf);
    return pick_pf<OPT, RW, EX, 1, 1>(pf);
}

template <bool OPT, int RW>
KernelFn pick_sliced(const GlmLaunchShape& s, int ex)
{
    const NarrowLayout& l = s.narrow_layout;
    if (ex == kByDie) return pick_row<OPT, RW, kByDie>(l.V, l.CPL, s.narrow_pf);
    return pick_row<OPT, RW, kTwoTrips>(l.V, l.CPL, s.narrow_pf);
}

template <bool OPT>
KernelFn narrow_kernel_opt(const GlmLaunchShape& s, int ex)
{
    const NarrowLayout& l = s.narrow_layout;
    if (s.reduce_mode == kReduceSliced) return s.narrow_rw == kRowWaves ? pick_sliced<OPT, kRowWaves>(s, ex) : pick_sliced<OPT, kNarrowMoreRows>(s, ex);
    if (l.width > 256) return pick_row<OPT, kNarrowMoreRows, 64>(l.V, l.CPL, s.narrow_pf);
    if (l.width > 128) return pick_row<OPT, kNarrowMoreRows, 32>(l.V, l.CPL, s.narrow_pf);
    if (l.width > 64) return pick_row<OPT, kNarrowMoreRows, 16>(l.V, l.CPL, s.narrow_pf);
    // Few columns, by more than 64 workgroups: as few pairs a wavefront as give all four some, so that a lane asks for eight workgroups' words at most.  us per
    // update with eight pairs a wavefront / so: 3.15 / 2.4 at p = 16 on 100, 3.2 / 2.3 at p = 30 on 100; but 2.1 / 2.3 and 2.15 / 2.35 on 32, 2.45 / 2.6 at p = 16 on 64.  (With state
    // and eight words a lane four pairs: 3.9 against 4.2 to 4.6 with two at p = 16 on 129 to 255.)
    if (l.width > 32 || s.G <= 64) return pick_row<OPT, kNarrowMoreRows, 8>(l.V, l.CPL, s.narrow_pf);
    if (l.width > 16 || (OPT && l.width > 8 && s.G > 128)) return pick_row<OPT, kNarrowMoreRows, 4>(l.V, l.CPL, s.narrow_pf);
    return pick_row<OPT, kNarrowMoreRows, 2>(l.V, l.CPL, s.narrow_pf);
}

// ex: of the sliced reduction, which of its exchanges
KernelFn narrow_kernel(const GlmLaunchShape& s, int ex) { return s.with_optimizer ? narrow_kernel_opt<true>(s, ex) : narrow_kernel_opt<false>(s, ex); }
int sliced_exchange(const GlmLaunchShape& s) { return glm_narrow_by_die(s.p, s.G) ? kByDie : kTwoTrips; }

size_t narrow_lds_bytes(const GlmLaunchShape& s, int p)
{
    const int stride = std::max((p + 15) & ~15, s.narrow_layout.V * s.narrow_layout.L * s.narrow_layout.CPL);
    return (size_t)((2 + s.narrow_rw) * stride + (kExchangeState + kExchangeRed) * kXWaves + 16) * sizeof(float);
}

}  // namespace

int glm_narrow_block(int rw) { return narrow_block(rw); }

bool glm_narrow_by_die(int64_t p, int G) { return glm_by_die(p, G, kXWaves); }

NarrowLayout glm_narrow_layout(int64_t p)
{
    NarrowLayout l;
    // Vectors of four (of what shorter rows are a multiple of where four would leave most lanes idle)
    l.V = p >= 8 || p % 4 == 0 ? 4 : p % 2 == 0 ? 2 : 1;
    const int64_t vectors = (p + l.V - 1) / l.V;
    l.L = 4;                                         // (the kernel's lanes work out residuals in fours)
    while (l.L < vectors && l.L < 64) l.L *= 2;
    l.CPL = 1;
    while (l.CPL * 64 < vectors) l.CPL *= 2;
    l.width = (int)(l.V == 1 ? (p + 1) / 2 * 2 : vectors * l.V);
    return l;
}

int glm_narrow_rows_in_flight(const NarrowLayout& l, int rw, int G, int64_t n)
{
    const int64_t slots = (int64_t)G * rw * (64 / l.L);
    const int64_t need = (n + slots - 1) / slots;
    const int pf = need <= 4 ? (int)need : need <= 8 ? 8 : 16;
    return narrow_shape_ok(l.V, l.CPL, pf, rw) ? pf : 0;
}

hipError_t glm_narrow_prepare(const GlmLaunchShape& s, int p, int* max_groups)
{
    const size_t lds = narrow_lds_bytes(s, p);
    KernelFn fn = narrow_kernel(s, sliced_exchange(s));
    if (!fn) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), narrow_block(s.narrow_rw), lds);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    *max_groups = per_cu * cus;
    return hipSuccess;
}

hipError_t glm_narrow_launch(const GlmLaunchShape& s, const GlmArgs& args, hipStream_t stream, hipEvent_t stop)
{
    KernelFn fn = narrow_kernel(s, sliced_exchange(s));
    const NarrowLayout& l = s.narrow_layout;
    const int64_t slots = (int64_t)s.G * s.narrow_rw * (64 / l.L);
    const bool one_trip = s.reduce_mode == kReduceRedundant;
    // what the kernel assumes: a row in the lanes' vectors, every row of a step in a register slot; two trips: slices of whole groups of
    // eight workgroups; one trip: columns that the exchange wavefronts hold as pairs
    if (!fn || args.s_begin >= args.s_end || args.reduce_mode != s.reduce_mode || args.p != s.p ||
        l.width > l.V * l.L * l.CPL + (l.V == 1) || (int64_t)args.n > slots * s.narrow_pf)
        return hipErrorInvalidValue;
    if (one_trip ? s.narrow_rw == kRowWaves || args.p > kNarrowOneTripMaxP || s.G < 1
                 : s.G < 8 || s.G % 8 != 0 || l.V != 4)
        return hipErrorInvalidValue;
    ExchangeArgs a = exchange_args(args, s.far);
    a.L = l.L;
    a.logL = 0;
    while ((1 << a.logL) < a.L) ++a.logL;
    a.width = l.width;
    a.shift = l.V == 4 ? l.width - args.p : 0;
    hipExtLaunchKernelGGL(fn, dim3(s.G), dim3(narrow_block(s.narrow_rw)), (uint32_t)narrow_lds_bytes(s, args.p), stream, nullptr, stop, 0u, a);
    return hipGetLastError();
}

}  // namespace bmgd
