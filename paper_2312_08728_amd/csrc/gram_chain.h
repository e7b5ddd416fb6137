// The chain of eq. (3.1) steps in one workgroup, for the kernel that runs it alone (gram_kernels.hip) and the one that forms the moment
// matrices first (gram_fused_kernel.hip).
#pragma once

#include "bmgd_internal.h"
#include "gram_layout.h"

namespace bmgd {
namespace {

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// The chain: one workgroup of L.nthr threads, theta in LDS (two copies, alternating), the matrices of the coming AHEAD steps
// already in registers.  Thread (i, seg) = (t / TPR, t % TPR); the TPR lanes of a row add up their parts.
// RULE: plain steps, momentum / NAG, or Adam: separate instantiations, none carries anything of the others.  What a rule adds
// sits on the step's critical path, so nothing of it is decided or read late: us per step at p = 37 for NAG 0.31 -> 0.23, for
// Adam 2.2 -> 0.37 (p = 100: 0.57 -> 0.53 and 2.4 -> 0.70), against one instantiation for all rules.
enum { kRulePlain = 0, kRuleMomentum = 1, kRuleAdam = 2 };
constexpr int kCorrSteps = 64;                    // steps whose bias corrections are formed together

// RATE: the learning rate of a step is alpha, an entry of a table in memory, or rates[step] in shared memory.
enum { kRateConstant = 0, kRateTable = 1, kRateShared = 2 };

template <int TPR, int KQ, int KS, int AHEAD, int RATE, int RULE>
__device__ __forceinline__ void gram_chain_steps(const float* __restrict__ gram, float* __restrict__ theta, const GramLayout& L, int nsteps,
                                                 int period, float alpha, const float* __restrict__ lr_tab, int lr_base, int lr_len,
                                                 const float* rates, const OptArgs& opt)
{
    constexpr bool TAB = RATE == kRateTable;
    __shared__ __align__(16) float th[2][kGramMaxP + 4 * 16];
    __shared__ float2 corr[2][RULE == kRuleAdam ? kCorrSteps : 1];
    const int t = threadIdx.x;
    const int i = t / TPR, seg = t % TPR;
    const int p = L.p;
    const bool row_ok = i < p;
    constexpr int NQ = KQ > 0 ? KQ : 1, NS = KS > 0 ? KS : 1;
    float4 sq[AHEAD][NQ];
    float ss[AHEAD][NS];
    float bb[AHEAD];
    float aa[AHEAD];                                  // learning rate of the step, from the optional table
    const int ib = row_ok ? i : 0;
    int fidx = 0;                                     // matrices to request next; wraps when passes share one partition
    // Addresses are a buffer at the matrices of a step (scalar registers), a per-thread byte offset that never changes and a scalar one per
    // load: a request is five scalar and no vector instructions besides its loads.  (They stand between a step's products and the
    // next: as 64-bit vector additions they were a third of a step of 37 features.)
    const unsigned off16 = (unsigned)t * 16u, off4 = (unsigned)t * 4u, offb = (unsigned)ib * 4u;
    const unsigned step_bytes = (unsigned)L.step_floats * 4u, plane = (unsigned)L.nthr * 4u, b_bytes = (unsigned)L.b_off * 4u;
    const char* g_next = reinterpret_cast<const char*>(gram);
    // TAB: the learning rate of a step comes from lr_tab (requested with the step's matrices), else it is alpha.
    const int lr_last = lr_len - 1;
    int lr_next = lr_base;
    auto fetch = [&](float4 (&q)[NQ], float (&sc)[NS], float& bv, float& av) {
        const __amdgpu_buffer_rsrc_t g = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(g_next), 0, (int)step_bytes, 0x00020000);
        const bool wrap = ++fidx == period;
        fidx = wrap ? 0 : fidx;
        g_next = wrap ? reinterpret_cast<const char*>(gram) : g_next + step_bytes;
#pragma unroll
        for (int k = 0; k < KQ; ++k)
            q[k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(g, off16, (unsigned)k * 4u * plane, 0));
#pragma unroll
        for (int j = 0; j < KS; ++j)
            sc[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(g, off4, (unsigned)(4 * KQ + j) * plane, 0));
        bv = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(g, offb, b_bytes, 0));
        if constexpr (TAB) {
            av = lr_tab[min(lr_next, lr_last)];
            lr_next += 1;
        }
    };
#pragma unroll
    for (int d = 0; d + 1 < AHEAD; ++d) fetch(sq[d], ss[d], bb[d], aa[d]);
    for (int c = t; c < kGramMaxP + 64; c += L.nthr) { th[0][c] = c < p ? theta[c] : 0.f; th[1][c] = 0.f; }
    // optimizer state of coordinate i lives in the registers of the lane that updates it
    const bool owner = seg == 0 && row_ok;
    float om = 0.f, os = 0.f;
    if (RULE != kRulePlain && owner) {
        om = opt.m[i];
        if (RULE == kRuleAdam) os = opt.s[i];
    }
    // The compiler is free to reorder these first requests; with all of them landed before the loop, the waits
    // it places inside the loop count only the requests of the loop itself, which are issued oldest slot first.  (The state as well: requested
    // behind the wait, its first use made every AHEAD-th step wait for all matrices under way, 0.23 us per step instead of 0.13 at p = 37.)
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
    __syncthreads();

    // Steps are taken AHEAD at a time without any branch around the loads (a branch would make the compiler
    // wait for every outstanding load); steps past the last one run with a zero learning rate.
    // Adam's bias corrections do not depend on theta: a wavefront forms those of kCorrSteps steps at once, one block ahead of
    // their use (two powers in every step, on its critical path, took 0.8 to 2 us of it)
    auto corrections = [&](int block) {
        if constexpr (RULE == kRuleAdam) {
            if (t < kCorrSteps) {
                float c1, c2;
                opt_corrections(opt, opt.k_base + block * kCorrSteps + t + 1, c1, c2);
                corr[block & 1][t] = make_float2(c1, c2);
            }
        }
    };
    if constexpr (RULE == kRuleAdam) {
        corrections(0);
        __syncthreads();
    }
    const float nag = RULE == kRuleMomentum && opt.kind == kOptNag ? opt.mu : 0.f;
    const bool is_nag = RULE == kRuleMomentum && opt.kind == kOptNag;
    int cur = 0;
    for (int sb = 0; sb < nsteps; sb += AHEAD) {
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) {
            const int step = sb + d;
            // (rates in shared memory are zero beyond the last step: no branch)
            const float a_eff = RATE == kRateShared ? rates[step] : step < nsteps ? (RATE == kRateTable ? aa[d] : alpha) : 0.f;
            // (steps come in order: the block after this one is formed at this one's first step, barriers away from its use)
            if (RULE == kRuleAdam && step % kCorrSteps == 0) corrections(step / kCorrSteps + 1);
            // theta first (its way from shared memory takes longer than the requests that follow)
            float4 tq[NQ];
            float ts[NS];
#pragma unroll
            for (int k = 0; k < KQ; ++k) tq[k] = *reinterpret_cast<const float4*>(&th[cur][4 * (seg + TPR * k)]);
#pragma unroll
            for (int j = 0; j < KS; ++j) ts[j] = th[cur][4 * TPR * KQ + TPR * j + seg];
            __builtin_amdgcn_sched_barrier(0);
            // Request step s + AHEAD - 1 into the ring slot the previous step has just used up, before this step's
            // arithmetic: the memory pipeline works on the requests of all wavefronts while they compute.
            const int prev = (d + AHEAD - 1) % AHEAD;
            fetch(sq[prev], ss[prev], bb[prev], aa[prev]);
            float dot0 = 0.f, dot1 = 0.f;
#pragma unroll
            for (int k = 0; k < KQ; ++k) {
                dot0 = fmaf(sq[d][k].x, tq[k].x, dot0);
                dot1 = fmaf(sq[d][k].y, tq[k].y, dot1);
                dot0 = fmaf(sq[d][k].z, tq[k].z, dot0);
                dot1 = fmaf(sq[d][k].w, tq[k].w, dot1);
            }
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                if (j & 1) dot1 = fmaf(ss[d][j], ts[j], dot1); else dot0 = fmaf(ss[d][j], ts[j], dot0);
            }
            float dot = dot0 + dot1;
            float own = th[cur][ib];                 // (read ahead of the sums below: the compiler would move it into the owner's branch)
            // Everything of the update that does not hang on the products: theta' = base - gain (S theta).  Momentum and NAG written out
            // in their old state: v' = mu v - a (S theta - b), theta' = theta + v' or theta + mu v' - a (S theta - b).
            float base = fmaf(a_eff, bb[d], own), gain = a_eff, kept = 0.f;
            if constexpr (RULE == kRuleMomentum) {
                kept = fmaf(opt.mu, om, a_eff * bb[d]);           // v' + a S theta
                gain = fmaf(nag, a_eff, a_eff);                   // nag: mu for NAG, 0 for momentum
                base = own + (is_nag ? fmaf(opt.mu, kept, a_eff * bb[d]) : kept);
            }
            float2 c = make_float2(1.f, 1.f);
            if constexpr (RULE == kRuleAdam) c = corr[(step / kCorrSteps) & 1][step % kCorrSteps];
            asm volatile("" : "+v"(own), "+v"(base), "+v"(kept));
            if (TPR >= 2) dot += dpp_mov<0xB1>(dot);      // lanes ^1
            if (TPR >= 4) dot += dpp_mov<0x4E>(dot);      // lanes ^2
            if (TPR >= 8) dot += dpp_mov<0x141>(dot);     // mirror within 8
            if (TPR >= 16) dot += dpp_mov<0x140>(dot);    // mirror within 16
            // (steps past the last one leave theta and the state alone)
            if constexpr (RULE != kRuleAdam) {
                const bool active = RULE == kRulePlain || step < nsteps;
                if (owner) th[cur ^ 1][i] = active ? fmaf(-gain, dot, base) : own;
                if constexpr (RULE == kRuleMomentum) om = active ? fmaf(-a_eff, dot, kept) : om;
            } else {
                const bool active = step < nsteps;
                float nm = om, ns = os;
                const float nv = opt_update(opt, own, dot - bb[d], a_eff, nm, ns, c.x, c.y);
                om = active ? nm : om;
                os = active ? ns : os;
                if (owner) th[cur ^ 1][i] = active ? nv : own;
            }
            __syncthreads();
            cur ^= 1;
        }
    }
    for (int c = t; c < p; c += L.nthr) theta[c] = th[cur][c];
    if (RULE != kRulePlain && owner) {
        opt.m[i] = om;
        if (RULE == kRuleAdam) opt.s[i] = os;
    }
}

}  // namespace
}  // namespace bmgd
