// Least squares with few features: the steps of a launch multiplied together instead of applied one by one.
//
// A step of eq. (3.1) is an affine map, theta <- (I - alpha_s Sxx_s) theta + alpha_s Sxy_s, which in homogeneous
// coordinates is the (p + 1) x (p + 1) matrix A_s = [[I - alpha_s Sxx_s, alpha_s Sxy_s], [0, 1]].  None of the A_s
// depends on theta, so the estimate after the N steps of a launch is [theta; 1] <- A_{N-1} ... A_1 A_0 [theta; 1]
// (the products of eq. (3.2)), and the product can be formed as a tree: N / 2 independent products of neighbours, then
// N / 4, ... -- log2 N launches of small dense products on the matrix cores (fp32 in, fp32 accumulate) in place of a
// chain of N dependent steps in one workgroup.  Same arithmetic as the chain up to the order of the fp32 operations;
// intermediate estimates are not formed.
#include "bmgd_internal.h"
#include "glm_device.h"
#include "gram_layout.h"

#include <hip/hip_ext.h>

#include <algorithm>

namespace bmgd {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct FirstLevel {                                  // where the steps' moment matrices are, and their learning rates
    const float* dense;                              // per mini-batch [Sxx | -Sxy], dense of order Q (gram_launch_moments, dense)
    int p;
    int period;                                      // step s uses matrix s % period
    float alpha;
    const float* lr_tab;                             // optional: step s uses lr_tab[min(lr_base + s, lr_len - 1)]
    int lr_base, lr_len;
};

constexpr int kMaxOrder = (kGramMaxP + 1 + 15) / 16 * 16;                       // 144
constexpr int pair_waves(int nt) { return (nt + 1) / 2; }                      // of a workgroup: half of a product's tile rows
constexpr size_t pair_lds(int nt) { return sizeof(float) * (size_t)(16 * nt) * (16 * nt + 4); }

// out[j] = in[2 j + 1] * in[2 j] (the later step on the left); a missing in[2 j + 1] counts as the identity.  Dense
// Q x Q matrices, row-major, Q = 16 NT.  Two workgroups a product, a wavefront to each 16-row tile row of it: the right factor stands in
// shared memory, where every wavefront reads it; a wavefront's rows of the left factor go straight from memory to the operands of
// its matrix instructions, 16 bytes a lane.  For that the sum over k takes in step q of a block of 16 the k = 4 (lane / 16) + q, in both
// operands.  The instruction (v_mfma_f32_16x16x4_f32: a = A[lane % 16][lane / 16], b = B[lane / 16][lane % 16], c[v] = C[4 (lane / 16) + v][lane % 16])
// forms the product's transpose, so that a lane ends with four neighbouring columns of a row and stores 16 bytes.  Row stride Q + 4 of the right
// factor: the eight or 32 lanes that are served together meet no bank twice.
// What bounds it is a trip to memory for what the kernel before wrote (6 us with the launch, 50 KB a product and workgroup at Q = 112), the
// matrix instructions (28 for each of a wavefront's seven tiles, 2.8 us) and the way out, one after the other in a workgroup and little more than
// one workgroup to a unit.  150 products of order 112: 17.3 us (19.1 under a profiler); four workgroups a product that staged 32 rows of the left factor too, with
// the loads of the largest order whatever the order was and stores of 4 bytes, 24.4.
// FIRST: the factors are the steps themselves, A_s = [[I - alpha_s Sxx_s, alpha_s Sxy_s], [0, 1]] padded with zeros:
// entry (r, c) is (r == c and r <= p) - alpha_s D_s(r, c) with D_s the dense matrix the moments kernel wrote.
// CHAIN_OUT: the product P goes out as [I - P | last column of P] in the layout the chain kernel reads (GramLayout), so
// that the chain's step theta - 1 * ((I - P) theta - d) applies it.
template <int NT, bool FIRST, bool CHAIN_OUT>
__global__ void __launch_bounds__(64 * pair_waves(NT)) affine_pair_kernel(FirstLevel f, const float* __restrict__ in, float* __restrict__ out,
                                                                         int count_in, GramLayout L)
{
    extern __shared__ __align__(16) float Rs[];      // right factor
    constexpr int Q = 16 * NT, QV = Q / 4, rs = Q + 4, threads = 64 * pair_waves(NT);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int j = blockIdx.y;
    const int tr = pair_waves(NT) * blockIdx.x + wave;           // this wavefront's tile row (NT, where it has none)
    const int right = 2 * j, left = 2 * j + 1;
    const bool has_left = left < count_in;
    const int lc = has_left ? left : right;          // (clamped: not used when the left factor is the identity)

    const float* Rm;
    const float* Lm;
    float a_r = 0.f, a_l = 0.f;
    if constexpr (FIRST) {
        Rm = f.dense + (size_t)(right % f.period) * Q * Q;
        Lm = f.dense + (size_t)(lc % f.period) * Q * Q;
        a_r = f.lr_tab ? f.lr_tab[min(f.lr_base + right, f.lr_len - 1)] : f.alpha;
        a_l = f.lr_tab ? f.lr_tab[min(f.lr_base + lc, f.lr_len - 1)] : f.alpha;
    } else {
        Rm = in + (size_t)right * Q * Q;
        Lm = in + (size_t)lc * Q * Q;
    }
    constexpr int nR = Q * QV, kRight = (nR + threads - 1) / threads;
    float4 rv[kRight], lv[NT];
    const int lrow = 16 * min(tr, NT - 1) + l16;
#pragma unroll
    for (int i = 0; i < kRight; ++i) rv[i] = *reinterpret_cast<const float4*>(Rm + 4 * min(tid + threads * i, nR - 1));
#pragma unroll
    for (int i = 0; i < NT; ++i) lv[i] = *reinterpret_cast<const float4*>(Lm + (size_t)lrow * Q + 16 * i + 4 * lq);
    // entry (r, c .. c + 3) of a factor from what was loaded for it
    auto entry = [&](float4 v, float alpha, int r, int c) {
        if constexpr (FIRST) {
            const bool in_map = r <= f.p;
            v.x = (in_map && r == c ? 1.f : 0.f) - alpha * v.x;
            v.y = (in_map && r == c + 1 ? 1.f : 0.f) - alpha * v.y;
            v.z = (in_map && r == c + 2 ? 1.f : 0.f) - alpha * v.z;
            v.w = (in_map && r == c + 3 ? 1.f : 0.f) - alpha * v.w;
        }
        return v;
    };
#pragma unroll
    for (int i = 0; i < kRight; ++i) {
        const int e = tid + threads * i;
        if (e < nR) {
            const int r = e / QV, c = 4 * (e - r * QV);
            float4 v = entry(rv[i], a_r, r, c);
            float* to = Rs + r * rs + c;
            if constexpr (FIRST) {
                // A step but for its last row and column is symmetric.  What stands here is its transpose: row p holds column p, and
                // column p row p (zeros and a one).
                const int e4 = f.p - c;              // column p is the e4-th of these four
                if (r == f.p) {
                    if (e4 <= 0) to[0] = v.x;
                    if (e4 <= 1) to[1] = v.y;
                    if (e4 <= 2) to[2] = v.z;
                    if (e4 <= 3) to[3] = v.w;
                    continue;
                }
                if (r < f.p && (unsigned)e4 < 4u) {
                    Rs[f.p * rs + r] = e4 == 0 ? v.x : e4 == 1 ? v.y : e4 == 2 ? v.z : v.w;
                    if (e4 == 0) v.x = 0.f;
                    if (e4 == 1) v.y = 0.f;
                    if (e4 == 2) v.z = 0.f;
                    if (e4 == 3) v.w = 0.f;
                }
            }
            *reinterpret_cast<float4*>(to) = v;
        }
    }
    __syncthreads();
    if (tr >= NT) return;

    floatx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const float* bp = FIRST ? Rs + l16 * rs + 4 * lq : Rs + 4 * lq * rs + l16;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int c = 16 * i + 4 * lq;
        const float4 v = has_left ? entry(lv[i], a_l, lrow, c)
                                  : make_float4(lrow == c ? 1.f : 0.f, lrow == c + 1 ? 1.f : 0.f, lrow == c + 2 ? 1.f : 0.f, lrow == c + 3 ? 1.f : 0.f);
        const float a[4] = {v.x, v.y, v.z, v.w};
        float4 b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if constexpr (FIRST) b[t] = *reinterpret_cast<const float4*>(bp + 16 * t * rs + 16 * i);
            else b[t] = make_float4(bp[16 * i * rs + 16 * t], bp[(16 * i + 1) * rs + 16 * t], bp[(16 * i + 2) * rs + 16 * t], bp[(16 * i + 3) * rs + 16 * t]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(q == 0 ? b[t].x : q == 1 ? b[t].y : q == 2 ? b[t].z : b[t].w, a[q], acc[t], 0, 0, 0);
    }
    // lane: row r, columns 16 t + 4 lq .. + 3
    float* o = out + (size_t)j * (CHAIN_OUT ? (size_t)L.step_floats : (size_t)Q * Q);
    const int r = 16 * tr + l16;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int c = 16 * t + 4 * lq;
        if constexpr (CHAIN_OUT) {
            if (r >= L.p) continue;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = c + i == L.p ? acc[t][i] : (r == c + i ? 1.f : 0.f) - acc[t][i];
            if (c + 3 < 4 * L.tpr * L.kq) {          // whole vectors of the chain's layout
                *reinterpret_cast<float4*>(o + gram_pos(L, r, c)) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c + i <= L.p) o[c + i == L.p ? L.b_off + r : gram_pos(L, r, c + i)] = v[i];
            }
        } else {
            *reinterpret_cast<float4*>(o + (size_t)r * Q + c) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
        }
    }
}

typedef void (*PairKernel)(FirstLevel, const float*, float*, int, GramLayout);
template <bool FIRST, bool CHAIN_OUT>
PairKernel pair_kernel(int nt)
{
    static const PairKernel table[] = {affine_pair_kernel<1, FIRST, CHAIN_OUT>, affine_pair_kernel<2, FIRST, CHAIN_OUT>, affine_pair_kernel<3, FIRST, CHAIN_OUT>,
                                       affine_pair_kernel<4, FIRST, CHAIN_OUT>, affine_pair_kernel<5, FIRST, CHAIN_OUT>, affine_pair_kernel<6, FIRST, CHAIN_OUT>,
                                       affine_pair_kernel<7, FIRST, CHAIN_OUT>, affine_pair_kernel<8, FIRST, CHAIN_OUT>, affine_pair_kernel<9, FIRST, CHAIN_OUT>};
    static_assert(sizeof(table) / sizeof(table[0]) * 16 == kMaxOrder, "a kernel for every order");
    return table[nt - 1];
}

// theta <- P[0 .. p) [theta; 1]: one workgroup; wavefront w takes rows w, w + 4, ..., its lanes the columns (all of a
// wavefront's rows are requested before any is summed).
__global__ void __launch_bounds__(256) affine_apply_kernel(const float* __restrict__ P, float* __restrict__ theta, int p, int Q)
{
    __shared__ float th[kMaxOrder + 64], nv[kGramMaxP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int RPW = (kGramMaxP + 3) / 4, CPL = (kMaxOrder + 63) / 64;      // rows per wavefront, columns per lane
    float v[RPW][CPL];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int k = 0; k < CPL; ++k)
            v[i][k] = P[(size_t)min(wave + 4 * i, p - 1) * Q + min(lane + 64 * k, Q - 1)];
    for (int c = tid; c < kMaxOrder + 64; c += 256) th[c] = c < p ? theta[c] : (c == p ? 1.f : 0.f);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < CPL; ++k) s = fmaf(v[i][k], th[lane + 64 * k], s);   // columns beyond p meet zeros
        s = group_sum(s, 64);                        // (lane butterflies: a shuffle through shared memory per stage and row would dominate)
        const int r = wave + 4 * i;
        if (lane == 0 && r < p) nv[r] = s;
    }
    __syncthreads();
    for (int c = tid; c < p; c += 256) theta[c] = nv[c];
}

int padded_order(int p) { return gram_dense_order(p); }

}  // namespace

size_t gram_products_scratch_floats(int64_t p, int64_t max_steps)
{
    const size_t Q = (size_t)padded_order((int)p);
    const size_t half = (size_t)(max_steps + 1) / 2, quarter = (half + 1) / 2;
    const size_t per = std::max(Q * Q, (size_t)make_layout((int)p).step_floats);       // dense, or in the chain's layout
    return (half + quarter) * per;
}

hipError_t gram_launch_apply(const float* product, float* theta, int p, hipStream_t stream, hipEvent_t start, hipEvent_t stop)
{
    if (p < 1 || p > kGramMaxP) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(affine_apply_kernel, dim3(1), dim3(256), 0u, stream, start, stop, 0u, product, theta, p, padded_order(p));
    return hipGetLastError();
}

namespace {

// what every launch of the pair kernel needs
struct PairSetup {
    int N, Q, NT;
    FirstLevel f;
};

template <bool FIRST, bool CHAIN_OUT>
hipError_t launch_pair_round(const PairSetup& s, const float* in, float* out, int count, int p, hipStream_t stream, hipEvent_t start, hipEvent_t stop)
{
    const dim3 grid(s.NT > 1 ? 2 : 1, (unsigned)((count + 1) / 2)), block(64 * pair_waves(s.NT));
    const PairKernel k = pair_kernel<FIRST, CHAIN_OUT>(s.NT);
    if (start || stop) hipExtLaunchKernelGGL(k, grid, block, (uint32_t)pair_lds(s.NT), stream, start, stop, 0u, s.f, in, out, count, make_layout(p));
    else hipLaunchKernelGGL(k, grid, block, pair_lds(s.NT), stream, s.f, in, out, count, make_layout(p));
    return hipGetLastError();
}

hipError_t pair_setup(const float* gram, int rows, int p, int n, int npass, int perm_stride, float alpha, const float* lr_tab,
                      int lr_base, int lr_len, PairSetup* out)
{
    if (p < 1 || p > kGramMaxP) return hipErrorInvalidValue;
    const int M = (rows + n - 1) / n;
    PairSetup s{};
    s.N = M * npass;
    s.Q = padded_order(p);
    s.NT = s.Q / 16;
    if (s.Q > kMaxOrder) return hipErrorInvalidValue;
    s.f.dense = gram;
    s.f.p = p;
    s.f.period = perm_stride == 0 ? M : s.N;
    s.f.alpha = alpha;
    s.f.lr_tab = lr_tab;
    s.f.lr_base = lr_base;
    s.f.lr_len = lr_len;
    *out = s;
    return hipSuccess;
}

}  // namespace

hipError_t gram_products_prepare(int64_t p)
{
    // the pair kernel stages up to 85 KB in shared memory (order 144): above the default limit of a launch for more than seven tile rows
    const int nt = padded_order((int)p) / 16;
    if (pair_lds(nt) <= 64 * 1024) return hipSuccess;
    for (const PairKernel k : {pair_kernel<true, true>(nt), pair_kernel<true, false>(nt), pair_kernel<false, false>(nt)}) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)pair_lds(nt));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t gram_launch_pairs(const float* gram, float* pairs_out, int rows, int p, int n, int npass, int perm_stride, float alpha,
                             const float* lr_tab, int lr_base, int lr_len, hipStream_t stream, hipEvent_t start, hipEvent_t stop)
{
    PairSetup s;
    hipError_t e = pair_setup(gram, rows, p, n, npass, perm_stride, alpha, lr_tab, lr_base, lr_len, &s);
    if (e != hipSuccess) return e;
    return launch_pair_round<true, true>(s, nullptr, pairs_out, s.N, p, stream, start, stop);
}

hipError_t gram_launch_products(const float* gram, float* theta, float* scratch, float* product_out, int rows, int p, int n, int npass,
                                int perm_stride, float alpha, const float* lr_tab, int lr_base, int lr_len, hipStream_t stream,
                                hipEvent_t start, hipEvent_t stop, bool pairs_then_chain)
{
    PairSetup ps;
    {
        hipError_t e0 = pair_setup(gram, rows, p, n, npass, perm_stride, alpha, lr_tab, lr_base, lr_len, &ps);
        if (e0 != hipSuccess) return e0;
    }
    const int N = ps.N, Q = ps.Q;
    if (pairs_then_chain) {
        // one round of products into the chain's layout, then the chain over half as many steps, each applied with rate 1
        hipError_t e = gram_launch_pairs(gram, scratch, rows, p, n, npass, perm_stride, alpha, lr_tab, lr_base, lr_len, stream, start,
                                         nullptr);
        if (e != hipSuccess) return e;
        OptArgs none{};
        none.kind = kOptSgd;
        const int half = (N + 1) / 2;
        return gram_launch_chain_steps(scratch, theta, p, half, half, 1.0f, nullptr, 0, 0, none, stream, nullptr, stop);
    }
    float* buf[2] = {scratch, scratch + (size_t)((N + 1) / 2) * Q * Q};
    // the round that leaves one matrix writes it where the caller wants the product of the launch
    float* fin = product_out ? product_out : buf[0];
    int count = N, which = 0;
    // round 0 reads the moment matrices; the start event rides on its dispatch, the stop event on the last one's
    hipError_t e = launch_pair_round<true, false>(ps, nullptr, count <= 2 ? fin : buf[0], count, p, stream, start, nullptr);
    if (e != hipSuccess) return e;
    const float* cur = count <= 2 ? fin : buf[0];
    count = (count + 1) / 2;
    while (count > 1) {
        float* dst = count <= 2 ? fin : buf[which ^ 1];
        if (dst == cur) dst = buf[which ^ 1];        // (no product_out: the last round must not write what it reads)
        if ((e = launch_pair_round<false, false>(ps, cur, dst, count, p, stream, nullptr, nullptr)) != hipSuccess) return e;
        cur = dst;
        count = (count + 1) / 2;
        which ^= 1;
    }
    return gram_launch_apply(cur, theta, p, stream, nullptr, stop);
}

}  // namespace bmgd
