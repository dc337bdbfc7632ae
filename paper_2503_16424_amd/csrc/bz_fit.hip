// bz_fit.hip -- parameter updates of the optimisation loop (Sec. 3.5).
//
// One Adam step over a few small arrays (control points, colours, opacities,
// widths), and the copy of the optimised values into the curve set's arrays.
// Both are bound by launches, not by memory: an optimisation of 2,048 strokes has
// 26,624 parameters (0.6 MB with moments and gradients), and as separate
// elementwise passes the update took about 40 launches of 2-4 us and the copy 6 (some 110 us of
// GPU time, and 1.1 ms of host time a step).  Here each is one launch of 4.6 us:
// groups share the grid, each thread takes one value.  512x512 step with 2,048
// strokes 380 -> 276 us, host 0.27 ms.
#include "bz_internal.h"

namespace bz {

namespace {

constexpr int kGroups = 8;
constexpr int kThreads = 256;

// First block of every group (groups are padded to whole blocks).
struct Blocks {
    uint32_t first[kGroups + 1];
};

template <typename G>
struct Groups {
    G g[kGroups];
    Blocks b;
    int n;
};

template <typename G>
__device__ inline int group_of(const Groups<G> &a, int64_t &i) {
    int k = 0;
    while (k + 1 < a.n && blockIdx.x >= a.b.first[k + 1]) ++k;    // uniform over the block
    i = (int64_t)(blockIdx.x - a.b.first[k]) * kThreads + threadIdx.x;
    return k;
}

__global__ __launch_bounds__(kThreads) void k_adam(Groups<bz_adam_group> a) {
    int64_t i;
    const bz_adam_group &p = a.g[group_of(a, i)];
    if (i >= p.n) return;
    // the gradient with respect to the stored parameter
    const float g = p.d[i] * (i & 1 ? p.scale_odd : p.scale_even);
    if (p.grad) p.grad[i] = g;
    const float m = fmaf(p.one_minus_beta1, g - p.m[i], p.m[i]);
    const float v = fmaf(p.one_minus_beta2 * g, g, p.beta2 * p.v[i]);
    p.m[i] = m;
    p.v[i] = v;
    float x = fmaf(-p.step_size, m / (sqrtf(v) / p.bias2_sqrt + p.eps), p.param[i]);
    // NaN stays NaN
    x = x < p.lo ? p.lo : x;
    x = x > p.hi ? p.hi : x;
    p.param[i] = x;
}

__global__ __launch_bounds__(kThreads) void k_affine(Groups<bz_affine_group> a) {
    int64_t i;
    const bz_affine_group &p = a.g[group_of(a, i)];
    if (i >= p.n) return;
    float x = p.src[i];
    if (p.add != 0.f) x += p.add;               // a plain copy keeps the sign of zero
    p.dst[i] = x * (i & 1 ? p.scale_odd : p.scale_even);
}

// Blocks of n_groups groups into a; false: too many for one grid.
template <typename G>
bool plan(const G *g, int n, Groups<G> &a) {
    int64_t blocks = 0;
    for (int k = 0; k < n; ++k) {
        a.g[k] = g[k];
        a.b.first[k] = (uint32_t)blocks;
        blocks += (g[k].n + kThreads - 1) / kThreads;
        if (blocks >= (int64_t(1) << 31)) return false;
    }
    a.b.first[n] = (uint32_t)blocks;
    a.n = n;
    return true;
}

bz_status done(hipError_t e) { return e == hipSuccess ? BZ_OK : BZ_ERR_HIP; }

}  // namespace

}  // namespace bz

extern "C" {

bz_status bz_adam_step(const bz_adam_group *groups, int32_t n_groups, hipStream_t s) {
    using namespace bz;
    if (n_groups < 0 || n_groups > kGroups || (n_groups > 0 && !groups)) return BZ_ERR_ARG;
    for (int k = 0; k < n_groups; ++k) {
        const bz_adam_group &g = groups[k];
        if (g.n < 0 || (g.n > 0 && (!g.param || !g.m || !g.v || !g.d))) return BZ_ERR_ARG;
    }
    Groups<bz_adam_group> a = {};
    if (!plan(groups, n_groups, a)) return BZ_ERR_UNSUPPORTED;
    if (a.b.first[n_groups] == 0) return BZ_OK;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_adam, dim3(a.b.first[n_groups]), dim3(kThreads), 0, s, a);
    return done(hipGetLastError());
}

bz_status bz_affine_copy(const bz_affine_group *groups, int32_t n_groups, hipStream_t s) {
    using namespace bz;
    if (n_groups < 0 || n_groups > kGroups || (n_groups > 0 && !groups)) return BZ_ERR_ARG;
    for (int k = 0; k < n_groups; ++k) {
        const bz_affine_group &g = groups[k];
        if (g.n < 0 || (g.n > 0 && (!g.dst || !g.src))) return BZ_ERR_ARG;
    }
    Groups<bz_affine_group> a = {};
    if (!plan(groups, n_groups, a)) return BZ_ERR_UNSUPPORTED;
    if (a.b.first[n_groups] == 0) return BZ_OK;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_affine, dim3(a.b.first[n_groups]), dim3(kThreads), 0, s, a);
    return done(hipGetLastError());
}

}  // extern "C"
