// bz_shape.hip -- per-curve shape terms: area, draw order by area, Xing loss.
//
// Area (Sec. 3.3, depth from area).  A closed curve encloses the region
// between its boundaries A and B; its area is the shoelace sum of the
// polygon A_0 .. A_{K-1}, B_{K-2} .. B_1 of boundary samples (the sampling
// grid of the Gaussians), taken relative to A_0.  An open stroke covers its
// polyline length times its width.  One wave per curve, FP64 samples and
// sums (the areas of a 2048-pixel canvas span eight decades).
//
// Draw order.  Curves sorted by area, smallest in front, ties by index (a
// stable LSD radix sort on the float bits of the non-negative areas, the
// binning's sort kernels; for a batch a second stable pass on the canvas
// index keeps every canvas's curves together), then the first Gaussian of
// every draw position by an exclusive scan of the per-curve Gaussian counts; up to
// 4096 curves all that is one workgroup's work.  Everything stays on
// the device, so the order can follow the curves every step.
//
// Xing loss (Sec. 3.5, the convexity term of LIVE).  Per cubic segment
// P0..P3 of a closed curve's boundaries: D1 = [cross(P1-P0, P2-P1) >= 0] (the
// turn at the first inner point), D2 = cross(P1-P0, P3-P2) / (|P1-P0||P3-P2|)
// (sine from the first control edge to the last); the segment costs
// D1 max(0, -D2) + (1 - D1) max(0, D2): a last edge that turns against the
// first turn (an S bend or a loop) is penalised.  One thread per curve; its
// gradient goes to the curve's own control points, so no atomics.
#include "bz_geom.h"

namespace bz {

namespace {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

__device__ inline double cross2(double2 a, double2 b) { return a.x * b.y - a.y * b.x; }
__device__ inline double2 sub2(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

__device__ inline double wave_sum_d(double v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

__global__ __launch_bounds__(64) void k_area(bz_curves c, float *__restrict__ area) {
    const int i = blockIdx.x;
    const int lane = threadIdx.x;
    const CurveView v = load_curve_by_id(c, i);
    const bool closed = v.kind == BZ_CLOSED;
    const double2 o = boundary_point(v, false, 0);
    double acc = 0.0;
    for (int k = lane; k < v.K - 1; k += 64) {
        const double2 a0 = boundary_point(v, false, k), a1 = boundary_point(v, false, k + 1);
        if (closed) {
            const double2 b0 = boundary_point(v, true, k), b1 = boundary_point(v, true, k + 1);
            acc += cross2(sub2(a0, o), sub2(a1, o)) - cross2(sub2(b0, o), sub2(b1, o));
        } else {
            const double2 d = sub2(a1, a0);
            acc += sqrt(d.x * d.x + d.y * d.y);
        }
    }
    acc = wave_sum_d(acc);
    if (lane == 0) area[i] = (float)(closed ? 0.5 * fabs(acc) : acc * (double)v.width);
}

// Float bits of an area: non-negative floats order as their bits, NaN goes last.
__device__ inline uint32_t area_key(float a) {
    return isnan(a) ? 0xffffffffu : __float_as_uint(fmaxf(a, 0.f));
}

// keys: area keys, values: curve index.
__global__ void k_area_keys(const float *area, int n, uint32_t *keys, uint32_t *vals) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = area_key(area[i]);
    vals[i] = (uint32_t)i;
}

// Second key of a batch's order: the canvas of the curve at each position.
__global__ void k_canvas_keys(const bz_canvas *cv, int n_canvas, const uint32_t *vals, int n,
                              uint32_t *keys) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    keys[p] = (uint32_t)batch_find(cv, n_canvas, (int64_t)vals[p],
                                   [](const bz_canvas &r) { return (int64_t)r.curve_off; });
}

// Gaussians of curve i.
__device__ inline uint32_t curve_gauss(const bz_curves &c, int i) {
    const int rows = c.kind[i] == BZ_CLOSED ? c.r_interior[i] + 2 : 1;
    return (uint32_t)(rows * c.k_samples[i]);
}

__global__ void k_order_counts(bz_curves c, const uint32_t *vals, int32_t *order, uint32_t *cnt) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= c.n_curves) return;
    const int i = (int)vals[p];
    order[p] = i;
    cnt[p] = curve_gauss(c, i);
}

// The whole order of up to kOrderMost curves in one workgroup: (canvas, area key,
// curve) packed in 64 bits (all different, so ties end by index as a stable sort leaves
// them), ordered in LDS, then the first Gaussian of each position by a scan.  m: the
// power of two (at least 64) the list is filled up to.
// - Up to kRankMost curves a key's place is the number of smaller keys, counted by a
//   thread per key (blockDim.x = m): every lane reads the same two keys at a time.
// - More are sorted bitonically (blockDim.x = min(1024, m / 2)).  A wave's 64 pairs of
//   a step of stride up to 64 lie in 128 consecutive keys that no other wave touches:
//   only longer strides need the block's barrier.  Bound by the chain of steps (45 for
//   512 keys, 78 for 4096): 14 us for 400 curves, where the ranks leave 8.6, against
//   130 us for four radix passes of four launches each, the counts and their scan.
constexpr int kOrderMost = 4096;
constexpr int kRankMost = 512;

// Ends with the block's barrier.
__device__ inline void bitonic_sort(uint64_t *key, int m, int t, int nt) {
    bool wide = false;                          // the step before crossed waves
    for (int k = 2; k <= m; k <<= 1) {
        for (int d = k >> 1; d > 0; d >>= 1) {
            if (wide || d > 64) __syncthreads();
            else wave_lds_sync();
            wide = d > 64;
            for (int p = t; p < m / 2; p += nt) {
                const int i = 2 * p - (p & (d - 1));
                const uint64_t a = key[i], b = key[i + d];
                if ((a > b) == ((i & k) == 0)) {
                    key[i] = b;
                    key[i + d] = a;
                }
            }
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(1024) void k_order_small(bz_curves c, const bz_canvas *cv, int n_canvas,
                                                      const float *area, int m, int32_t *order,
                                                      int64_t *gauss_off) {
    __shared__ __align__(16) uint64_t key[kOrderMost];
    __shared__ uint64_t s_wave[16];
    const int n = c.n_curves, t = threadIdx.x, nt = blockDim.x;
    for (int i = t; i < m; i += nt) {
        uint64_t k = ~0ull;                     // after every curve
        if (i < n) {
            const uint32_t canvas =
                cv ? (uint32_t)batch_find(cv, n_canvas, (int64_t)i,
                                          [](const bz_canvas &r) { return (int64_t)r.curve_off; })
                   : 0u;
            k = ((uint64_t)canvas << 48) | ((uint64_t)area_key(area[i]) << 16) | (uint64_t)i;
        }
        key[i] = k;
    }
    __syncthreads();
    if (m <= kRankMost) {
        // a key's place is the number of smaller ones: a thread per key, two keys per
        // LDS read, the same for all lanes
        const uint64_t mine = key[t];
        int rank = 0;
        for (int i = 0; i < n; i += 2) {
            const ulonglong2 two = *reinterpret_cast<const ulonglong2 *>(&key[i]);
            rank += (two.x < mine) + (two.y < mine);
        }
        __syncthreads();
        if (t < n) key[rank] = mine;
        __syncthreads();
    } else
        bitonic_sort(key, m, t, nt);
    // per thread consecutive positions; the scan as in the binning
    const int per = (m + nt - 1) / nt, p0 = t * per;
    uint64_t sum = 0;
    for (int q = 0; q < per && p0 + q < n; ++q) {
        const int i = (int)(key[p0 + q] & 0xffffu);
        order[p0 + q] = i;
        sum += curve_gauss(c, i);
    }
    uint64_t incl = sum;
    const int lane = t & 63, w = t >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t v = __shfl_up(incl, d, 64);
        if (lane >= d) incl += v;
    }
    if (lane == 63) s_wave[w] = incl;
    __syncthreads();
    uint64_t at = incl - sum, total = 0;
    for (int i = 0; i < nt / 64; ++i) {
        if (i < w) at += s_wave[i];
        total += s_wave[i];
    }
    for (int q = 0; q < per && p0 + q < n; ++q) {
        gauss_off[p0 + q] = (int64_t)at;
        at += curve_gauss(c, (int)(key[p0 + q] & 0xffffu));
    }
    if (t == 0) gauss_off[n] = (int64_t)total;
}

__global__ void k_widen(const uint32_t *offs, int n, int64_t *gauss_off) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) gauss_off[p] = (int64_t)offs[p];
}

__global__ void k_zero1(float *p) {
    if (threadIdx.x == 0) p[0] = 0.f;
}

// kAlone: one workgroup has every curve and stores the loss; otherwise each adds its
// part to a loss that is zero already.
template <int NT, bool kAlone>
__global__ __launch_bounds__(NT) void k_xing(bz_curves c, float weight, float *loss,
                                             float *d_ctrl) {
    const int i = blockIdx.x * NT + threadIdx.x;
    double l = 0.0;
    if (i < c.n_curves && c.kind[i] == BZ_CLOSED) {
        const CurveView v = load_curve_by_id(c, i);
        const int m = 3 * v.S;
        float *g = d_ctrl + 2 * (int64_t)c.ctrl_off[i];
        for (int b = 0; b < 2; ++b) {
            for (int s = 0; s < v.S; ++s) {
                double2 P[4];
                int idx[4];
                for (int j = 0; j < 4; ++j) {
                    const int jj = 3 * s + j;
                    P[j] = ctrl_point(v, b == 1, jj);
                    idx[j] = (b == 1 && jj != 0 && jj != m) ? m + jj : jj;
                }
                const double2 e1 = sub2(P[1], P[0]), e2 = sub2(P[2], P[1]), e3 = sub2(P[3], P[2]);
                const double n1 = sqrt(e1.x * e1.x + e1.y * e1.y);
                const double n3 = sqrt(e3.x * e3.x + e3.y * e3.y);
                if (!(n1 > 0.0 && n3 > 0.0)) continue;
                const bool d1 = cross2(e1, e2) >= 0.0;
                const double d2 = cross2(e1, e3) / (n1 * n3);
                const double f = d1 ? (d2 < 0.0 ? -d2 : 0.0) : (d2 > 0.0 ? d2 : 0.0);
                if (f == 0.0) continue;
                l += f;
                const double dfd = d1 ? -1.0 : 1.0;               // d f / d D2 where f > 0
                // d D2 / d e1, d D2 / d e3
                const double inv = 1.0 / (n1 * n3);
                const double g1x = (e3.y * inv - d2 * e1.x / (n1 * n1)) * dfd * weight;
                const double g1y = (-e3.x * inv - d2 * e1.y / (n1 * n1)) * dfd * weight;
                const double g3x = (-e1.y * inv - d2 * e3.x / (n3 * n3)) * dfd * weight;
                const double g3y = (e1.x * inv - d2 * e3.y / (n3 * n3)) * dfd * weight;
                g[2 * idx[1]] += (float)g1x;
                g[2 * idx[1] + 1] += (float)g1y;
                g[2 * idx[0]] -= (float)g1x;
                g[2 * idx[0] + 1] -= (float)g1y;
                g[2 * idx[3]] += (float)g3x;
                g[2 * idx[3] + 1] += (float)g3y;
                g[2 * idx[2]] -= (float)g3x;
                g[2 * idx[2] + 1] -= (float)g3y;
            }
        }
    }
    if (loss) {
        __shared__ double part[NT / 64];
        double s = wave_sum_d(l);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int w = 0; w < NT / 64; ++w) sum += part[w];
            if (kAlone)
                loss[0] = (float)(weight * sum);
            else
                atomicAdd(loss, (float)(weight * sum));
        }
    }
}

}  // namespace

// Workspace of the draw-order pipeline (bytes), 256-byte aligned pieces.
struct OrderLayout {
    int64_t keys, vals, keys2, vals2, hist, part, status, total;
};

OrderLayout order_layout(int64_t n) {
    OrderLayout L;
    int64_t off = 0, m = n > 0 ? n : 1;
    L.keys = off;
    off = align256(off + 4 * m);
    L.vals = off;
    off = align256(off + 4 * m);
    L.keys2 = off;
    off = align256(off + 4 * m);
    L.vals2 = off;
    off = align256(off + 4 * m);
    L.hist = off;
    off = align256(off + 4 * 256 * sort_hist_blocks(m));
    L.part = off;
    off = align256(off + 8 * sort_part_elems(m));
    L.status = off;
    off = align256(off + 16);
    L.total = off;
    return L;
}

int64_t order_workspace_bytes(int64_t n_curves) { return order_layout(n_curves).total; }

hipError_t launch_area(const bz_curves &c, float *area, hipStream_t s) {
    if (c.n_curves > 0) hipLaunchKernelGGL(k_area, dim3(c.n_curves), dim3(64), 0, s, c, area);
    return hipGetLastError();
}

hipError_t launch_area_order(const bz_curves &c, const bz_batch *batch, float *area,
                             int32_t *order, int64_t *gauss_off, void *ws, hipStream_t s) {
    const int n = c.n_curves;
    if (n == 0) return hipGetLastError();
    OrderLayout L = order_layout(n);
    char *w = (char *)ws;
    uint32_t *keys = (uint32_t *)(w + L.keys), *vals = (uint32_t *)(w + L.vals);
    uint32_t *keys2 = (uint32_t *)(w + L.keys2), *vals2 = (uint32_t *)(w + L.vals2);
    uint32_t *hist = (uint32_t *)(w + L.hist);
    uint64_t *part = (uint64_t *)(w + L.part);
    int64_t *status = (int64_t *)(w + L.status);
    hipLaunchKernelGGL(k_area, dim3(n), dim3(64), 0, s, c, area);
    if (n <= kOrderMost && (!batch || batch->n_canvas <= 65536)) {
        int m = 64;
        while (m < n) m *= 2;
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(m <= kRankMost ? m : m > 2048 ? 1024 : m / 2), 0, s,
                           c, batch ? batch->canvas : nullptr, batch ? batch->n_canvas : 0,
                           (const float *)area, m, order, gauss_off);
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)cdiv(n, 256);
    hipLaunchKernelGGL(k_area_keys, dim3(nb), dim3(256), 0, s, (const float *)area, n, keys, vals);
    hipError_t e = sort_pairs_u32(keys, vals, keys2, vals2, n, 32, hist, part, status, s);
    if (e != hipSuccess) return e;
    if (batch) {      // stable by canvas on top: canvas-major, area inside each canvas
        hipLaunchKernelGGL(k_canvas_keys, dim3(nb), dim3(256), 0, s, batch->canvas,
                           batch->n_canvas, (const uint32_t *)vals, n, keys);
        e = sort_pairs_u32(keys, vals, keys2, vals2, n, 16, hist, part, status, s);
        if (e != hipSuccess) return e;
    }
    // after the sort keys2 / vals2 are free: counts and offsets
    hipLaunchKernelGGL(k_order_counts, dim3(nb), dim3(256), 0, s, c, (const uint32_t *)vals,
                       order, keys2);
    e = exclusive_scan_u32(keys2, vals2, n, part, gauss_off + n, status, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_widen, dim3(nb), dim3(256), 0, s, (const uint32_t *)vals2, n, gauss_off);
    return hipGetLastError();
}

hipError_t launch_xing(const bz_curves &c, float weight, float *loss, float *d_ctrl,
                       hipStream_t s) {
    // one workgroup, one launch: 9 -> 5 us for 400 curves
    if (c.n_curves > 0 && c.n_curves <= 512) {
        hipLaunchKernelGGL((k_xing<512, true>), dim3(1), dim3(512), 0, s, c, weight, loss, d_ctrl);
        return hipGetLastError();
    }
    if (loss) hipLaunchKernelGGL(k_zero1, dim3(1), dim3(64), 0, s, loss);
    if (c.n_curves > 0)
        hipLaunchKernelGGL((k_xing<256, false>), dim3((unsigned)cdiv(c.n_curves, 256)), dim3(256), 0,
                           s, c, weight, loss, d_ctrl);
    return hipGetLastError();
}

}  // namespace bz
