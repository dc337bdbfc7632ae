// cnn.hip -- BF16 implicit-GEMM convolutions on the gfx950 matrix cores.
//
// All three passes of a convolution are one GEMM C[m][n] = sum_k A[m][k] B[k][n]
// whose operands are gathered on the fly (no im2col buffer):
//
//   forward      m = output pixel, n = output channel, k = (dy, dx, in channel)
//                A = shifted input pixels, B = filters
//   input grad   m = input pixel,  n = in channel,     k = (dy, dx, out channel)
//                A = the output gradients that pixel fed, B = filters; one GEMM
//                per parity class of the input pixels modulo the stride, over
//                the taps that reach that class only
//   filter grad  m = out channel,  n = (dy, dx, in channel), k = output pixel
//                A = output gradients, B = shifted input pixels
//
// Layers whose channel counts are multiples of 8 (every layer of the proposal network
// but its first filter gradient) take the vector kernels, k_conv_rows and k_wgrad, the
// others k_igemm:
//
// A workgroup (4 waves) computes a 64 x 64 tile of C in steps of 32 along k:
// the 256 threads gather the A and B slices (8 consecutive k per thread) into
// LDS with k contiguous, then each wave runs 2 x 2 v_mfma_f32_16x16x32_bf16 on
// its 32 x 32 quarter.  For that instruction lane l supplies row (l mod 16)
// of A and column (l mod 16) of B, each with the 8 k values 8 (l / 16) ..
// 8 (l / 16) + 7, and receives rows 4 (l / 16) .. 4 (l / 16) + 3 of column
// (l mod 16) of the 16 x 16 result.  The filter gradient splits its long k
// (all output pixels) over workgroups and adds the partial tiles with float
// atomics.
#include "bz_internal.h"
#include "../../include/bz_cnn.h"
#include "cnn_rows.h"

namespace bz {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr int kBM = 64, kBN = 64, kBK = 32;
constexpr int kLdsK = kBK + 8;          // row pitch in bf16 (80 bytes) against bank conflicts
// Filter gradient: output pixels per workgroup.  256 by default; 128 when
// 256 would leave fewer than 512 workgroups (small late layers).  Measured on
// the 256-patch training step: 1024 rows per workgroup ran the first layer's
// 256 workgroups at one per CU (140 us), 128 rows made its 1,728 outputs
// take too many float atomics (141 us); 256 gives 100 us.
constexpr int kSplitRows = 256, kSplitRowsSmall = 128, kSplitMinGroups = 512;

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ inline __bf16 bf_bits(uint16_t u) { return __builtin_bit_cast(__bf16, u); }
__device__ inline float bf_to_f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }

// float -> bfloat16 bits, round to nearest even (finite inputs; NaN stays NaN)
__device__ inline uint16_t f_to_bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// two of them, nearest even, by the instruction that converts a pair
__device__ inline uint32_t pack_bf16(float a, float b) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// Input pixel read by output pixel m through filter tap `tap`, or -1 (padding).
__device__ inline int in_pixel(const Shape &S, int m, int tap) {
    const int hw = (int)S.ho * S.wo;
    const int b = m / hw;
    const int rem = (int)(m - b * hw);
    const int oy = rem / S.wo, ox = rem - (rem / S.wo) * S.wo;
    const int ky = tap / S.r, kx = tap - (tap / S.r) * S.r;
    const int iy = oy * S.s - S.p + ky, ix = ox * S.s - S.p + kx;
    if (iy < 0 || ix < 0 || iy >= S.h || ix >= S.w) return -1;
    return (b * S.h + iy) * S.w + ix;
}

// Output pixel that input pixel m feeds through tap `tap`, or -1.
__device__ inline int out_pixel(const Shape &S, int m, int tap) {
    const int hw = (int)S.h * S.w;
    const int b = m / hw;
    const int rem = (int)(m - b * hw);
    const int iy = rem / S.w, ix = rem - (rem / S.w) * S.w;
    const int ky = tap / S.r, kx = tap - (tap / S.r) * S.r;
    const int ty = iy + S.p - ky, tx = ix + S.p - kx;
    if (ty < 0 || tx < 0 || ty % S.s || tx % S.s) return -1;
    const int oy = ty / S.s, ox = tx / S.s;
    if (oy >= S.ho || ox >= S.wo) return -1;
    return (b * S.ho + oy) * S.wo + ox;
}

// Input pixel of class row m (input gradient).
__device__ inline int cls_pixel(const GemmArgs &g, int m) {
    if (g.S.s == 1) return m;                   // one class: every pixel
    const int hw = (int)g.hq * g.wq;
    const int b = m / hw;
    const int rem = (int)(m - b * hw);
    const int qy = rem / g.wq, qx = rem - (rem / g.wq) * g.wq;
    return (b * g.S.h + qy * g.S.s + g.cy) * g.S.w + qx * g.S.s + g.cx;
}

// Filter tap of the class's j-th (ky, kx) pair (input gradient).
__device__ inline int cls_tap(const GemmArgs &g, int j) {
    if (g.S.s == 1) return j;                   // one class: every tap
    const int a = j / g.nkx, b = j - (j / g.nkx) * g.nkx;
    return (g.ky0 + a * g.S.s) * g.S.r + g.kx0 + b * g.S.s;
}

// Operand slices travel in two halves so that one k step's loads are in
// flight while the previous step multiplies: fetch_* issues the global loads
// into 8 raw 32-bit registers per thread, put_tiles converts them to BF16 and
// writes LDS after the next barrier.  Raw forms: BF16 vector (4 words of 2
// elements), FP32 (8 float bit patterns, rounded at put), BF16 element (8
// zero-extended halves).
enum RawKind { kRawBf16Vec = 0, kRawF32 = 1, kRawBf16 = 2 };

__device__ inline void raw_to_bf16(int kind, const uint32_t (&r)[8], uint16_t (&v)[8]) {
    if (kind == kRawBf16Vec) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = (uint16_t)r[i];
            v[2 * i + 1] = (uint16_t)(r[i] >> 16);
        }
    } else if (kind == kRawF32) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = f_to_bf(__uint_as_float(r[j]));
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (uint16_t)r[j];
    }
}

// A[m][k .. k+7] and B[k .. k+7][n] for each mode, element by element (zeros
// outside the GEMM); FP32 output gradients stay FP32 (raw) until put.
template <int MODE>
__device__ inline void gather_a(const GemmArgs &g, int m, int k0, int kend,
                                uint32_t (&v)[8]) {
    const Shape &S = g.S;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        uint32_t u = 0;
        if (m < g.M && k < kend) {
            if (MODE == kFwd) {
                const int tap = (int)(k / S.c), ci = (int)(k - (int)tap * S.c);
                const int px = in_pixel(S, m, tap);
                if (px >= 0) u = g.x[px * S.c + ci];
            } else if (MODE == kBwdData) {
                const int j = (int)(k / S.k), co = (int)(k - (int)j * S.k);
                const int px = out_pixel(S, cls_pixel(g, m), cls_tap(g, j));
                if (px >= 0) u = __float_as_uint(g.dy[px * S.k + co]);
            } else {   // m = out channel, k = output pixel
                u = __float_as_uint(g.dy[k * S.k + m]);
            }
        }
        v[j] = u;
    }
}

template <int MODE>
__device__ inline void gather_b(const GemmArgs &g, int n, int k0, int kend,
                                uint32_t (&v)[8]) {
    const Shape &S = g.S;
    const int kf = (int)S.r * S.r * S.c;     // filter length per output channel
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        uint32_t u = 0;
        if (n < g.N && k < kend) {
            if (MODE == kFwd) {
                u = g.w[n * kf + k];
            } else if (MODE == kBwdData) {        // n = in channel, k = (tap, out channel)
                const int j = (int)(k / S.k), co = (int)(k - (int)j * S.k);
                u = g.w[(int)co * kf + (int)cls_tap(g, j) * S.c + n];
            } else {                              // n = (tap, in channel), k = output pixel
                const int tap = (int)(n / S.c), ci = (int)(n - (int)tap * S.c);
                const int px = in_pixel(S, k, tap);
                if (px >= 0) u = g.x[px * S.c + ci];
            }
        }
        v[j] = u;
    }
}

// Filter gradient, B without vector loads (input channels not a multiple of
// 8): B[k .. k+7][n] = the input channel of n at the pixel that output pixels
// k .. k+7 read through the tap of n.  The output pixels are consecutive, so
// the first one's (image, row, column) is divided out once and the others
// follow by stepping along the row (gather_b's element path divides for each).
__device__ inline void gather_b_wgrad(const GemmArgs &g, int n, int k0, int kend,
                                      uint32_t (&v)[8]) {
    const Shape &S = g.S;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = 0;
    if (n >= g.N || k0 >= kend) return;
    const int tap = (int)(n / S.c), ci = (int)(n - (int)tap * S.c);
    const int ky = tap / S.r, kx = tap - (tap / S.r) * S.r;
    const int hw = (int)S.ho * S.wo;
    int b = k0 / hw;
    const int rem = (int)(k0 - b * hw);
    int oy = rem / S.wo, ox = rem - (rem / S.wo) * S.wo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (k0 + j < kend) {
            const int iy = oy * S.s - S.p + ky, ix = ox * S.s - S.p + kx;
            if (iy >= 0 && ix >= 0 && iy < S.h && ix < S.w)
                v[j] = g.x[((b * S.h + iy) * S.w + ix) * S.c + ci];
        }
        if (++ox == S.wo) {
            ox = 0;
            if (++oy == S.ho) {
                oy = 0;
                ++b;
            }
        }
    }
}

// 8 bf16 from a 16-byte aligned address (4 raw words), or zeros.
__device__ inline void fetch8_bf16(const uint16_t *p, bool ok, uint32_t (&r)[8]) {
    uint4 q = make_uint4(0, 0, 0, 0);
    if (ok) q = *reinterpret_cast<const uint4 *>(p);
    r[0] = q.x; r[1] = q.y; r[2] = q.z; r[3] = q.w;
    r[4] = r[5] = r[6] = r[7] = 0;
}

// 8 floats from a 32-byte aligned address (raw bits), or zeros.
__device__ inline void fetch8_f32(const float *p, bool ok, uint32_t (&r)[8]) {
    uint4 a = make_uint4(0, 0, 0, 0), b = a;
    if (ok) {
        a = reinterpret_cast<const uint4 *>(p)[0];
        b = reinterpret_cast<const uint4 *>(p)[1];
    }
    r[0] = a.x; r[1] = a.y; r[2] = a.z; r[3] = a.w;
    r[4] = b.x; r[5] = b.y; r[6] = b.z; r[7] = b.w;
}

// How each operand of a mode moves.  VA / VB: the operand's contiguous
// dimension holds whole groups of 8, so a thread moves 8 neighbours with one
// vector load: along k for operands stored k-contiguous (forward input and
// filters, input-gradient output gradients), along m or n otherwise (written
// transposed, "mn-major").  Else the element gather, k-major.
template <int MODE, bool VA>
struct OpA {
    static constexpr bool kMn = MODE == kBwdWeight && VA;
    static constexpr int kKind = (MODE == kFwd) ? (VA ? kRawBf16Vec : kRawBf16) : kRawF32;
};
template <int MODE, bool VB>
struct OpB {
    static constexpr bool kMn = (MODE == kBwdData || MODE == kBwdWeight) && VB;
    static constexpr int kKind = VB ? kRawBf16Vec : kRawBf16;
};

// Global loads of one k step's slices into registers.
template <int MODE, bool VA, bool VB>
__device__ inline void fetch_tiles(const GemmArgs &g, int m0, int n0, int k0,
                                   int kend, uint32_t (&ra)[8], uint32_t (&rb)[8]) {
    const Shape &S = g.S;
    const int t = threadIdx.x;
    const int lrow = t >> 2, lk = (t & 3) * 8;          // k-major slot: row, 8 k
    const int tk = t >> 3, tc = (t & 7) * 8;            // mn-major slot: k, 8 rows
    const int kf = (int)S.r * S.r * S.c;
    // ---- A ----
    if (MODE == kFwd && VA) {
        const int m = m0 + lrow, k = k0 + lk;
        const int tap = (int)(k / S.c), ci = (int)(k - (int)tap * S.c);
        const int px = (m < g.M && k < kend) ? in_pixel(S, m, tap) : -1;
        fetch8_bf16(g.x + (px >= 0 ? px * S.c + ci : 0), px >= 0, ra);
    } else if (MODE == kBwdData && VA) {
        const int m = m0 + lrow, k = k0 + lk;
        const int j = (int)(k / S.k), co = (int)(k - (int)j * S.k);
        const int px =
            (m < g.M && k < kend) ? out_pixel(S, cls_pixel(g, m), cls_tap(g, j)) : -1;
        fetch8_f32(g.dy + (px >= 0 ? px * S.k + co : 0), px >= 0, ra);
    } else if (MODE == kBwdWeight && VA) {              // A[co][pixel] = dy[pixel][co]
        const int k = k0 + tk, m = m0 + tc;
        const bool ok = k < kend && m < g.M;
        fetch8_f32(g.dy + (ok ? k * S.k + m : 0), ok, ra);
    } else {
        gather_a<MODE>(g, m0 + lrow, k0 + lk, kend, ra);
    }
    // ---- B ----
    if (MODE == kFwd && VB) {
        const int n = n0 + lrow, k = k0 + lk;
        const bool ok = n < g.N && k < kend;
        fetch8_bf16(g.w + (ok ? n * kf + k : 0), ok, rb);
    } else if (MODE == kBwdData && VB) {                // B[(tap, co)][ci] = w[co][tap][ci]
        const int k = k0 + tk, n = n0 + tc;
        const int j = (int)(k / S.k), co = (int)(k - (int)j * S.k);
        const bool ok = k < kend && n < g.N;
        fetch8_bf16(g.w + (ok ? (int)co * kf + (int)cls_tap(g, j) * S.c + n : 0), ok, rb);
    } else if (MODE == kBwdWeight && VB) {              // B[pixel][(tap, ci)] = x[shifted pixel][ci]
        const int k = k0 + tk, n = n0 + tc;
        const int tap = (int)(n / S.c), ci = (int)(n - (int)tap * S.c);
        const int px = (k < kend && n < g.N) ? in_pixel(S, k, tap) : -1;
        fetch8_bf16(g.x + (px >= 0 ? px * S.c + ci : 0), px >= 0, rb);
    } else if (MODE == kBwdWeight) {
        gather_b_wgrad(g, n0 + lrow, k0 + lk, kend, rb);
    } else {
        gather_b<MODE>(g, n0 + lrow, k0 + lk, kend, rb);
    }
}

// The fetched slices, rounded to BF16, into LDS (k contiguous in sA[m][.],
// sB[n][.]).
template <int MODE, bool VA, bool VB>
__device__ inline void put_tiles(const uint32_t (&ra)[8], const uint32_t (&rb)[8],
                                 uint16_t (*sA)[kLdsK], uint16_t (*sB)[kLdsK]) {
    const int t = threadIdx.x;
    const int lrow = t >> 2, lk = (t & 3) * 8;
    const int tk = t >> 3, tc = (t & 7) * 8;
    uint16_t v[8];
    raw_to_bf16(OpA<MODE, VA>::kKind, ra, v);
    if (OpA<MODE, VA>::kMn) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sA[tc + j][tk] = v[j];
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) sA[lrow][lk + j] = v[j];
    }
    raw_to_bf16(OpB<MODE, VB>::kKind, rb, v);
    if (OpB<MODE, VB>::kMn) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sB[tc + j][tk] = v[j];
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) sB[lrow][lk + j] = v[j];
    }
}

template <int MODE, bool VA, bool VB>
__global__ __launch_bounds__(256) void k_igemm(GemmArgs args) {
    __shared__ __align__(16) uint16_t sA[kBM][kLdsK];
    __shared__ __align__(16) uint16_t sB[kBN][kLdsK];
    GemmArgs g = args;
    if (MODE == kBwdData) set_class(g, (int)blockIdx.z);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int m0 = (int)blockIdx.x * kBM, n0 = (int)blockIdx.y * kBN;
    if (m0 >= g.M) return;                            // this class has fewer rows
    int kbeg = 0, kend = g.K;
    if (MODE == kBwdWeight) {
        kbeg = (int)blockIdx.z * g.k_chunk;
        kend = kbeg + g.k_chunk < g.K ? kbeg + g.k_chunk : g.K;
    }
    const int wm = wave >> 1, wn = wave & 1;
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint32_t ra[8], rb[8];
    fetch_tiles<MODE, VA, VB>(g, m0, n0, kbeg, kend, ra, rb);
    for (int k0 = kbeg; k0 < kend; k0 += kBK) {
        __syncthreads();                              // previous step's reads are done
        put_tiles<MODE, VA, VB>(ra, rb, sA, sB);
        __syncthreads();
        // the next step's loads fly while this one multiplies (past kend
        // they are masked off and give zeros)
        fetch_tiles<MODE, VA, VB>(g, m0, n0, k0 + kBK, kend, ra, rb);
        const int r16 = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bf16x8 a;
#pragma unroll
            for (int j = 0; j < 8; ++j) a[j] = bf_bits(sA[wm * 32 + i * 16 + r16][kq + j]);
#pragma unroll
            for (int jn = 0; jn < 2; ++jn) {
                bf16x8 b;
#pragma unroll
                for (int j = 0; j < 8; ++j) b[j] = bf_bits(sB[wn * 32 + jn * 16 + r16][kq + j]);
                acc[i][jn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i][jn], 0, 0, 0);
            }
        }
    }
    // epilogue: lane holds rows 4 (lane / 16) + e, column lane mod 16 of each block
    const int col = lane & 15, rq = (lane >> 4) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = m0 + wm * 32 + i * 16 + rq + e;
                const int n = n0 + wn * 32 + jn * 16 + col;
                if (m >= g.M || n >= g.N) continue;
                float v = acc[i][jn][e];
                if (MODE == kFwd) {
                    if (g.bias) v += g.bias[n];
                    if (g.relu) v = fmaxf(v, 0.f);
                    if (g.out_f) g.out_f[m * g.N + n] = v;
                    if (g.out_b) g.out_b[m * g.N + n] = f_to_bf(v);
                } else if (MODE == kBwdData) {
                    const int px = cls_pixel(g, m);
                    if (g.mask && !(bf_to_f(g.mask[px * g.N + n]) > 0.f)) v = 0.f;
                    g.out_f[px * g.N + n] = v;
                } else {
                    atomicAdd(&g.out_f[m * g.N + n], v);
                }
            }
}

// ---------------------------------------------------------------------------
// Forward and input gradient, vector form
// ---------------------------------------------------------------------------
//
// For channel counts that are multiples of 8 and outputs that are multiples of
// 4 (every layer of the proposal network).  Same sums in the same order as
// k_igemm (k ascending in steps of 32 through the same instruction), but the
// filters are operand A and the pixels operand B, so that
//  - a lane's 8 consecutive k of a pixel are one 16-byte load of BF16 (two of
//    FP32) straight from global memory into the operand, without index divisions
//    or barriers: where a k slice lies relative to a pixel is a table entry per 8
//    k;
//  - a block lays its columns' filters out in LDS once, lane by lane as the
//    instruction takes them, and each of its waves then goes through row tiles of
//    16 pixels on its own, the next k steps' pixels in flight in a second set of
//    registers.
// Bound by HBM: the first layer writes 134 MB of BF16 at 1024 images, the second
// layer's input gradient moves 470 MB (FP32 gradients and the mask).  Before (k_igemm
// on every shape) -> now, at 1024 images of 32 x 32: first layer 83 -> 52 us (2.9
// TB/s), second 62 -> 45, its input gradient 292 -> 148 us (3.2 TB/s); at 256: 26
// -> 20, 22 -> 17, 78 -> 37 us, the 1 x 1 head 18 -> 12.  k steps in flight: 4
// (forward) and 2 (the FP32 side); half as many cost the second layer's input
// gradient 14%, twice as many the last layers' 15%.

// LDS of a block: the filters of its columns, lane by lane; the slice table; the
// classes; an output tile of 16 pixels per wave.
__host__ __device__ inline int conv_pitch(int nb, int out_bytes) { return 16 * nb * out_bytes + 16; }
inline size_t conv_rows_lds(int64_t steps, int classes, int nb, int out_bytes, int waves) {
    return (size_t)steps * (nb * 1024 + 4 * sizeof(ConvTab)) + classes * sizeof(ConvClass) +
           (size_t)waves * 16 * conv_pitch(nb, out_bytes);
}

template <int MODE, int NB>
__global__ __launch_bounds__(1024) void k_conv_rows(GemmArgs args, int most_steps,
                                                    int classes) {
    constexpr int KS = MODE == kFwd ? 4 : 2;       // steps of 32 k in flight at a time
    constexpr int kV = MODE == kFwd ? 1 : 2;    // 16-byte loads per slice
    constexpr int kOutB = MODE == kFwd ? 2 : 4; // bytes per output
    constexpr int kPer = 16 / kOutB;            // channels per 16 bytes
    extern __shared__ __align__(16) unsigned char s_conv[];
    GemmArgs g = args;
    const Shape &S = g.S;
    const int t = threadIdx.x, nt = blockDim.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j = lane & 15, q = lane >> 4;
    const int n0 = (int)blockIdx.y * 16 * NB;
    const int kf = S.r * S.r * S.c;
    // sW[step][nb][lane][8 k]
    uint16_t *sW = reinterpret_cast<uint16_t *>(s_conv);
    ConvTab *s_tab = reinterpret_cast<ConvTab *>(s_conv + (size_t)most_steps * NB * 1024);
    ConvClass *s_cls = reinterpret_cast<ConvClass *>(s_tab + 4 * most_steps);
    unsigned char *out = reinterpret_cast<unsigned char *>(s_cls + classes) +
                         wave * 16 * conv_pitch(NB, kOutB);
    for (int z = 0, first = 0; z < classes; ++z) {
        if (MODE == kBwdData) set_class(g, (int)blockIdx.z * classes + z);
        const int steps = conv_steps(g.K);
        if (t == 0) s_cls[z] = ConvClass{first, steps, g.cy, g.cx};
        for (int i = t; i < 4 * steps; i += nt) s_tab[4 * first + i] = conv_tab<MODE>(g, 8 * i);
        uint16_t *const dst = sW + first * NB * 512;
        if (MODE == kFwd) {
            // 8 k of one output channel per load, one lane's slice
            for (int u = t; u < steps * NB * 64; u += nt) {
                const int ln = u & 63, nb = (u >> 6) % NB, st = u / (64 * NB);
                const int n = n0 + 16 * nb + (ln & 15), k = 32 * st + 8 * (ln >> 4);
                uint4 w = make_uint4(0, 0, 0, 0);
                if (n < g.N && k < g.K) w = *reinterpret_cast<const uint4 *>(g.w + (n * kf + k));
                *reinterpret_cast<uint4 *>(dst + 8 * u) = w;
            }
        } else {
            // one k of 8 input channels per load, a column of 8 lanes' slices
            for (int u = t; u < steps * 32 * 2 * NB; u += nt) {
                const int n8 = u % (2 * NB), k = u / (2 * NB), n = n0 + 8 * n8;
                uint4 w = make_uint4(0, 0, 0, 0);
                if (n < g.N && k < g.K) {
                    const int jt = k / S.k, co = k - jt * S.k;
                    w = *reinterpret_cast<const uint4 *>(g.w +
                                                         (co * kf + cls_tap(g, jt) * S.c + n));
                }
                const int ln = ((k >> 3) & 3) * 16 + (n8 & 1) * 8;
                uint16_t *d = dst + 8 * (((k >> 5) * NB + (n8 >> 1)) * 64 + ln) + (k & 7);
                const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) d[8 * e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
            }
        }
        first += steps;
    }
    __syncthreads();                            // the block's only barrier
    const Divisor image = conv_image<MODE>(S), line = conv_line<MODE>(S);
    const int tiles = conv_tiles(S, image);
    const int nwaves = (nt >> 6) * (int)gridDim.x;
    // workgroup b runs on XCD b % 8: neighbouring row tiles, which share input
    // pixels, go to the same one
    const int gx = (int)gridDim.x, bx = (int)blockIdx.x;
    const int vb = gx % 8 ? bx : (bx % 8) * (gx / 8) + bx / 8;
    int tile = vb * (nt >> 6) + wave;
    int z = 0, c = 0;                           // the class and the chunk being multiplied
    if (tile >= tiles || n0 >= g.N) return;
    floatx4 acc[NB];
    floatx4 bias[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        acc[nb] = bias[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int n = n0 + 16 * nb + 4 * q;
        if (MODE == kFwd && g.bias && n < g.N) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[nb][e] = g.bias[n + e];
        }
    }
    const int nc = g.N - n0 < 16 * NB ? g.N - n0 : 16 * NB;   // channels of this block
    const int per_px = conv_pieces<MODE>(nc);   // 16-byte pieces of a pixel
    const int px0 = lane / per_px, ch0 = lane - px0 * per_px;
    const bool via_lds = MODE == kBwdData || (g.out_b && g.N % kPer == 0);

    auto load = [&](const ConvRow &r, const ConvClass &cls, int ch, uint4 (&px)[KS][kV]) {
#pragma unroll
        for (int st = 0; st < KS; ++st) {
#pragma unroll
            for (int v = 0; v < kV; ++v) px[st][v] = make_uint4(0, 0, 0, 0);
            if (ch * KS + st >= cls.steps) continue;        // uniform
            const ConvTab e = s_tab[4 * (cls.first + ch * KS + st) + q];
            if (conv_reads<MODE>(S, r, e)) {
                const uint4 *p =
                    MODE == kFwd ? reinterpret_cast<const uint4 *>(g.x + (r.base + e.off))
                                 : reinterpret_cast<const uint4 *>(g.dy + (r.base + e.off));
#pragma unroll
                for (int v = 0; v < kV; ++v) px[st][v] = p[v];
            }
        }
    };
    auto multiply = [&](const ConvClass &cls, int ch, const uint4 (&px)[KS][kV]) {
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            if (ch * KS + st >= cls.steps) continue;        // uniform
            bf16x8 p;
            if (MODE == kFwd) {
                p = __builtin_bit_cast(bf16x8, px[st][0]);
            } else {
                const floatx4 lo = __builtin_bit_cast(floatx4, px[st][0]);
                const floatx4 hi = __builtin_bit_cast(floatx4, px[st][kV - 1]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    p[e] = (__bf16)lo[e];                   // nearest even
                    p[e + 4] = (__bf16)hi[e];
                }
            }
            const uint16_t *w = sW + 8 * ((cls.first + ch * KS + st) * NB * 64 + lane);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    *reinterpret_cast<const bf16x8 *>(w + 8 * 64 * nb), p, acc[nb], 0, 0, 0);
        }
    };
    constexpr int kPieces = (4 * NB * kOutB + 15) / 16;     // of 16 bytes per lane
    // A lane holds channels 4 q .. 4 q + 3 of each 16 for pixel j.  Stored from
    // there, an instruction would write 32 or 64 bytes of each of 16 pixels;
    // through LDS consecutive lanes write consecutive 16 bytes.
    auto store = [&](int opix) {
        constexpr int kPitch = 16 * NB * kOutB + 16;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = n0 + 16 * nb + 4 * q;
            floatx4 v = acc[nb];
            acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (n >= g.N) continue;
            const int at = opix * g.N + n;
            if (MODE == kFwd) {
                if (g.bias) v += bias[nb];
                if (g.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
                }
                if (g.out_f && opix >= 0) *reinterpret_cast<floatx4 *>(g.out_f + at) = v;
                if (g.out_b) {
                    const uint2 h = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
                    if (via_lds)
                        *reinterpret_cast<uint2 *>(out + j * kPitch + (n - n0) * kOutB) = h;
                    else if (opix >= 0)
                        *reinterpret_cast<uint2 *>(g.out_b + at) = h;
                }
            } else {
                *reinterpret_cast<floatx4 *>(out + j * kPitch + (n - n0) * kOutB) = v;
            }
        }
        if (!via_lds) return;
        wave_lds_sync();
        int px = px0, piece = ch0;
#pragma unroll
        for (int it = 0; it < kPieces; ++it) {
            const int po = __shfl(opix, px & 15);
            uint4 d = *reinterpret_cast<const uint4 *>(out + (px & 15) * kPitch + 16 * piece);
            const bool ok = px < 16 && po >= 0;
            const int o = po * g.N + n0 + piece * kPer;
            px += 64 / per_px;
            piece += 64 % per_px;
            if (piece >= per_px) {
                piece -= per_px;
                ++px;
            }
            if (!ok) continue;
            if (MODE == kFwd) {
                *reinterpret_cast<uint4 *>(g.out_b + o) = d;
            } else {
                if (g.mask) {
                    const uint2 h = *reinterpret_cast<const uint2 *>(g.mask + o);
                    if (!(bf_to_f((uint16_t)h.x) > 0.f)) d.x = 0u;
                    if (!(bf_to_f((uint16_t)(h.x >> 16)) > 0.f)) d.y = 0u;
                    if (!(bf_to_f((uint16_t)h.y) > 0.f)) d.z = 0u;
                    if (!(bf_to_f((uint16_t)(h.y >> 16)) > 0.f)) d.w = 0u;
                }
                *reinterpret_cast<uint4 *>(g.out_f + o) = d;
            }
        }
        wave_lds_sync();
    };
    // Two sets of registers in turn: one chunk's pixels travel while the other's
    // are multiplied, across the ends of classes and tiles too.
    auto class_of = [&](int i) {
        const ConvClass v = s_cls[i];
        return ConvClass{__builtin_amdgcn_readfirstlane(v.first),
                         __builtin_amdgcn_readfirstlane(v.steps),
                         __builtin_amdgcn_readfirstlane(v.cy), __builtin_amdgcn_readfirstlane(v.cx)};
    };
    ConvRow row = conv_row<MODE>(g, image, line, tile, j);
    ConvClass cls = class_of(0);
    uint4 pa[KS][kV], pb[KS][kV];
    load(row, cls, 0, pa);
    auto advance = [&](const uint4 (&cur)[KS][kV], uint4 (&nxt)[KS][kV]) {
        const bool done = (c + 1) * KS >= cls.steps;        // the class's last chunk
        const int opix = conv_out<MODE>(g, row, tile, j, cls);
        const ConvClass ccls = cls;
        const int cc = c;
        if (!done) {
            ++c;
        } else {
            c = 0;
            if (++z == classes) {
                z = 0;
                tile += nwaves;
                if (tile < tiles) row = conv_row<MODE>(g, image, line, tile, j);
            }
            if (MODE == kBwdData) cls = class_of(z);
        }
        if (tile < tiles) load(row, cls, c, nxt);
        multiply(ccls, cc, cur);
        if (done) store(opix);
        return tile < tiles;
    };
    while (advance(pa, pb) && advance(pb, pa)) {}
}

inline bool aligned(const void *p, uintptr_t n) { return ((uintptr_t)p & (n - 1)) == 0; }

// Does the vector form serve the call?  Its loads and stores are 16 and 8 bytes
// wide: channel counts and pointers decide.
template <int MODE>
bool conv_rows_serves(const GemmArgs &g) {
    const Shape &S = g.S;
    if (S.c % 8 || g.N % 4 || (MODE == kBwdData && S.k % 8)) return false;
    // 16-bit rows and columns of the slice table; blockIdx.y
    const int most = 0x2000;
    if (S.h >= most || S.w >= most || g.N >= (1 << 19)) return false;
    return aligned(MODE == kFwd ? (const void *)g.x : (const void *)g.dy, 16) && aligned(g.w, 16) &&
           aligned(g.out_f, 16) && aligned(g.out_b, 16) && aligned(g.mask, 8);
}

// Workgroups of a vector convolution: waves per block and blocks per column and class.
struct ConvGrid {
    int waves;
    size_t lds;
    int64_t gx, most;           // blocks wanted (one row tile per wave), resident
};

template <int MODE>
ConvGrid conv_grid(int64_t rows, int64_t n, int64_t steps, int classes, int groups, int nb) {
    constexpr int kOutB = MODE == kFwd ? 2 : 4;
    ConvGrid c;
    // the filters' LDS decides how many blocks a CU holds: 16 waves in one block
    // where two blocks do not fit
    c.waves = conv_rows_lds(steps, classes, nb, kOutB, 8) > 80 * 1024 ? 16 : 8;
    c.lds = conv_rows_lds(steps, classes, nb, kOutB, c.waves);
    const int64_t per_cu = c.lds > 80 * 1024 || c.waves == 16 ? 1 : c.lds > 53 * 1024 ? 2 : 3;
    c.gx = cdiv(cdiv(rows, 16), c.waves);
    // rounded down: two blocks more than the chip holds run alone at the end (384 to 384
    // channels, 1 x 1, 65,536 pixels: 171 us for the input gradient)
    c.most = 256 * per_cu / (cdiv(n, 16 * nb) * groups);
    if (c.most < 1) c.most = 1;
    return c;
}

template <int MODE, int NB>
void launch_conv_rows(const GemmArgs &g, int64_t rows, int steps, int classes, int groups,
                      hipStream_t s) {
    const ConvGrid c = conv_grid<MODE>(rows, g.N, steps, classes, groups, NB);
    // resident blocks only: a wave takes several tiles, its filters loaded once
    hipLaunchKernelGGL((k_conv_rows<MODE, NB>),
                       dim3((unsigned)(c.gx < c.most ? c.gx : c.most),
                            (unsigned)cdiv(g.N, 16 * NB), (unsigned)groups),
                       dim3(64 * c.waves), c.lds, s, g, steps, classes);
}

// rows: output pixels, or blocks of stride x stride input pixels.  Steps of 32 k:
// over all classes, and in the class with most.  False: k_igemm is to be used.
//
// A block takes 64 output channels and, for the input gradient, all classes of its
// pixel blocks (their output gradients are then read once, and no class's waves
// end early: 163 -> 147 us for the second layer at 1024 images against a class per
// block).  Where that would leave CUs without a block, or the filters do not fit, it takes
// one class, and below that 16 channels (all classes together there: the third layer at
// 256 images 14 -> 23 us).
//
// With 16 channels a block each pixel is read by n / 16 blocks, where k_igemm's read it
// n / 64 times.  That pays while 64-channel blocks would be few (narrow_pays): 128 to 128
// channels, 3 x 3, input gradient, 47 -> 20 us at 4,096 pixels, but 58 -> 90 at 16,384
// and 134 -> 255 at 65,536 (forward 21 -> 12, 24 -> 50, 54 -> 133; 384 channels at
// 65,536 pixels 409 -> 1,873).  Up to 128 such blocks it was always at least even; above,
// where the 16-channel blocks are all resident at once: 256 to 256 at 4,096 pixels (128
// wide blocks) 86 -> 61, 96 to 96 at 16,384 (256 of them) 19 -> 16, but 19 -> 22 with a
// stride of 2, whose rows lie apart, hence the bound of 192 there.
template <int MODE>
bool try_conv_rows(const GemmArgs &g, int64_t rows, int64_t steps, int64_t longest, int classes,
                   hipStream_t s) {
    constexpr int kOutB = MODE == kFwd ? 2 : 4;
    constexpr size_t kMost = 144 * 1024;
    if (!conv_rows_serves<MODE>(g) || longest > 4096) return false;
    const int64_t wide = cdiv(rows, 16 * 8) * cdiv(g.N, 64);
    const auto narrow_pays = [&] {
        const ConvGrid c = conv_grid<MODE>(rows, g.N, longest, 1, classes, 1);
        return wide < 128 || (c.gx <= c.most && (wide < 192 || g.S.s == 1));
    };
    if (wide >= 192 && conv_rows_lds(steps, classes, 4, kOutB, 16) <= kMost)
        launch_conv_rows<MODE, 4>(g, rows, (int)steps, classes, 1, s);
    else if (wide * classes >= 192 && conv_rows_lds(longest, 1, 4, kOutB, 16) <= kMost)
        launch_conv_rows<MODE, 4>(g, rows, (int)longest, 1, classes, s);
    else if (conv_rows_lds(longest, 1, 1, kOutB, 16) <= kMost && narrow_pays())
        launch_conv_rows<MODE, 1>(g, rows, (int)longest, 1, classes, s);
    else
        return false;
    return true;
}

// ---------------------------------------------------------------------------
// Filter and bias gradient, vector form
// ---------------------------------------------------------------------------
//
// For channel counts that are multiples of 8.  A workgroup takes 64 output
// channels by 64 (tap, input channel) columns over k_chunk output pixels, 128
// at a time: a thread loads 8 channels of 4 consecutive pixels of each operand
// (16 bytes per load) and writes them to LDS with the pixels contiguous, as the
// matrix instruction takes them, 8 bytes per channel; the next 128 pixels'
// loads are in flight meanwhile.  The first column block also sums the output
// gradients (FP32) into the bias gradient.  Bound by the operands' way from
// the L2 (each of the 9 column tiles of a 64-channel 3 x 3 layer reads both), so
// the tiles of a chunk share an XCD: second layer at 1024 images 137 -> 100 us.
// Before (k_igemm and a bias pass) -> now: that layer 176 -> 89 us, at 256 images
// 60 -> 35, the three after it 29 -> 15, 18 -> 11 and 16 -> 11 us.
// Workgroups of the filter gradient: more of them mean more float atomics on dw
// (64-byte requests to memory at about 20 G/s), fewer a longer tail.  The third
// layer at 256 images takes 15 us with 512 and 17 with 1024; the second at 1024
// images 100 and 89 (and 140 with 256).
constexpr int kWgGroups = 512;
constexpr int kWgPix = 128;
constexpr int kWgPitch = kWgPix + 4;        // 66 words: eight rows apart, other banks

__global__ __launch_bounds__(256) void k_wgrad(GemmArgs g, float *db) {
    __shared__ __align__(16) uint16_t sA[64][kWgPitch], sB[64][kWgPitch];
    __shared__ float s_db[8][64];
    const Shape &S = g.S;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int cg = t & 7, pg = t >> 3;          // 8 channels, 4 pixels
    // workgroup b runs on XCD b % 8: the tiles of a chunk of pixels, which read the
    // same operands, on one XCD; fewer than eight chunks over all XCDs, tile by tile
    // (512 to 512 channels, 3 x 3, two chunks: 947 us on two XCDs)
    const int tm = (g.M + 63) / 64, tn = (g.N + 63) / 64, tiles = tm * tn;
    const int chunks = (g.K + g.k_chunk - 1) / g.k_chunk;
    int tile, chunk;
    if (chunks >= 8) {
        const int b8 = (int)blockIdx.x / (8 * tiles), in8 = (int)blockIdx.x - b8 * 8 * tiles;
        tile = in8 / 8;
        chunk = b8 * 8 + in8 % 8;
        if (chunk >= chunks) return;
    } else {
        chunk = (int)blockIdx.x / tiles;
        tile = (int)blockIdx.x - chunk * tiles;
    }
    const int m0 = (tile % tm) * 64, n0 = (tile / tm) * 64;
    const int kbeg = chunk * g.k_chunk;
    const int kend = kbeg + g.k_chunk < g.K ? kbeg + g.k_chunk : g.K;
    const int co = m0 + 8 * cg, n = n0 + 8 * cg;
    const int tap = n / S.c, ci = n - tap * S.c, ky = tap / S.r, kx = tap - ky * S.r;
    const bool ok_a = co < g.M, ok_b = n < g.N;
    const bool sum_db = db && n0 == 0;
    floatx4 a[4][2];
    uint4 b[4];
    float bs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bs[e] = 0.f;
    auto fetch = [&](int k0) {
        const int k = k0 + 4 * pg;
        const int hw = S.ho * S.wo;
        int img = k / hw;
        const int rem = k - img * hw;
        int oy = rem / S.wo, ox = rem - oy * S.wo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i][0] = a[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            b[i] = make_uint4(0, 0, 0, 0);
            if (k + i < kend) {
                if (ok_a) {
                    const floatx4 *p = reinterpret_cast<const floatx4 *>(g.dy + ((k + i) * S.k + co));
                    a[i][0] = p[0];
                    a[i][1] = p[1];
                }
                const int iy = oy * S.s - S.p + ky, ix = ox * S.s - S.p + kx;
                if (ok_b && (unsigned)iy < (unsigned)S.h && (unsigned)ix < (unsigned)S.w)
                    b[i] = *reinterpret_cast<const uint4 *>(
                        g.x + (((img * S.h + iy) * S.w + ix) * S.c + ci));
            }
            if (++ox == S.wo) {
                ox = 0;
                if (++oy == S.ho) {
                    oy = 0;
                    ++img;
                }
            }
        }
    };
    const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, q = lane >> 4;
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jn = 0; jn < 2; ++jn) acc[i][jn] = floatx4{0.f, 0.f, 0.f, 0.f};
    fetch(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += kWgPix) {
        __syncthreads();                        // the previous pixels are read
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v0 = a[0][e >> 2][e & 3], v1 = a[1][e >> 2][e & 3];
            const float v2 = a[2][e >> 2][e & 3], v3 = a[3][e >> 2][e & 3];
            if (sum_db) bs[e] += (v0 + v1) + (v2 + v3);
            *reinterpret_cast<uint2 *>(&sA[8 * cg + e][4 * pg]) =
                make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t w4[4] = {b[i].x, b[i].y, b[i].z, b[i].w};
                w[i] = w4[e >> 1];
            }
            // the low or high halves of two pixels side by side
            const uint32_t sel = e & 1 ? 0x07060302u : 0x05040100u;
            *reinterpret_cast<uint2 *>(&sB[8 * cg + e][4 * pg]) =
                make_uint2(__builtin_amdgcn_perm(w[1], w[0], sel),
                           __builtin_amdgcn_perm(w[3], w[2], sel));
        }
        __syncthreads();
        if (k0 + kWgPix < kend) fetch(k0 + kWgPix);
#pragma unroll
        for (int ks = 0; ks < kWgPix / 32; ++ks) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint2 *pa =
                    reinterpret_cast<const uint2 *>(&sA[wm * 32 + i * 16 + r16][ks * 32 + 8 * q]);
                const uint2 *pb =
                    reinterpret_cast<const uint2 *>(&sB[wn * 32 + i * 16 + r16][ks * 32 + 8 * q]);
                const uint2 a0 = pa[0], a1 = pa[1], b0 = pb[0], b1 = pb[1];
                fa[i] = __builtin_bit_cast(bf16x8, make_uint4(a0.x, a0.y, a1.x, a1.y));
                fb[i] = __builtin_bit_cast(bf16x8, make_uint4(b0.x, b0.y, b1.x, b1.y));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int jn = 0; jn < 2; ++jn)
                    acc[i][jn] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[jn], acc[i][jn], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = m0 + wm * 32 + i * 16 + 4 * q + e;
                const int nn = n0 + wn * 32 + jn * 16 + r16;
                if (m < g.M && nn < g.N) atomicAdd(&g.out_f[m * g.N + nn], acc[i][jn][e]);
            }
    if (!sum_db) return;                        // uniform over the block
    // the 32 pixel groups' sums of a channel: 8 lanes apart in a wave, then the waves
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bs[e] += __shfl_xor(bs[e], 8);
        bs[e] += __shfl_xor(bs[e], 16);
        bs[e] += __shfl_xor(bs[e], 32);
        if (lane < 8) s_db[wave][8 * cg + e] = bs[e];
    }
    __syncthreads();
    if (t < 64 && m0 + t < g.M)
        atomicAdd(&db[m0 + t], (s_db[0][t] + s_db[1][t]) + (s_db[2][t] + s_db[3][t]));
}

// Dispatch on which operands can move 8 at a time.
template <int MODE>
void launch_igemm(const GemmArgs &g, bool va, bool vb, dim3 grid, hipStream_t s) {
    if (va && vb)
        hipLaunchKernelGGL((k_igemm<MODE, true, true>), grid, dim3(256), 0, s, g);
    else if (va)
        hipLaunchKernelGGL((k_igemm<MODE, true, false>), grid, dim3(256), 0, s, g);
    else if (vb)
        hipLaunchKernelGGL((k_igemm<MODE, false, true>), grid, dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL((k_igemm<MODE, false, false>), grid, dim3(256), 0, s, g);
}

// Filter and bias gradients cleared, in one launch (db may be null).
__global__ void k_fill0(float *p, int64_t n, float *db, int k) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (db)
        for (int64_t o = i; o < k; o += stride) db[o] = 0.f;
    for (; i < n; i += stride) p[i] = 0.f;
}

// db[o] = sum over output pixels of dy[.][o].  Workgroup (chunk, group): 64
// channels x 4 row phases over `chunk` rows, so each wave reads 64
// consecutive floats of a row; the phases meet in LDS and one atomic per
// channel adds the chunk's sum (db is cleared first).  The atomics of all
// workgroups meet on the few lines of db, so chunks are sized for about 256
// workgroups (bias_chunk): at 262,144 rows, chunks of 256 rows took 34 us,
// of 1024 rows 17 us.
inline int64_t bias_chunk(int64_t rows) {
    int64_t c = 256;
    while (c * 256 < rows) c *= 2;
    return c;
}

__global__ __launch_bounds__(256) void k_bias_grad(const float *__restrict__ dy, int64_t rows,
                                                   int64_t chunk, int k, float *db) {
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int o = blockIdx.y * 64 + tx;
    const int64_t r0 = (int64_t)blockIdx.x * chunk;
    const int64_t r1 = rows < r0 + chunk ? rows : r0 + chunk;
    // four independent sums keep four loads of each thread in flight
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (o < k) {
        int64_t r = r0 + ty;
        for (; r + 12 < r1; r += 16) {
            s0 += dy[r * k + o];
            s1 += dy[(r + 4) * k + o];
            s2 += dy[(r + 8) * k + o];
            s3 += dy[(r + 12) * k + o];
        }
        for (; r < r1; r += 4) s0 += dy[r * k + o];
    }
    const float s = (s0 + s1) + (s2 + s3);
    __shared__ float part[4][64];
    part[ty][tx] = s;
    __syncthreads();
    if (ty == 0 && o < k) atomicAdd(&db[o], (part[0][tx] + part[1][tx]) + (part[2][tx] + part[3][tx]));
}

// The same for k a multiple of 4 up to 64 with 16-byte loads: lane l of a wave
// reads channels 4 (l % 16) .. +3 of row phase l / 16, so a wave covers four
// 256-byte rows per load and a workgroup 16 row phases.
__global__ __launch_bounds__(256) void k_bias_grad4(const float *__restrict__ dy, int64_t rows,
                                                    int64_t chunk, int k, float *db) {
    const int t = threadIdx.x, c4 = 4 * (t & 15), ph = t >> 4;     // 16 phases
    const int64_t r0 = (int64_t)blockIdx.x * chunk;
    const int64_t r1 = rows < r0 + chunk ? rows : r0 + chunk;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (c4 < k) {
        int64_t r = r0 + ph;
        for (; r + 16 < r1; r += 32) {
            const float4 u = *reinterpret_cast<const float4 *>(dy + r * k + c4);
            const float4 v = *reinterpret_cast<const float4 *>(dy + (r + 16) * k + c4);
            a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
            b.x += v.x; b.y += v.y; b.z += v.z; b.w += v.w;
        }
        for (; r < r1; r += 16) {
            const float4 u = *reinterpret_cast<const float4 *>(dy + r * k + c4);
            a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
        }
    }
    __shared__ float part[16][64];
    part[ph][c4] = a.x + b.x;
    part[ph][c4 + 1] = a.y + b.y;
    part[ph][c4 + 2] = a.z + b.z;
    part[ph][c4 + 3] = a.w + b.w;
    __syncthreads();
    if (t < k) {
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < 16; ++p) s += part[p][t];
        atomicAdd(&db[t], s);
    }
}

// Filter and bias gradients of the first layer's shape: 3 x 3 filters, stride
// 1, padding 1, at most 3 input channels, 64 output channels, rows of 32
// pixels.  The generic split-K path spends most of its time in float atomics
// there (1,728 outputs per 256 output pixels, all meeting on 54 lines).
//
// One workgroup per image.  The image (h x 32 x C BF16) goes into LDS three
// times, shifted by kx = 0, 1, 2 columns and stored channel-planar with a zero
// border, so the 8 consecutive output pixels a lane feeds the matrix core
// through tap (ky, kx) and channel ci are one aligned 16-byte LDS read.  A
// wave takes whole output rows: a row of 32 pixels is one k step of
// C[co][(tap, ci)] += dy_row^T x shifted input row (4 x 2 blocks of
// v_mfma_f32_16x16x32_bf16), with the next row's dy loads in flight, and the
// bias gradient sums the same dy values in FP32.  The waves meet in LDS; one
// float atomic per output adds the image's share (dw and db are cleared
// first): 1,792 atomics per 1,024 pixels.
constexpr int kWg0Waves = 8;

inline bool wgrad_first_shape(const bz_conv &c) {
    return c.r == 3 && c.stride == 1 && c.pad == 1 && c.c >= 1 && c.c <= 3 && c.k == 64 &&
           c.w == 32 && c.h >= 1 && c.h <= 64;
}

inline size_t wgrad_first_lds(const bz_conv &c) {
    return (size_t)3 * (c.h + 2) * c.c * 32 * sizeof(uint16_t);
}

// dy of output row oy, pixels 8q .. 8q + 7, channels 16 mb + r (mb = 0..3)
__device__ inline void wgrad_first_row(const float *__restrict__ dy, int64_t row, int q, int r,
                                       float (&v)[4][8]) {
    const float *p = dy + (row * 32 + 8 * q) * 64 + r;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) v[mb][j] = p[j * 64 + 16 * mb];
}

// Rows a wave has in flight at once (its rows are wave, wave + 8, ...).
constexpr int kWg0Rows = 4;

template <int C>
__global__ __launch_bounds__(64 * kWg0Waves) void k_wgrad_first(const float *__restrict__ dy,
                                                                const uint16_t *__restrict__ x,
                                                                int h, float *dw, float *db) {
    extern __shared__ __align__(16) uint16_t s_img[];    // [kx][h + 2][C][32]
    // each wave's result blocks, lane-major (the waves meet by plain sums:
    // LDS float atomics from eight waves took longer than the rows)
    __shared__ floatx4 s_part[kWg0Waves][8][64];
    __shared__ float s_bpart[kWg0Waves][64];
    constexpr int kThreads = 64 * kWg0Waves, kPitch = C * 32, kN = 9 * C;
    const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int rows = h + 2, plane = rows * kPitch;
    const int r = lane & 15, q = lane >> 4;
    // the first kWg0Rows rows of dy go in flight before the image is staged
    float v[kWg0Rows][4][8];
#pragma unroll
    for (int i = 0; i < kWg0Rows; ++i)
        if (wave + kWg0Waves * i < h) wgrad_first_row(dy, (int64_t)b * h + wave + kWg0Waves * i, q, r, v[i]);
    // clear the copies (their borders stay zero) and the sums
    for (int i = t; i < 3 * plane / 8; i += kThreads)
        reinterpret_cast<uint4 *>(s_img)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    // s_img[kx][iy + 1][ci][ix + 1 - kx] = x[b][iy][ix][ci]: the image is
    // 64 h C bytes (a multiple of 16, as is its offset), 8 elements per load
    const uint4 *src = reinterpret_cast<const uint4 *>(x + (int64_t)b * h * 32 * C);
    for (int i = t; i < 4 * h * C; i += kThreads) {
        const uint4 u = src[i];
        const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = 8 * i + j;                        // (iy * 32 + ix) * C + ci
            const int px = e / C, ci = e - px * C;
            const int iy = px >> 5, ix = px & 31;
            const uint16_t u16 = (uint16_t)(w4[j >> 1] >> (16 * (j & 1)));
            uint16_t *d = s_img + (iy + 1) * kPitch + ci * 32 + ix + 1;
            if (ix < 31) d[0] = u16;                        // kx = 0
            d[plane - 1] = u16;                             // kx = 1
            if (ix > 0) d[2 * plane - 2] = u16;             // kx = 2
        }
    }
    __syncthreads();
    // B column n = 16 nb + r is (tap, ci) = (n / C, n mod C); lane q feeds
    // output pixels 8q .. 8q + 7 of the row.  Offset of row oy = 0, or -1
    // for the padding columns n >= 9C.
    int boff[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int n = 16 * nb + r;
        boff[nb] = -1;
        if (n < kN) {
            const int tap = n / C, ci = n - tap * C, ky = tap / 3, kx = tap - 3 * ky;
            boff[nb] = (kx * rows + ky) * kPitch + ci * 32 + 8 * q;
        }
    }
    floatx4 acc[4][2];
    float bsum[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
        bsum[mb] = 0.f;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    for (int oy0 = wave; oy0 < h; oy0 += kWg0Waves * kWg0Rows) {
#pragma unroll
        for (int i = 0; i < kWg0Rows; ++i) {
            const int oy = oy0 + kWg0Waves * i;
            if (oy >= h) break;
            bf16x8 bv[2];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                bf16x8 z;
#pragma unroll
                for (int j = 0; j < 8; ++j) z[j] = bf_bits(0);
                bv[nb] = boff[nb] >= 0
                             ? *reinterpret_cast<const bf16x8 *>(s_img + boff[nb] + oy * kPitch)
                             : z;
            }
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) {
                bf16x8 a;
                float sm = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    a[j] = (__bf16)v[i][mb][j];             // v_cvt_pk_bf16_f32, nearest even
                    sm += v[i][mb][j];
                }
                bsum[mb] += sm;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    acc[mb][nb] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bv[nb], acc[mb][nb], 0, 0, 0);
            }
            // refill the slot with the row kWg0Rows ahead (images taller than
            // kWg0Waves * kWg0Rows rows)
            const int on = oy + kWg0Waves * kWg0Rows;
            if (on < h) wgrad_first_row(dy, (int64_t)b * h + on, q, r, v[i]);
        }
    }
    // lane holds C[16 mb + 4q + e][16 nb + r] in acc[mb][nb][e]
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) s_part[wave][2 * mb + nb][lane] = acc[mb][nb];
        float sm = bsum[mb];
        sm += __shfl_xor(sm, 16);
        sm += __shfl_xor(sm, 32);
        if (q == 0) s_bpart[wave][16 * mb + r] = sm;
    }
    __syncthreads();
    for (int o = t; o < 64 * kN + 64; o += kThreads) {
        float sum = 0.f;
        if (o < 64 * kN) {
            const int m = o / kN, n = o - m * kN;
            const int blk = 2 * (m >> 4) + (n >> 4), ln = 16 * ((m >> 2) & 3) + (n & 15), e = m & 3;
#pragma unroll
            for (int w = 0; w < kWg0Waves; ++w) sum += s_part[w][blk][ln][e];
            atomicAdd(&dw[o], sum);
        } else if (db) {
#pragma unroll
            for (int w = 0; w < kWg0Waves; ++w) sum += s_bpart[w][o - 64 * kN];
            atomicAdd(&db[o - 64 * kN], sum);
        }
    }
}

template <int C>
void launch_wgrad_first(const bz_conv &c, const float *dy, const uint16_t *x, float *dw,
                        float *db, hipStream_t s) {
    hipLaunchKernelGGL(k_wgrad_first<C>, dim3((unsigned)c.n), dim3(64 * kWg0Waves),
                       wgrad_first_lds(c), s, dy, x, c.h, dw, db);
}

__global__ void k_to_bf16(const float *src, uint16_t *dst, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dst[i] = f_to_bf(src[i]);
}

// Patches: a thread takes kN consecutive pixels of a row (4 where the side allows: 24
// bytes in three stores), workgroups of blockIdx.y one patch at a time.  A thread per
// value, with its divisions, took 13.6 us for 1,024 patches of 32 x 32; this 8.3.
template <int kN>
__global__ __launch_bounds__(256) void k_patches(const float *img, int W, int H, const int32_t *xy,
                                                 int np, int side, float fill, uint16_t *out) {
    const int64_t plane = (int64_t)W * H;
    const int groups = side * side / kN;
    const Divisor row = divisor(side / kN);
    for (int p = blockIdx.y; p < np; p += gridDim.y) {
        const int px = xy[2 * p], py = xy[2 * p + 1];
        for (int q = blockIdx.x * 256 + threadIdx.x; q < groups; q += gridDim.x * 256) {
            const int r = divide(q, row), x = px + (q - r * (int)row.d) * kN, y = py + r;
            float v[3 * kN];
#pragma unroll
            for (int i = 0; i < kN; ++i) {
                const bool in = x + i >= 0 && x + i < W && y >= 0 && y < H;
                const int64_t at = (int64_t)y * W + x + i;
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) v[3 * i + ch] = in ? img[ch * plane + at] : fill;
            }
            uint16_t *o = out + ((int64_t)p * groups + q) * (3 * kN);
            if (kN == 4) {
                uint32_t h[6];
#pragma unroll
                for (int i = 0; i < 6; ++i)
                    h[i] = (uint32_t)f_to_bf(v[2 * i % (3 * kN)]) |
                           ((uint32_t)f_to_bf(v[(2 * i + 1) % (3 * kN)]) << 16);
                uint2 *o2 = reinterpret_cast<uint2 *>(o);
                o2[0] = make_uint2(h[0], h[1]);
                o2[1] = make_uint2(h[2], h[3]);
                o2[2] = make_uint2(h[4], h[5]);
            } else {
#pragma unroll
                for (int i = 0; i < 3 * kN; ++i) o[i] = f_to_bf(v[i]);
            }
        }
    }
}

// Pixels of c <= 8 channels to pixels of 8, zeros behind.
__global__ __launch_bounds__(256) void k_pad8(const uint16_t *src, int64_t n_pix, int c, uint4 *dst) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (; i < n_pix; i += stride) {
        uint16_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = j < c ? src[i * c + j] : (uint16_t)0;
        dst[i] = make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16),
                            (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                            (uint32_t)v[4] | ((uint32_t)v[5] << 16),
                            (uint32_t)v[6] | ((uint32_t)v[7] << 16));
    }
}

// Raw outputs to normalised curve parameters, one value per thread.  As five elementwise
// passes and a concatenation 20 us for 1,024 patches, bound by launches.
__global__ __launch_bounds__(256) void k_decode(const float *z, int64_t n, int per, int points,
                                                float scale, float shift, float *out) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (; i < n; i += stride) {
        const float s = 1.f / (1.f + expf(-z[i]));
        float v = s;
        if ((int)(i % per) < points) {
            _Pragma("clang fp contract(off)") v = s * scale;
            v = v - shift;
        }
        out[i] = v;
    }
}

Shape shape_of(const bz_conv &c) {
    return Shape{c.n, c.h, c.w, c.c, c.k, c.r, c.stride, c.pad, c.ho, c.wo};
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_conv_fwd(const bz_conv &c, const uint16_t *x, const uint16_t *w,
                           const float *bias, int relu, float *y, uint16_t *yb, hipStream_t s) {
    GemmArgs g = {};
    g.S = shape_of(c);
    g.M = (int64_t)c.n * c.ho * c.wo;
    g.N = c.k;
    g.K = (int64_t)c.r * c.r * c.c;
    g.x = x;
    g.w = w;
    g.bias = bias;
    g.relu = relu;
    g.out_f = y;
    g.out_b = yb;
    if (try_conv_rows<kFwd>(g, g.M, cdiv(g.K, 32), cdiv(g.K, 32), 1, s)) return hipGetLastError();
    dim3 grid((unsigned)cdiv(g.M, kBM), (unsigned)cdiv(g.N, kBN), 1);
    // A: 8 input channels per load (c % 8); B: 8 filter taps-channels per load (K % 8)
    launch_igemm<kFwd>(g, c.c % 8 == 0, g.K % 8 == 0 && c.c % 8 == 0, grid, s);
    return hipGetLastError();
}

hipError_t launch_conv_bwd_data(const bz_conv &c, const float *dy, const uint16_t *w,
                                const uint16_t *mask, float *dx, hipStream_t s) {
    // One GEMM per parity class of the input pixels (stride^2 of them, one
    // launch, blockIdx.z = class): a tap reaches input row iy only if
    // iy + pad - ky is a multiple of the stride, so each class gathers only its
    // own taps (for 3x3 stride 2: 1, 2, 2 or 4 of the 9) instead of zeros.
    GemmArgs g = {};
    g.S = shape_of(c);
    g.N = c.c;
    g.dy = dy;
    g.w = w;
    g.mask = mask;
    g.out_f = dx;
    const int st = c.stride;
    const int64_t rows = (int64_t)c.n * ((c.h + st - 1) / st) * ((c.w + st - 1) / st);  // class 0
    int64_t steps = 0, longest = 0;             // of 32 k
    for (int ky = 0; ky < st && ky < c.r; ++ky)
        for (int kx = 0; kx < st && kx < c.r; ++kx) {
            const int64_t n = cdiv((int64_t)cdiv(c.r - ky, st) * cdiv(c.r - kx, st) * c.k, 32);
            steps += n;
            longest = longest < n ? n : longest;
        }
    if (try_conv_rows<kBwdData>(g, rows, steps, longest, st * st, s)) return hipGetLastError();
    dim3 grid((unsigned)cdiv(rows, kBM), (unsigned)cdiv(g.N, kBN), (unsigned)(st * st));
    // A: 8 output channels of dy (k % 8); B: 8 input channels of a filter row (c % 8)
    launch_igemm<kBwdData>(g, c.k % 8 == 0, c.c % 8 == 0, grid, s);
    return hipGetLastError();
}

hipError_t launch_conv_bwd_weight(const bz_conv &c, const float *dy, const uint16_t *x,
                                  float *dw, float *db, bool cleared, hipStream_t s) {
    GemmArgs g = {};
    g.S = shape_of(c);
    g.M = c.k;
    g.N = (int64_t)c.r * c.r * c.c;
    g.K = (int64_t)c.n * c.ho * c.wo;
    g.dy = dy;
    g.x = x;
    g.out_f = dw;
    const int64_t tiles = cdiv(g.M, kBM) * cdiv(g.N, kBN);
    const int64_t nz = (int64_t)g.M * g.N;
    if (!cleared)
        hipLaunchKernelGGL(k_fill0, dim3((unsigned)cdiv(nz, 256) < 4096 ? (unsigned)cdiv(nz, 256) : 4096),
                           dim3(256), 0, s, dw, nz, db, c.k);
    if (wgrad_first_shape(c) && ((uintptr_t)x & 15) == 0) {     // 16-byte image loads
        if (c.c == 1) launch_wgrad_first<1>(c, dy, x, dw, db, s);
        else if (c.c == 2) launch_wgrad_first<2>(c, dy, x, dw, db, s);
        else launch_wgrad_first<3>(c, dy, x, dw, db, s);
        return hipGetLastError();
    }
    if (c.k % 8 == 0 && c.c % 8 == 0 && aligned(dy, 16) && aligned(x, 16)) {
        // about kWgGroups workgroups, twice as many over 1024 pixels for each
        int64_t splits = cdiv(kWgGroups, tiles);
        if (g.K > 1024 * splits) splits *= 2;
        g.k_chunk = (int)(cdiv(cdiv(g.K, splits), kWgPix) * kWgPix);
        const int64_t chunks = cdiv(g.K, g.k_chunk);
        hipLaunchKernelGGL(k_wgrad, dim3((unsigned)(tiles * (chunks >= 8 ? cdiv(chunks, 8) * 8 : chunks))),
                           dim3(256), 0, s, g, db);
        return hipGetLastError();
    }
    g.k_chunk = cdiv(g.K, kSplitRows) * tiles < kSplitMinGroups ? kSplitRowsSmall : kSplitRows;
    dim3 grid((unsigned)cdiv(g.M, kBM), (unsigned)cdiv(g.N, kBN), (unsigned)cdiv(g.K, g.k_chunk));
    // A: 8 output channels of dy (k % 8); B: 8 input channels of a shifted pixel (c % 8)
    launch_igemm<kBwdWeight>(g, c.k % 8 == 0, c.c % 8 == 0, grid, s);
    if (db) {
        // dy rows are 16-byte aligned when k % 4 == 0 (dy itself is)
        const int64_t chunk = bias_chunk(g.K);
        if (c.k % 4 == 0 && c.k <= 64 && ((uintptr_t)dy & 15) == 0)
            hipLaunchKernelGGL(k_bias_grad4, dim3((unsigned)cdiv(g.K, chunk)), dim3(256), 0, s,
                               dy, g.K, chunk, c.k, db);
        else
            hipLaunchKernelGGL(k_bias_grad, dim3((unsigned)cdiv(g.K, chunk), (unsigned)cdiv(c.k, 64)),
                               dim3(256), 0, s, dy, g.K, chunk, c.k, db);
    }
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *src, uint16_t *dst, int64_t n, hipStream_t s) {
    if (n > 0) {
        int64_t b = cdiv(n, 256);
        hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)(b < 4096 ? b : 4096)), dim3(256), 0, s, src,
                           dst, n);
    }
    return hipGetLastError();
}

hipError_t launch_patches(const float *img, int W, int H, const int32_t *xy, int np, int side,
                          float fill, uint16_t *out, hipStream_t s) {
    if (np > 0) {
        const bool four = side % 4 == 0 && aligned(out, 8);
        const int64_t groups = (int64_t)side * side / (four ? 4 : 1);
        const dim3 grid((unsigned)cdiv(groups, 256), (unsigned)(np < 32768 ? np : 32768));
        if (four)
            hipLaunchKernelGGL(k_patches<4>, grid, dim3(256), 0, s, img, W, H, xy, np, side, fill,
                               out);
        else
            hipLaunchKernelGGL(k_patches<1>, grid, dim3(256), 0, s, img, W, H, xy, np, side, fill,
                               out);
    }
    return hipGetLastError();
}

}  // namespace bz

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace bz;

extern "C" {

bz_status bz_conv_shape(bz_conv *cv) {
    if (!cv) return BZ_ERR_ARG;
    if (cv->n < 1 || cv->h < 1 || cv->w < 1 || cv->c < 1 || cv->k < 1) return BZ_ERR_ARG;
    if (cv->r != 1 && cv->r != 3) return BZ_ERR_ARG;
    if (cv->stride < 1 || cv->stride > 4 || cv->pad < 0 || cv->pad >= cv->r) return BZ_ERR_ARG;
    const int64_t ho = ((int64_t)cv->h + 2 * cv->pad - cv->r) / cv->stride + 1;
    const int64_t wo = ((int64_t)cv->w + 2 * cv->pad - cv->r) / cv->stride + 1;
    if ((int64_t)cv->h + 2 * cv->pad < cv->r || (int64_t)cv->w + 2 * cv->pad < cv->r || ho < 1 ||
        wo < 1)
        return BZ_ERR_ARG;
    const int64_t lim = int64_t(1) << 30;      // index arithmetic stays in 32 bits
    if ((int64_t)cv->n * cv->h * cv->w * cv->c >= lim || (int64_t)cv->n * ho * wo * cv->k >= lim ||
        (int64_t)cv->k * cv->r * cv->r * cv->c >= lim)
        return BZ_ERR_UNSUPPORTED;
    cv->ho = (int32_t)ho;
    cv->wo = (int32_t)wo;
    return BZ_OK;
}

static bz_status check_conv(const bz_conv *cv) {
    if (!cv) return BZ_ERR_ARG;
    bz_conv c = *cv;
    bz_status st = bz_conv_shape(&c);
    if (st != BZ_OK) return st;
    if (c.ho != cv->ho || c.wo != cv->wo) return BZ_ERR_ARG;
    return BZ_OK;
}

static bz_status done(hipError_t e) { return e == hipSuccess ? BZ_OK : BZ_ERR_HIP; }

bz_status bz_conv_fwd(const bz_conv *cv, const uint16_t *x, const uint16_t *w, const float *bias,
                      int32_t relu, float *y, uint16_t *y_bf16, hipStream_t s) {
    bz_status st = check_conv(cv);
    if (st != BZ_OK) return st;
    if (!x || !w || (!y && !y_bf16) || (relu != 0 && relu != 1)) return BZ_ERR_ARG;
    (void)hipGetLastError();
    return done(launch_conv_fwd(*cv, x, w, bias, relu, y, y_bf16, s));
}

bz_status bz_conv_bwd_data(const bz_conv *cv, const float *dy, const uint16_t *w,
                           const uint16_t *x_mask, float *dx, hipStream_t s) {
    bz_status st = check_conv(cv);
    if (st != BZ_OK) return st;
    if (!dy || !w || !dx) return BZ_ERR_ARG;
    (void)hipGetLastError();
    return done(launch_conv_bwd_data(*cv, dy, w, x_mask, dx, s));
}

bz_status bz_conv_bwd_weight(const bz_conv *cv, const float *dy, const uint16_t *x, float *dw,
                             float *db, hipStream_t s) {
    bz_status st = check_conv(cv);
    if (st != BZ_OK) return st;
    if (!dy || !x || !dw) return BZ_ERR_ARG;
    (void)hipGetLastError();
    return done(launch_conv_bwd_weight(*cv, dy, x, dw, db, false, s));
}

bz_status bz_conv_bwd_weight_add(const bz_conv *cv, const float *dy, const uint16_t *x, float *dw,
                                 float *db, hipStream_t s) {
    bz_status st = check_conv(cv);
    if (st != BZ_OK) return st;
    if (!dy || !x || !dw) return BZ_ERR_ARG;
    (void)hipGetLastError();
    return done(launch_conv_bwd_weight(*cv, dy, x, dw, db, true, s));
}

bz_status bz_decode(const float *z, int64_t n_curves, int32_t per, int32_t points, float scale,
                    float shift, float *out, hipStream_t s) {
    if (n_curves < 0 || per < 1 || points < 0 || points > per) return BZ_ERR_ARG;
    if (n_curves == 0) return BZ_OK;
    if (!z || !out) return BZ_ERR_ARG;
    if (n_curves >= (int64_t(1) << 40) / per) return BZ_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    const int64_t n = n_curves * per, b = cdiv(n, 256);
    hipLaunchKernelGGL(k_decode, dim3((unsigned)(b < 8192 ? b : 8192)), dim3(256), 0, s, z, n, per,
                       points, scale, shift, out);
    return done(hipGetLastError());
}

bz_status bz_pad_channels(const uint16_t *src, int64_t n_pix, int32_t c, uint16_t *dst,
                          hipStream_t s) {
    if (n_pix < 0 || c < 1 || c > 8) return BZ_ERR_ARG;
    if (n_pix == 0) return BZ_OK;
    if (!src || !dst || ((uintptr_t)dst & 15)) return BZ_ERR_ARG;
    if (n_pix >= (int64_t(1) << 40)) return BZ_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    const int64_t b = cdiv(n_pix, 256);
    hipLaunchKernelGGL(k_pad8, dim3((unsigned)(b < 8192 ? b : 8192)), dim3(256), 0, s, src, n_pix, c,
                       reinterpret_cast<uint4 *>(dst));
    return done(hipGetLastError());
}

bz_status bz_f32_to_bf16(const float *src, uint16_t *dst, int64_t n, hipStream_t s) {
    if (n < 0 || (n > 0 && (!src || !dst))) return BZ_ERR_ARG;
    (void)hipGetLastError();
    return done(launch_to_bf16(src, dst, n, s));
}

bz_status bz_extract_patches(const float *image, int32_t width, int32_t height, const int32_t *xy,
                             int32_t n_patch, int32_t side, float fill, uint16_t *out,
                             hipStream_t s) {
    if (width < 1 || height < 1 || n_patch < 0 || side < 1 || side > 4096) return BZ_ERR_ARG;
    if (n_patch > 0 && (!image || !xy || !out)) return BZ_ERR_ARG;
    if ((int64_t)side * side * 3 * n_patch >= (int64_t(1) << 40)) return BZ_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    return done(launch_patches(image, width, height, xy, n_patch, side, fill, out, s));
}

}  // extern "C"
