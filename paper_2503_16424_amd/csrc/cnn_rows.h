// cnn_rows.h -- index arithmetic of the convolutions: the parity classes of the input
// gradient, and which slice of which pixel a lane of k_conv_rows reads.  Plain integer
// code without the runtime's headers, so that every address can also be enumerated on
// the host.
#ifndef BZ_CNN_ROWS_H
#define BZ_CNN_ROWS_H

#include <stdint.h>

namespace bz {

namespace {

struct Shape {
    int n, h, w, c, k, r, s, p, ho, wo;
};

enum Mode { kFwd = 0, kBwdData = 1, kBwdWeight = 2 };

struct GemmArgs {
    Shape S;
    int M, N, K;          // GEMM sizes
    const uint16_t *x;        // input activations (bf16)
    const uint16_t *w;        // filters (bf16)
    const float *dy;          // output gradients (f32)
    const float *bias;
    const uint16_t *mask;     // bwd data: zero where the layer input is <= 0
    int relu;
    float *out_f;             // fwd y, bwd-data dx, bwd-weight dw
    uint16_t *out_b;          // fwd y in bf16
    int k_chunk;          // bwd weight: k range per workgroup
    // bwd data, one parity class: rows are the input pixels (iy, ix) with
    // iy = cy, ix = cx (mod stride), hq x wq of them per image; only taps
    // ky = ky0, kx = kx0 (mod stride) reach them, nkx of them along x
    int cy, cx, hq, wq, ky0, kx0, nkx;
};

// Input gradient: the parity class of workgroup row z (cy = z / stride,
// cx = z mod stride), its GEMM rows M and its k extent K.
__host__ __device__ inline void set_class(GemmArgs &g, int z) {
    const Shape &S = g.S;
    const int st = S.s;
    g.cy = z / st;
    g.cx = z - (z / st) * st;
    g.hq = g.cy < S.h ? (S.h - g.cy + st - 1) / st : 0;
    g.wq = g.cx < S.w ? (S.w - g.cx + st - 1) / st : 0;
    g.ky0 = (g.cy + S.p) % st;
    g.kx0 = (g.cx + S.p) % st;
    const int nky = g.ky0 < S.r ? (S.r - g.ky0 + st - 1) / st : 0;
    const int nkx = g.kx0 < S.r ? (S.r - g.kx0 + st - 1) / st : 0;
    g.nkx = nkx > 0 ? nkx : 1;                  // no taps: K = 0, the class gets zeros
    g.M = (int)S.n * g.hq * g.wq;
    g.K = (int)nky * nkx * S.k;
}

struct ConvTab {
    int off;              // elements from the pixel's base to the slice
    int16_t dy, dx;       // rows and columns from it (bounds test)
};

// A parity class (forward: the only one): its steps of 32 k and where they start.
struct ConvClass {
    int first, steps, cy, cx;
};

// The slice at class k `k` of g's current class, relative to the pixel's base.
template <int MODE>
__host__ __device__ inline ConvTab conv_tab(const GemmArgs &g, int k) {
    const Shape &S = g.S;
    ConvTab e;
    const int sc = MODE == kFwd ? S.c : S.k;
    const int j = k / sc, ch = k - j * sc;
    if (MODE == kFwd) {
        const int ky = j / S.r, kx = j - ky * S.r;
        e.dy = (int16_t)ky;
        e.dx = (int16_t)kx;
        e.off = (ky * S.w + kx) * S.c + ch;
    } else {
        const int y = j / g.nkx, x = j - y * g.nkx;
        const int dy = (g.cy + S.p - g.ky0) / S.s - y, dx = (g.cx + S.p - g.kx0) / S.s - x;
        e.dy = (int16_t)dy;
        e.dx = (int16_t)dx;
        e.off = (dy * S.wo + dx) * S.k + ch;
    }
    if (k >= g.K) e.dy = 0x4000;                // no such slice: see conv_reads
    return e;
}

// Steps of 32 k.
__host__ __device__ inline int conv_steps(int K) { return (K + 31) / 32; }

// 16-byte pieces of nc output channels of a pixel (2 bytes each forward, 4 backward), for
// blocks that store through LDS.  At least 1: a forward block of 4 channels has no whole
// piece and stores its sums directly, but its lanes' places are divided all the same.
template <int MODE>
__host__ __device__ inline int conv_pieces(int nc) {
    const int pieces = nc / (MODE == kFwd ? 8 : 4);
    return pieces > 0 ? pieces : 1;
}

// Division of 0 <= m < 2^31 by d >= 1 without a divide per tile (Granlund and
// Montgomery 1994): with 2^(s-1) < d <= 2^s and mul = ceil(2^(31+s) / d) < 2^32,
// m / d = (m * mul) >> (31 + s).
struct Divisor {
    uint32_t d, mul;
    int sh;
};

__host__ __device__ inline Divisor divisor(int d) {
    const int s = d > 1 ? 32 - __builtin_clz(d - 1) : 1;
    return Divisor{(uint32_t)d, (uint32_t)(((1ull << (31 + s)) + d - 1) / (unsigned)d), s - 1};
}

__host__ __device__ inline int divide(int m, const Divisor &v) {
    return v.d == 1 ? m : (int)((((uint64_t)(uint32_t)m * v.mul) >> 32) >> v.sh);
}

// Rows of a tensor as k_conv_rows divides them: output pixels, or blocks of stride x
// stride input pixels, per image and per line; tiles of 16.
template <int MODE>
__host__ __device__ inline Divisor conv_image(const Shape &S) {
    return divisor(MODE == kFwd ? S.ho * S.wo : ((S.h + S.s - 1) / S.s) * ((S.w + S.s - 1) / S.s));
}
template <int MODE>
__host__ __device__ inline Divisor conv_line(const Shape &S) {
    return divisor(MODE == kFwd ? S.wo : (S.w + S.s - 1) / S.s);
}
__host__ __device__ inline int conv_tiles(const Shape &S, const Divisor &image) {
    return (int)(((int64_t)S.n * image.d + 15) / 16);
}

// One row tile as a wave reads it: this lane's output pixel, or its block of
// stride x stride input pixels, one of each class (input gradient).
struct ConvRow {
    int base, y0, x0, b;
};

template <int MODE>
__host__ __device__ inline ConvRow conv_row(const GemmArgs &g, const Divisor &image,
                                            const Divisor &line, int tile, int j) {
    const Shape &S = g.S;
    ConvRow r;
    const int m = tile * 16 + j;
    r.b = divide(m, image);
    const int rem = m - r.b * (int)image.d;
    const int ry = divide(rem, line), rx = rem - ry * (int)line.d;
    r.y0 = MODE == kFwd ? ry * S.s - S.p : ry;
    r.x0 = MODE == kFwd ? rx * S.s - S.p : rx;
    r.base = MODE == kFwd ? ((r.b * S.h + r.y0) * S.w + r.x0) * S.c
                          : ((r.b * S.ho + ry) * S.wo + rx) * S.k;
    if (r.b >= S.n) r.y0 = 0x4000;              // no such row: see conv_reads
    return r;
}

// Whether the lane's pixel has the slice.  A slice past K and a row past the last
// image carry 0x4000 in their y: row and slice offsets are otherwise at least -2 and a
// side is below 0x2000 + 8, so one marker alone is out of the bound, and two add up
// further out (markers of opposite signs would cancel).
template <int MODE>
__host__ __device__ inline bool conv_reads(const Shape &S, const ConvRow &r, const ConvTab &e) {
    const int sh = MODE == kFwd ? S.h : S.ho, sw = MODE == kFwd ? S.w : S.wo;
    return (unsigned)(r.y0 + e.dy) < (unsigned)sh && (unsigned)(r.x0 + e.dx) < (unsigned)sw;
}

// The pixel that the lane's sums belong to, or -1.
template <int MODE>
__host__ __device__ inline int conv_out(const GemmArgs &g, const ConvRow &r, int tile, int j,
                                        const ConvClass &cls) {
    const Shape &S = g.S;
    if (r.b >= S.n) return -1;
    if (MODE == kFwd) return tile * 16 + j;
    const int iy = r.y0 * S.s + cls.cy, ix = r.x0 * S.s + cls.cx;
    return iy < S.h && ix < S.w ? (r.b * S.h + iy) * S.w + ix : -1;
}

}  // namespace

}  // namespace bz

#endif
