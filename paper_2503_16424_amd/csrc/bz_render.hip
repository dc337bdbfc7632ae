// bz_render.hip -- per-tile blending (Sec. 3.4) and its reverse pass.
//
// Work decomposition (forward and backward stage 1): one workgroup per tile,
// one wave per 8x8 pixel quad of the tile; in the forward one pixel per lane, in
// the backward one list entry and a quarter of the pixels (BwdWave).  Waves are
// independent: each walks its tile's list in batches of 64 entries; lane j
// loads entry j's record, tests the entry's truncated support against the
// quad (exact minimum of the quadratic form over the quad's pixel centres),
// and writes the derived per-Gaussian constants into the wave's LDS slice.
// A ballot of the test gives the batch's mask; the wave then iterates only
// over the surviving entries, every lane reading the entry's constants from
// the same LDS address (three 16-byte reads), so pixels never spend ALU on
// Gaussians that cannot reach their quad.  A wave stops when all 64 of its pixels have terminated.  (In the
// backward the quads of a tile also share a sum table in LDS, so its waves
// meet at the tile's start and end.)
//
// Blocks are mapped to tiles in runs per XCD: the dispatcher deals blocks
// round robin to the 8 XCDs, so block b runs on XCD b mod 8; each XCD takes
// runs of consecutive tiles in turn (xcd_tile), so its L2 sees neighbouring
// tiles, which share most of their Gaussians, and dense and empty parts of a
// canvas or batch are spread over all of them.
//
// The forward can also write the L2 loss gradient of Sec. 3.5 as it writes
// each pixel (k_fwd_l2), which spares the step a pass over the image.
//
// Stage 2 of the backward pass is per curve (one workgroup per curve: 64
// threads for curves of at most 64 Gaussians, 256 for larger ones, part of a
// wave for short curves in large sets; no atomics): it chains the per-Gaussian gradients through the sampling of
// Sec. 3.3.
#include <cstddef>

#include "bz_geom.h"

namespace bz {

namespace {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Tile of workgroup b: the XCDs (b mod 8) take runs of `run` consecutive tiles
// in turn.
__device__ inline int xcd_tile(int b, int run) {
    const int i = b >> 3, c = i / run;
    return (8 * c + (b & 7)) * run + (i - c * run);
}

// Longest run.  One band of consecutive tiles per XCD left the XCD with the
// densest band working alone at the end: with runs of 32 the backward takes 596
// instead of 770 us on 16 uneven canvases (the forward 271, 347), 100 instead of
// 126 on a 512x512 scene and 1,030 instead of 1,075 on the 2048x2048 frame.  Runs
// of 4 to 32 differ by 2%, 128 gave back a third of the batch's gain.  Few tiles: runs
// short enough for eight of them on every XCD.
constexpr int kXcdRun = 32;

// Minimum over the box [x0,x1]x[y0,y1] (offsets from the mean) of
// f(d) = qa dx^2 + 2 qb dx dy + qc dy^2, compared against thr.
__device__ inline bool box_hit(float x0, float x1, float y0, float y1, float qa, float qb,
                               float qc, float thr) {
    if (x0 <= 0.f && x1 >= 0.f && y0 <= 0.f && y1 >= 0.f) return true;
    float best = 3.0e38f;
    // hardware reciprocals: an error in the clamped edge point moves the value
    // of the quadratic form only to second order (the slack on thr covers it)
    float ia = __builtin_amdgcn_rcpf(qa), ic = __builtin_amdgcn_rcpf(qc);
    // vertical edges: dx fixed, minimise over dy
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        float dx = e ? x1 : x0;
        float dy = fminf(fmaxf(-qb * dx * ic, y0), y1);
        best = fminf(best, qa * dx * dx + 2.f * qb * dx * dy + qc * dy * dy);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        float dy = e ? y1 : y0;
        float dx = fminf(fmaxf(-qb * dy * ia, x0), x1);
        best = fminf(best, qa * dx * dx + 2.f * qb * dx * dy + qc * dy * dy);
    }
    return best <= thr;
}

struct TileArgs {
    const float4 *rec;
    const uint32_t *ids;
    const uint32_t *ranges;
    const int64_t *status;
    int W, H, tile_w, tile_h, tiles_x, n_tiles, xcd_run, quads_x;
    float bg0, bg1, bg2;
    float g_min, alpha_max, t_min, inv_1mg, box_thr;
    float *image;
    float *t_final;
    uint32_t *n_last;
    uint32_t *n_contrib;
    uint64_t *visit;          // per (quad plane, tile batch) contribution masks
    int64_t words_per_plane;
    const bz_canvas *canvas;  // batch canvases (null: one canvas W x H)
    int n_canvas;
    uint32_t *counter;        // persistent launch: next tile (null: one workgroup per tile)
    int tab_cap;              // positions of the backward's per-tile sum table
    // backward
    const float *d_image;
    float *d_gauss;           // 9 planes of n_gauss, or (packed) 9 floats per Gaussian
    bool packed;
    int64_t n_gauss;
    // forward with the L2 loss gradient: target, d_image out, loss sum, scale
    const float *l2_target;
    float *l2_grad;
    float *l2_loss;
    int64_t l2_min_pairs;     // from so many pairs the blocks add to l2_loss themselves
    float l2_scale;
};

// Entry of the wave's LDS slice.  The shape as two scaled axis vectors: with
// e' = e sqrt(log2(e) / 2) and f = k e', the base-2 exponent of the kernel at
// offset d = pixel - mean is p2 = u^2 + w^2, u = e' . d, w = f x d (= f.x dy
// - f.y dx), a sum of two squares.  The mean is taken relative to the quad's
// first pixel centre (qx0, qy0): the record's mean is hi + lo and hi - qx0 is
// exact for any Gaussian near the quad, so the relative mean m' is rounded
// once, and a pixel's offset is its place in the quad l (0..7 in x and y)
// minus m'.
// - With u0 = e' . m' and w0 = f x m' staged, u = e' . l - u0 and
//   w = f x l - w0 cost two FMAs each and no offsets.
// - The reverse pass stages the same form relative to the tile centre, with l
//   the pixel centre from it.
struct Staged {
    float4 m;   // -u0, -w0, e'.x, e'.y
    float4 q;   // f.x, f.y, k, o' = o / (1 - g_min)
    float4 c;   // r, g, b, o' * g_min
};

// sqrt(log2(e) / 2): scales the record's axis e so that the squares sum to p2.
constexpr float kHalfLog2eSqrt = 0.84932180028801907f;

// Load a record and compute its LDS constants.  q receives the record's shape
// (e.x, e.y, k, o), mean the relative mean m'.
__device__ inline void stage_record(const TileArgs &a, uint32_t id, float qx0, float qy0,
                                    Staged &st, float4 &q, float2 &mean) {
    const float4 m = a.rec[3 * (int64_t)id];
    q = a.rec[3 * (int64_t)id + 1];
    const float4 c = a.rec[3 * (int64_t)id + 2];
    const float op = q.w * a.inv_1mg;
    const float ex = kHalfLog2eSqrt * q.x, ey = kHalfLog2eSqrt * q.y;
    const float fx = q.z * ex, fy = q.z * ey;
    const float mx = (m.x - qx0) + m.z, my = (m.y - qy0) + m.w;
    const float nu0 = -fmaf(ex, mx, ey * my);      // -(e' . m')
    const float nw0 = -fmaf(fx, my, -fy * mx);     // -(f x m')
    st.m = make_float4(nu0, nw0, ex, ey);
    st.q = make_float4(fx, fy, q.z, op);
    st.c = make_float4(c.x, c.y, c.z, op * a.g_min);
    mean = make_float2(mx, my);
}

// Load a tile-list entry, compute its LDS constants and test its support
// against the wave's 8x8 quad (first pixel centre qx0, qy0).
__device__ inline bool stage_entry(const TileArgs &a, uint32_t id, float qx0, float qy0,
                                   Staged &st) {
    float4 q;
    float2 m;
    stage_record(a, id, qx0, qy0, st, q, m);
    // offsets of the quad's first pixel centre from the mean
    const float x0 = -m.x, y0 = -m.y;
    float qxx, qxy, qyy;
    shape_conic(q.x, q.y, q.z, qxx, qxy, qyy);
    return box_hit(x0, x0 + 7.f, y0, y0 + 7.f, qxx, qxy, qyy, a.box_thr);
}

// The test of stage_entry with the mean relative to the tile centre (ox, oy), the
// quad's first pixel centre at (bx, by) from it.
__device__ inline bool entry_hit_bwd(const TileArgs &a, uint32_t id, float ox, float oy, float bx,
                                     float by) {
    const float4 m = a.rec[3 * (int64_t)id], q = a.rec[3 * (int64_t)id + 1];
    const float x0 = bx - ((m.x - ox) + m.z), y0 = by - ((m.y - oy) + m.w);
    float qxx, qxy, qyy;
    shape_conic(q.x, q.y, q.z, qxx, qxy, qyy);
    return box_hit(x0, x0 + 7.f, y0, y0 + 7.f, qxx, qxy, qyy, a.box_thr);
}

// Base-2 exponent p2 = (e' . d)^2 + (f x d)^2 of a staged entry at the
// pixel centre (lx, ly) from the staging origin.
__device__ inline float exponent2(const Staged &st, float lx, float ly) {
    const float u = fmaf(st.m.z, lx, fmaf(st.m.w, ly, st.m.x));
    const float w = fmaf(st.q.x, ly, fmaf(-st.q.y, lx, st.m.y));
    return fmaf(u, u, w * w);
}

// Word of the visit mask of batch k of tile t inside one quad plane: tile t's
// batches occupy [start_t / 64 + t, start_t / 64 + t + ceil(len_t / 64)), which
// never overlaps the next tile's range, so every word has one writer.
__device__ inline int64_t visit_word(uint32_t start, int tile) {
    return (int64_t)(start >> 6) + tile;
}

// Canvas geometry of a (wave-uniform) global tile.
struct TileGeo {
    int W, H;          // canvas size
    int tx, ty;        // tile coordinates inside the canvas
    int64_t pix0;      // first pixel of the canvas
    float bg0, bg1, bg2;
};

__device__ inline TileGeo tile_geo(const TileArgs &a, int tile) {
    TileGeo g;
    if (a.canvas) {
        const int c = batch_find(a.canvas, a.n_canvas, (int64_t)tile,
                                 [](const bz_canvas &r) { return r.tile_off; });
        const bz_canvas &cv = a.canvas[c];
        const int local = tile - (int)cv.tile_off;
        g.W = cv.width;
        g.H = cv.height;
        g.ty = local / cv.tiles_x;
        g.tx = local - g.ty * cv.tiles_x;
        g.pix0 = cv.pix_off;
        g.bg0 = cv.bg[0];
        g.bg1 = cv.bg[1];
        g.bg2 = cv.bg[2];
    } else {
        g.W = a.W;
        g.H = a.H;
        g.ty = tile / a.tiles_x;
        g.tx = tile - g.ty * a.tiles_x;
        g.pix0 = 0;
        g.bg0 = a.bg0;
        g.bg1 = a.bg1;
        g.bg2 = a.bg2;
    }
    return g;
}

// Tile loop of a launch: one tile per workgroup (xcd_tile), or, when
// the launch is persistent, tiles taken from a counter until they run out.
template <typename Body>
__device__ inline void for_tiles(const TileArgs &a, Body body) {
    if (!a.counter) {
        const int tile = xcd_tile(blockIdx.x, a.xcd_run);
        if (tile < a.n_tiles) body(tile);
        return;
    }
    __shared__ int s_next;
    for (;;) {
        __syncthreads();                        // the previous tile is done with LDS
        if (threadIdx.x == 0) s_next = (int)atomicAdd(a.counter, 1u);
        __syncthreads();
        const int tile = __builtin_amdgcn_readfirstlane(s_next);
        if (tile >= a.n_tiles) break;
        body(tile);
    }
}

// min(x, hi) for finite x and a wave-uniform hi, as one VALU instruction:
// fminf would canonicalise both operands first (IEEE mode), two more per use.
__device__ inline float min_amax(float x, float hi) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "s"(hi), "v"(x));
    return r;
}

// Per lane: bit `lane` of the wave-uniform mask m ? on : off, as one
// v_cndmask with m in scalar registers (a bool built from m would cost a shift,
// an and and a compare per lane).
__device__ inline float select_lanes(uint64_t m, float on, float off) {
    float r;
    asm("v_cndmask_b32_e64 %0, %2, %1, %3" : "=v"(r) : "v"(on), "v"(off), "s"(m));
    return r;
}
__device__ inline uint32_t select_lanes_u32(uint64_t m, uint32_t on, uint32_t off) {
    return __float_as_uint(select_lanes(m, __uint_as_float(on), __uint_as_float(off)));
}

// Clear bit b of a wave-uniform mask: one scalar instruction (the compiler's
// mask & (mask - 1) or mask & ~(1 << b) take two or three).
__device__ inline void clear_bit(uint64_t &mask, int b) {
    asm("s_bitset0_b64 %0, %1" : "+s"(mask) : "s"(b));
}

// A wave-uniform float moved to a scalar register.
__device__ inline float uniform_f32(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// A staged record as three 16-byte LDS reads (the compiler splits the read
// around fields the sweep leaves unused, five LDS instructions), waited for
// in the same block; off is the record's LDS byte offset (the low 32 bits
// of a flat address into LDS).  The outputs are early-clobber: the address
// register must not be shared with a destination while later reads use it.
__device__ inline Staged read_staged_at(uint32_t off) {
    float4 m, q, c;
    asm volatile("ds_read_b128 %0, %3\n\t"
                 "ds_read_b128 %1, %3 offset:16\n\t"
                 "ds_read_b128 %2, %3 offset:32\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(m), "=&v"(q), "=&v"(c)       // early clobber: off is read by all three
                 : "v"(off)
                 : "memory");
    return Staged{m, q, c};
}

// LDS offset of entry b of a wave's staged slice (base: the slice's offset,
// held in a vector register) as one VALU multiply-add from the scalar index:
// the compiler's scalar multiply, add and move to a vector register cost two
// scalar instructions more per visited entry.
// The slice's offset in a vector register, produced once: an inline-asm
// value is kept in its register rather than moved back from a scalar one
// inside the loop.
__device__ inline uint32_t vector_copy(uint32_t v) {
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}
__device__ inline uint32_t staged_off(uint32_t base, int b) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, 48, %2" : "=v"(r) : "s"(b), "v"(base));
    return r;
}

// Result of a front-to-back sweep for one pixel.
struct Sweep {
    float T, C0, C1, C2;   // transmittance after the last contributor, colour sum
    uint32_t last;         // list positions the reverse pass must consider (see below)
    uint32_t cnt;          // contributors (kCount only)
};

// Front-to-back blend (Sec. 3.4) of one wave's 8x8 quad over tile-list
// positions [start, end): per batch of 64 entries, every lane stages one entry
// into the wave's LDS slice and box-tests it against the quad; the wave then
// visits the hits in list order.  Per pixel and hit: alpha = min(alpha_max,
// o (G - g_min) / (1 - g_min)) when G > g_min, colour += alpha T c, T *= 1 - alpha;
// a pixel stops after the first contributor that takes T below t_min, and the
// wave leaves when all its pixels have stopped.  sink(k, bits) receives, for
// batch k, the entries that changed at least one pixel of the quad.
//
// A pixel has stopped exactly when T < t_min (T never grows; lanes outside the
// canvas start at T = -1), so the wave keeps that set as one 64-bit mask.
// last: for a pixel that stopped, 1 + the list position of the contributor
// that stopped it; otherwise the end of the last batch that changed a pixel of
// the quad (capped at the list length).  Either way no entry at or beyond it
// contributed to the pixel, and every earlier entry with G > g_min did, which
// is all the reverse pass needs; recording it costs the loop nothing except
// when a pixel stops.
template <bool kColor, bool kCount, typename Sink>
__device__ inline Sweep fwd_sweep(const TileArgs &a, Staged *my, uint32_t start, uint32_t end,
                                  float lx, float ly, float qx0, float qy0, bool valid, int lane,
                                  Sink sink) {
    Sweep r = {valid ? 1.f : -1.f, 0.f, 0.f, 0.f, 0u, 0u};
    const float g_min = a.g_min, amax = a.alpha_max, tmin = a.t_min;
    uint64_t stopped = __builtin_amdgcn_ballot_w64(r.T < tmin);
    uint32_t k = 0, k_used = 0;
    const uint32_t my_off = vector_copy((uint32_t)(uintptr_t)my);   // LDS offset of the slice
    for (uint32_t base = start; base < end; base += 64, ++k) {
        const uint32_t j = base + lane;
        bool hit = false;
        if (j < end) {
            Staged st;
            hit = stage_entry(a, a.ids[j], qx0, qy0, st);
            my[lane] = st;
        }
        uint64_t mask = __ballot(hit);
        // the batch's entries that change a pixel: every hit, less the
        // (rarer) ones that change none
        uint64_t vbits = mask;
        wave_lds_sync();
        while (mask) {
            const int b = __builtin_ctzll(mask);
            clear_bit(mask, b);
            const Staged st = read_staged_at(staged_off(my_off, b));
            const float G = __builtin_amdgcn_exp2f(-exponent2(st, lx, ly));
            // contributors: inside the support and not stopped, as a lane mask
            const uint64_t cm = __builtin_amdgcn_ballot_w64(G > g_min) & ~stopped;
            const float araw = fmaf(st.q.w, G, -st.c.w);
            const float al = select_lanes(cm, min_amax(araw, amax), 0.f);
            const float wgt = al * r.T;
            if (kColor) {
                r.C0 = fmaf(wgt, st.c.x, r.C0);
                r.C1 = fmaf(wgt, st.c.y, r.C1);
                r.C2 = fmaf(wgt, st.c.z, r.C2);
            }
            {
                // T (1 - alpha) as T - wgt, after wgt has used T: no copy of T
                _Pragma("clang fp contract(off)") r.T = r.T - wgt;
            }
            if (kCount) r.cnt = select_lanes_u32(cm, r.cnt + 1u, r.cnt);
            if (__builtin_expect(cm == 0, 0)) clear_bit(vbits, b);
            const uint64_t now = __builtin_amdgcn_ballot_w64(r.T < tmin);
            if (__builtin_expect(now != stopped, 0)) {     // some pixel stopped here
                r.last = select_lanes_u32(now & ~stopped, k * 64 + b + 1, r.last);
                stopped = now;
            }
        }
        if (vbits) k_used = k + 1;
        sink(k, vbits);
        if (stopped == ~0ull) break;
        wave_lds_sync();
    }
    r.last = select_lanes_u32(stopped, r.last, min(k_used * 64u, end - start));
    return r;
}

// Forward pass.  With kState the blend state the backward reads is written:
// T after the last contributor, a bound on its position, and per (quad, batch) the mask
// of entries that contributed; without it only the image.  With kL2, as each
// pixel is written, also the L2 loss gradient scale * (image - target) (the
// same float arithmetic as k_l2) and the lane's sum of squared errors in l2.
template <bool kState, bool kCount, bool kL2>
__device__ inline void fwd_tile(const TileArgs &a, int tile, float &l2) {
    extern __shared__ Staged s_stage[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const TileGeo tg = tile_geo(a, tile);
    const int qx = w % a.quads_x, qy = w / a.quads_x;
    const int x0 = tg.tx * a.tile_w + qx * kQuad, y0 = tg.ty * a.tile_h + qy * kQuad;
    if (x0 >= tg.W || y0 >= tg.H) return;
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    const bool valid = x < tg.W && y < tg.H;
    const float lx = (float)(lane & 7), ly = (float)(lane >> 3);   // pixel - first pixel of the quad
    // wave-uniform: held in scalar registers
    const float qx0 = uniform_f32((float)x0 + 0.5f), qy0 = uniform_f32((float)y0 + 0.5f);
    Staged *my = s_stage + w * 64;

    const int64_t pix = tg.pix0 + (int64_t)y * tg.W + x;
    const int64_t plane = (int64_t)tg.W * tg.H;
    float *img = a.image + 2 * tg.pix0;     // canvas image: 3 planes from 3 * pix0
    if (a.status[1] & Status::kOverflow) {
        if (valid) {
            float nan = __int_as_float(0x7fc00000);
            img[pix] = nan;
            img[plane + pix] = nan;
            img[2 * plane + pix] = nan;
            if (kL2) {
                float *dimg = a.l2_grad + 2 * tg.pix0;
                dimg[pix] = nan;
                dimg[plane + pix] = nan;
                dimg[2 * plane + pix] = nan;
                l2 = nan;
            }
            if (kState) {
                a.t_final[pix] = nan;
                a.n_last[pix] = 0;
                if (kCount) a.n_contrib[pix] = 0;
            }
        }
        return;
    }
    const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
    uint64_t *vis = kState ? a.visit + (int64_t)w * a.words_per_plane + visit_word(start, tile)
                           : nullptr;
    const Sweep r = fwd_sweep<true, kCount>(a, my, start, end, lx, ly, qx0, qy0, valid, lane,
                                            [&](uint32_t k, uint64_t bits) {
                                                if (kState && lane == 0) vis[k] = bits;
                                            });
    if (valid) {
        const float v0 = fmaf(r.T, tg.bg0, r.C0), v1 = fmaf(r.T, tg.bg1, r.C1),
                    v2 = fmaf(r.T, tg.bg2, r.C2);
        img[pix] = v0;
        img[plane + pix] = v1;
        img[2 * plane + pix] = v2;
        if (kL2) {
            const float *tgt = a.l2_target + 2 * tg.pix0;
            float *dimg = a.l2_grad + 2 * tg.pix0;
            const float e0 = v0 - tgt[pix], e1 = v1 - tgt[plane + pix],
                        e2 = v2 - tgt[2 * plane + pix];
            dimg[pix] = a.l2_scale * e0;
            dimg[plane + pix] = a.l2_scale * e1;
            dimg[2 * plane + pix] = a.l2_scale * e2;
            l2 = fmaf(e0, e0, fmaf(e1, e1, fmaf(e2, e2, l2)));
        }
        if (kState) {
            a.t_final[pix] = r.T;
            a.n_last[pix] = r.last;
            if (kCount) a.n_contrib[pix] = r.cnt;
        }
    }
}

// Forward pass.  With kState the blend state the backward reads is written:
// T after the last contributor, a bound on its position, and per (quad, batch) the mask
// of entries that contributed; without it only the image.
template <bool kState, bool kCount>
__global__ __launch_bounds__(1024) void k_fwd(TileArgs a) {
    float unused = 0.f;
    for_tiles(a, [&](int tile) { fwd_tile<kState, kCount, false>(a, tile, unused); });
}

// Sum over the wave's 64 lanes, wave-uniform: an inclusive DPP scan (row
// shifts of 1, 2, 4, 8 lanes with zeros shifted in, then row_bcast 15 and 31
// across rows), whose last lane holds the total.
template <int CTRL, int ROWS, bool BOUND>
__device__ inline float dpp_f32(float x) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xF, BOUND));
}
__device__ inline float wave_sum(float v) {
    v += dpp_f32<0x111, 0xF, true>(v);
    v += dpp_f32<0x112, 0xF, true>(v);
    v += dpp_f32<0x114, 0xF, true>(v);
    v += dpp_f32<0x118, 0xF, true>(v);
    v += dpp_f32<0x142, 0xA, false>(v);
    v += dpp_f32<0x143, 0xC, false>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The forward with the L2 loss gradient.  Every lane sums its squared errors
// over the block's tiles; the block's waves add their sums in LDS and the last
// one out adds the block's total to the loss, one global atomic per block (or,
// with fewer than l2_min_pairs pairs, a pass of its own over image and target
// sums the loss afterwards).  Every wave of the block reaches the end exactly once (waves outside the
// canvas leave fwd_tile early, not the kernel).
template <bool kState, bool kCount>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_fwd_l2(TileArgs a) {
    __shared__ float s_loss;
    __shared__ int s_done;
    if (threadIdx.x == 0) {
        s_loss = 0.f;
        s_done = 0;
    }
    __syncthreads();
    float l2 = 0.f;
    for_tiles(a, [&](int tile) { fwd_tile<kState, kCount, true>(a, tile, l2); });
    if (!a.l2_loss || a.status[0] < a.l2_min_pairs) return;
    l2 = wave_sum(l2);
    if ((threadIdx.x & 63) == 0) {
        __hip_atomic_fetch_add(&s_loss, l2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int waves = (int)(blockDim.x >> 6);
        if (__hip_atomic_fetch_add(&s_done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) ==
            waves - 1) {
            const float total =
                __hip_atomic_load(&s_loss, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (total != 0.f) atomicAdd(a.l2_loss, total);
        }
    }
}

// A lane's 64-bit value as a wave-uniform (scalar) one.  The builtin returns a
// signed int: each half goes through uint32_t so that the low half is
// zero-extended, not sign-extended into the high word.
__device__ inline uint64_t lane_u64(uint64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | (uint64_t)lo;
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

// Inclusive scans over the 16 lanes of each row, of 4 registers at once: four
// DPP row shifts, in place; a lane without a source is left as it is, which is
// the identity for product and sum alike.  The steps of the four registers
// alternate, so a DPP read comes three instructions after the write it
// depends on (two are required); the leading s_nop covers the inputs.
#define BZ_ROW_SCAN4(OP, v)                                                             \
    asm("s_nop 1\n\t"                                                                   \
        OP " %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %1, %1, %1 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %2, %2, %2 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %3, %3, %3 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %1, %1, %1 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %2, %2, %2 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %3, %3, %3 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %1, %1, %1 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %2, %2, %2 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %3, %3, %3 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %1, %1, %1 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %2, %2, %2 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"                       \
        OP " %3, %3, %3 row_shr:8 row_mask:0xf bank_mask:0xf"                           \
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]))

// v[lane] = v[lane - 1] * f[lane] for the row's lanes 1, 2, .. 15 in turn (4 registers
// at once): a product taken strictly in order from the row's first lane, whose v is
// left as it is.  Every step runs in all lanes; the k-th is final for lane k.
#define BZ_ROW_MUL_STEP4(v, f)                                                          \
    asm("s_nop 1\n\t"                                                                   \
        "v_mul_f32_dpp %0, %0, %4 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"             \
        "v_mul_f32_dpp %1, %1, %5 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"             \
        "v_mul_f32_dpp %2, %2, %6 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"             \
        "v_mul_f32_dpp %3, %3, %7 row_shr:1 row_mask:0xf bank_mask:0xf"                 \
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3])                                \
        : "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]))

// v of the lane before in the row of 16; the row's first lane gets `first`.
__device__ inline float row_shifted(float first, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v),
                                                      0x111, 0xF, 0xF, false));
}

// A constant or wave-uniform float in a vector register: an FMA, add or
// multiply with an operand in a scalar register takes 4 cycles on this part,
// with all operands in vector registers (or inline constants) 2.5.
__device__ inline float vector_f32(float v) {
    float r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}

// min(a, b) of finite values, both in vector registers, as one instruction
// (fminf canonicalises its operands first).
__device__ inline float min_f32(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The reverse pass of one wave (an 8x8 quad, 64 pixels) takes 16 list entries
// ("slots") at a time.  Lane (q = l / 16, j = l mod 16) works on slot j and a
// quarter of the pixels: register r of block b = 0..3 is pixel 16 b + 4 q + r
// of the quad (row-major), so x = 4 (q & 1) + r and y = 2 b + (q >> 1).
//  - T and the sum behind run over the slots as scans across the 16 lanes of a
//    row; everything else of a (pixel, slot) is independent.
//  - A slot's sums over the quad's pixels are sums over a lane's own 16
//    registers (moments in r and b, whose factors are constants) and then over
//    four lanes, where one lane per pixel needs a reduction over 64 lanes for
//    each slot (100 of 287 cycles a slot in that form).
constexpr int kGroup = 16;
// Staged rows of a slot: -u0, e'.x, e'.y, -w0, k | o' | r, g, b | m'.x, m'.y
constexpr int kStageRows = 11;

// A wave's LDS.  The recomputing form's front-to-back sweep stages its 64
// records (3072 bytes) over rec and pos before they are in use.
struct __align__(16) BwdWave {
    float rec[kStageRows][64];   // staged slots
    uint32_t pos[128];           // list positions waiting, descending; the first 64 staged
    uint32_t nl[64];             // per pixel: bound on its contributors' positions
    float g[3][64];              // image gradient
    // per pixel, in front of the slots taken so far: transmittance, and the sum
    // of alpha T (c . g) behind
    float T[64], H[64];
};
static_assert(offsetof(BwdWave, nl) >= 64 * sizeof(Staged), "sweep overlay");

constexpr int kSums = 10;     // sums over pixels of one Gaussian

// What a Gaussian's sums hold.  With f the alpha gradient, o' the scaled
// opacity, G = 2^-p2, p2 = u^2 + w^2 (u = e' . d, w = f x d, d = pixel - mean)
// and P = f o' G = -dL/dp (p = d^T Q d / 2, Q the conic):
//   dL/dmean = 2 ln 2 P (u e'.x - w f.y, u e'.y + w f.x)
//            = 2 ln 2 o' [A B; B C] sum(f G d),
//     A = e'.x^2 + f.y^2, B = e'.x e'.y - f.x f.y, C = e'.y^2 + f.x^2;
//   dL/dQ = -P (dx^2 / 2, dx dy, dy^2 / 2);  dL/do = f (G - g_min) / (1 - g_min);
//   dL/dcolour = alpha T g.
// Sums 0-9 are f G (1, dx, dy, dx^2, dx dy, dy^2), alpha T g (3) and f;
// planes_of turns them into the planes with the record's shape.
//
// In the packed form the three of the conic are kept in the Gaussian's principal frame
// (t the tangent, n across): abar = -o' sum(f G t^2) / 2, bbar = -o' sum(f G n^2) / 2 and
// D = -o' sum(f G t n), which are what stage 2 needs.  In x and y the moments along a
// stroke, (sigma_x / sigma_y)^2 times those across it, would round the latter away in
// every addition to memory, and a width's gradient is made of them alone: its error
// against FP64 on the 2048x2048 frame 2e-5 that way, 1.5e-6 this way (the width of a
// table's sums is double, so turning them costs the stage 1.2%, and stage 2 gets 6%
// back).
__device__ inline void planes_of(const TileArgs &a, uint32_t id, const double (&D)[kSums],
                                 float (&out)[kGradPlanes]) {
    const float4 q = a.rec[3 * (int64_t)id + 1];
    float S[kSums];
#pragma unroll
    for (int v = 0; v < kSums; ++v) S[v] = (float)D[v];
    const float ex = kHalfLog2eSqrt * q.x, ey = kHalfLog2eSqrt * q.y;
    const float fx = q.z * ex, fy = q.z * ey;
    const float op = q.w * a.inv_1mg;
    const float A = fmaf(ex, ex, fy * fy), B = fmaf(ex, ey, -fx * fy), C = fmaf(ey, ey, fx * fx);
    const float k2 = 1.38629436112f * op;        // 2 ln 2 o'
    out[0] = k2 * fmaf(A, S[1], B * S[2]);
    out[1] = k2 * fmaf(B, S[1], C * S[2]);
    if (a.packed) {
        const float inv = __frsqrt_rn(fmaf(q.x, q.x, q.y * q.y));
        const double c = (double)(q.x * inv), s = (double)(q.y * inv), cs = c * s;
        out[2] = -0.5f * op * (float)(c * c * D[3] + 2.0 * cs * D[4] + s * s * D[5]);
        out[3] = -op * (float)(cs * (D[5] - D[3]) + (c * c - s * s) * D[4]);
        out[4] = -0.5f * op * (float)(s * s * D[3] - 2.0 * cs * D[4] + c * c * D[5]);
    } else {
        out[2] = -0.5f * op * S[3];
        out[3] = -op * S[4];
        out[4] = -0.5f * op * S[5];
    }
    out[5] = fmaf(-a.g_min, S[9], S[0]) * a.inv_1mg;
    out[6] = S[6];
    out[7] = S[7];
    out[8] = S[8];
}

// Add the nine values of up to n (<= 64) Gaussians to d_gauss: val[v][.] and
// the Gaussian ids (kNoGauss: none) in the wave's LDS, one Gaussian per column.
// Float atomics at device scope pass the L2 (its eight copies are one per XCD)
// and go to memory one 64-byte line per request, at about 20 G requests/s
// however few of a line's floats they touch.  In the packed form consecutive
// lanes take consecutive values of a Gaussian, so that a Gaussian costs one or
// two requests instead of nine: on the 2048x2048 frame 16.9 M requests a launch
// (0.82 ms of them alone) became 6.5 M.
constexpr uint32_t kNoGauss = 0xffffffffu;
__device__ inline void add_grads(const TileArgs &a, const float *val, int pitch,
                                 const uint32_t *ids, int n, int lane) {
    if (a.packed) {
        int e = lane / kGradPlanes, v = lane - e * kGradPlanes;
        for (int i = lane; i < kGradPlanes * n; i += 64) {
            const uint32_t id = ids[e];
            const float x = val[v * pitch + e];
            if (id != kNoGauss && x != 0.f) atomicAdd(a.d_gauss + (int64_t)id * kGradPlanes + v, x);
            e += 7;                              // 64 = 7 * 9 + 1
            if (++v == kGradPlanes) {
                v = 0;
                ++e;
            }
        }
    } else if (lane < n && ids[lane] != kNoGauss) {
#pragma unroll
        for (int v = 0; v < kGradPlanes; ++v) {
            const float x = val[v * pitch + lane];
            if (x != 0.f) atomicAdd(a.d_gauss + (int64_t)v * a.n_gauss + ids[lane], x);
        }
    }
}

// Tile-list positions pooled in LDS by the backward, as doubles: an LDS float
// atomic takes 2.8 CU cycles for every lane (177 for a full wave, whatever the
// addresses), a double one 8 for the whole wave.  With 16x16 tiles a block takes
// 4 x 4.8 KiB for its waves and 10 x 258 x 8 B of sums = 39.2 KiB, so four blocks
// (the four waves per SIMD its registers allow) share a CU's 160 KiB of LDS; 128
// positions ran 5% slower on the 2048x2048 frame, 160 at five waves per SIMD 25%
// (the registers spill).  The recomputing backward also keeps its batch masks in
// LDS; its table gives up their bytes (table_cap), so both forms hold the same
// LDS per block.
constexpr int kTableCap = 256;
constexpr int kTabPad = 2;

// Backward stage 1.  Each wave walks its tile list from the last entry any of
// its pixels used down to the first, over the entries the forward marked (at
// least one pixel of the quad used them).  Per pixel and contributor, in
// reverse order: T before it = T after / (1 - alpha); colour gradient alpha T
// g; with H the sum of alpha T (c . g) over everything behind it (the
// background first), alpha gradient = T (c . g) - H / (1 - alpha); then, unless
// alpha was clamped, the opacity gradient and dL/dp = -alpha_bar o' G.  The
// marked entries are compacted into a queue of list positions, staged 64 at a
// time and taken 16 at a time; the sums of 16 entries go, one LDS atomic per
// sum, to the tile's table (positions below its capacity) or straight to the
// per-Gaussian planes in HBM; the table is added to the planes when the tile
// is done.
//
// kRecompute: the blend state (T after the last contributor, the bound on its position and
// the per-batch contribution masks) is not read from memory but recomputed by
// a front-to-back sweep of the same quad (colour omitted), with the
// instruction sequence of the forward pass, so T and the positions are those
// the forward pass had.  The masks of the first kVisCap batches stay in LDS;
// later batches are box-tested again (a superset of the contributors: the
// others add exact zeros).
constexpr int kVisCap = 128;

// Lane constants of the reverse pass: the lane's pixel centres relative to the
// tile centre (x of register r, y of block b), and constants kept in vector
// registers.
struct BwdLane {
    float x[4], y[4], g_min, amax, three, nine;
};

// One group of 16 staged slots against the quad's 64 pixels; s: this lane's
// slot, last: the lane of the row's last slot.  check: some slot of the group may
// lie at or past a pixel's bound.  Returns three sums of slot j: q = 0: 0, 1, 2;
// q = 1: 3, 4; q = 2: 5, 6, 7; q = 3: 8, 9.
// u, w, G and alpha take the operations of the front-to-back sweep in its order
// (one rounding more or less can turn the decision whether alpha is clamped,
// where the gradient jumps).
//
// kInOrder: T before the slots as T times one factor 1 / (1 - alpha) after the other.
// Otherwise the factors' products come first, which is a scan of 4 steps instead of 15
// but needs 16 factors to stay finite: inf times a T of zero (a pixel outside the
// canvas, or T below the smallest float where t_min allows it) would be NaN.
template <bool kInOrder>
__device__ inline void bwd_group(BwdWave &wl, int s, int q, bool last, bool check,
                                 const BwdLane &L, float (&out)[3]) {
    const float nu0 = wl.rec[0][s], ex = wl.rec[1][s], ey = wl.rec[2][s];
    const float nw0 = wl.rec[3][s], k = wl.rec[4][s], mfy = -(k * ey), fx = k * ex;
    const float cr = wl.rec[6][s], cgr = wl.rec[7][s], cb = wl.rec[8][s];
    const float op = wl.rec[5][s], mog = -(op * L.g_min);
    const uint32_t pos = wl.pos[s];
    float wx[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) wx[r] = fmaf(mfy, L.x[r], nw0);
    // sums over the lane's pixels: f G (1, r, r^2, b, r b, b^2), f, alpha T g
    float S0 = 0.f, Sr = 0.f, Srr = 0.f, Sb = 0.f, Srb = 0.f, Sbb = 0.f, Sf = 0.f;
    float Sc0 = 0.f, Sc1 = 0.f, Sc2 = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int p4 = 16 * b + 4 * q;
        const floatx4 g0 = *reinterpret_cast<const floatx4 *>(&wl.g[0][p4]);
        const floatx4 g1 = *reinterpret_cast<const floatx4 *>(&wl.g[1][p4]);
        const floatx4 g2 = *reinterpret_cast<const floatx4 *>(&wl.g[2][p4]);
        const floatx4 T = *reinterpret_cast<const floatx4 *>(&wl.T[p4]);
        const floatx4 H = *reinterpret_cast<const floatx4 *>(&wl.H[p4]);
        float G[4], al[4], rho[4], Tb[4], Hb[4], x[4], cg[4], f[4];
        bool shaped[4];
        const float uy = fmaf(ey, L.y[b], nu0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float u = fmaf(ex, L.x[r], uy), w = fmaf(fx, L.y[b], wx[r]);
            G[r] = __builtin_amdgcn_exp2f(-fmaf(u, u, w * w));
        }
        if (check) {                         // wave-uniform
            const uint4 n4 = *reinterpret_cast<const uint4 *>(&wl.nl[p4]);
            G[0] = pos < n4.x ? G[0] : 0.f;
            G[1] = pos < n4.y ? G[1] : 0.f;
            G[2] = pos < n4.z ? G[2] : 0.f;
            G[3] = pos < n4.w ? G[3] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float araw = fmaf(op, G[r], mog);
            const bool c = G[r] > L.g_min;            // contributes
            shaped[r] = c && araw <= L.amax;          // and alpha is not clamped
            const float acl = min_f32(araw, L.amax);
            al[r] = c ? acl : 0.f;
            rho[r] = __builtin_amdgcn_rcpf(1.f - al[r]);
            Tb[r] = kInOrder ? rho[r] * T[r] : rho[r];
            cg[r] = fmaf(cr, g0[r], fmaf(cgr, g1[r], cb * g2[r]));
        }
        if (kInOrder) {
            for (int i = 1; i < kGroup; ++i) BZ_ROW_MUL_STEP4(Tb, rho);
        } else {
            BZ_ROW_SCAN4("v_mul_f32_dpp", Tb);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (!kInOrder) Tb[r] *= T[r];             // T before the slot
            al[r] *= Tb[r];                           // its weight alpha T
            x[r] = al[r] * cg[r];
            Sc0 = fmaf(al[r], g0[r], Sc0);
            Sc1 = fmaf(al[r], g1[r], Sc1);
            Sc2 = fmaf(al[r], g2[r], Sc2);
            Hb[r] = row_shifted(H[r], x[r]);
        }
        BZ_ROW_SCAN4("v_add_f32_dpp", Hb);            // the sum behind the slot
        if (last) {
            *reinterpret_cast<floatx4 *>(&wl.T[p4]) = floatx4{Tb[0], Tb[1], Tb[2], Tb[3]};
            *reinterpret_cast<floatx4 *>(&wl.H[p4]) =
                floatx4{Hb[0] + x[0], Hb[1] + x[1], Hb[2] + x[2], Hb[3] + x[3]};
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // T (c . g) - H / (1 - alpha).  The slot's own term stays out of H: at
            // alpha near 1 two terms that both hold it would nearly cancel.
            const float ab = fmaf(Tb[r], cg[r], -rho[r] * Hb[r]);
            f[r] = shaped[r] ? ab : 0.f;
            Sf += f[r];
            f[r] *= G[r];
        }
        const float R = (f[0] + f[1]) + (f[2] + f[3]);
        const float X = fmaf(f[3], L.three, fmaf(f[2], 2.f, f[1]));
        const float XX = fmaf(f[3], L.nine, fmaf(f[2], 4.f, f[1]));
        S0 += R;
        Sr += X;
        Srr += XX;
        if (b == 1) {
            Sb += R;
            Srb += X;
            Sbb += R;
        } else if (b > 1) {
            const float fb = b == 2 ? 2.f : L.three;
            Sb = fmaf(R, fb, Sb);
            Srb = fmaf(X, fb, Srb);
            Sbb = fmaf(R, b == 2 ? 4.f : L.nine, Sbb);
        }
        // The block's sums are finished here: left to the compiler they sink
        // past the next blocks' branches, with every factor of theirs kept
        // until then, and spill.
        asm volatile("" : "+v"(S0), "+v"(Sr), "+v"(Srr), "+v"(Sb), "+v"(Srb), "+v"(Sbb), "+v"(Sf),
                     "+v"(Sc0), "+v"(Sc1), "+v"(Sc2));
    }
    // moments about the mean: dx = x[0] - m'.x + r, dy = y[0] - m'.y + 2 b.  Where f G
    // is not small the lane is near the mean; about the tile centre the moments of a
    // small Gaussian lose (8 / sigma)^2 of their precision when they are moved.
    const float X0 = L.x[0] - wl.rec[9][s], Y0 = L.y[0] - wl.rec[10][s];
    float v[10];
    v[0] = S0;
    v[1] = fmaf(X0, S0, Sr);
    v[2] = fmaf(Sb, 2.f, Y0 * S0);
    v[3] = fmaf(X0, v[1] + Sr, Srr);
    v[4] = fmaf(Y0, v[1], 2.f * fmaf(X0, Sb, Srb));
    v[5] = fmaf(Y0, fmaf(Sb, 2.f, v[2]), 4.f * Sbb);
    v[6] = Sc0;
    v[7] = Sc1;
    v[8] = Sc2;
    v[9] = Sf;
    // over the four lanes of the slot: halves exchanged with lane l ^ 32, then
    // thirds with lane l ^ 16
    float y[5], z[3];
    asm("s_nop 1\n\t"
        "v_permlane32_swap_b32 %0, %5\n\t"
        "v_permlane32_swap_b32 %1, %6\n\t"
        "v_permlane32_swap_b32 %2, %7\n\t"
        "v_permlane32_swap_b32 %3, %8\n\t"
        "v_permlane32_swap_b32 %4, %9"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),
          "+v"(v[7]), "+v"(v[8]), "+v"(v[9]));
#pragma unroll
    for (int i = 0; i < 5; ++i) y[i] = v[i] + v[i + 5];
    float pad = 0.f;
    asm("s_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %3\n\t"
        "v_permlane16_swap_b32 %1, %4\n\t"
        "v_permlane16_swap_b32 %2, %5"
        : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]), "+v"(y[4]), "+v"(pad));
    z[0] = y[0] + y[3];
    z[1] = y[1] + y[4];
    z[2] = y[2] + pad;
    out[0] = z[0];
    out[1] = z[1];
    out[2] = z[2];
}

template <bool kRecompute, bool kInOrder>
__device__ inline void bwd_tile(const TileArgs &a, int tile) {
    // dynamic LDS: per wave a BwdWave, the sum table, and (kRecompute)
    // [waves][kVisCap] batch masks
    extern __shared__ __align__(16) unsigned char s_bwd[];
    __shared__ uint32_t s_top[16];
    const int nwaves = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const TileGeo tg = tile_geo(a, tile);
    const int qx = w % a.quads_x, qy = w / a.quads_x;
    const int x0 = tg.tx * a.tile_w + qx * kQuad, y0 = tg.ty * a.tile_h + qy * kQuad;
    const bool wave_on = x0 < tg.W && y0 < tg.H;         // quad inside the canvas
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    const bool valid = wave_on && x < tg.W && y < tg.H;
    const float lx = (float)(lane & 7), ly = (float)(lane >> 3);   // pixel - first pixel of the quad
    const float qx0 = (float)x0 + 0.5f, qy0 = (float)y0 + 0.5f;
    // The reverse pass measures from the tile centre (ox, oy): the moments the
    // quads of a tile add to one table need one origin.  (bx, by): the quad's
    // first pixel centre relative to it.
    const float ox = (float)(tg.tx * a.tile_w) + 0.5f * (float)a.tile_w;
    const float oy = (float)(tg.ty * a.tile_h) + 0.5f * (float)a.tile_h;
    const float bx = qx0 - ox, by = qy0 - oy;
    BwdWave &wl = reinterpret_cast<BwdWave *>(s_bwd)[w];
    // Per-tile sums, plane-major [kSums][tab_cap + kTabPad], indexed by
    // tile-list position: the quads of a tile share most of their Gaussians, so
    // their sums meet here and leave the block with one global atomic per
    // (Gaussian, plane).
    const int tab_cap = a.tab_cap, tab_p = tab_cap + kTabPad;
    double *table = reinterpret_cast<double *>(s_bwd + (size_t)nwaves * sizeof(BwdWave));
    // kRecompute: per-wave batch masks after the table
    uint64_t *s_vis = reinterpret_cast<uint64_t *>(table + kSums * tab_p) + w * kVisCap;

    // wave-uniform: held in scalar registers
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ranges[2 * tile]);
    const uint32_t len =
        (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ranges[2 * tile + 1]) - start;
    const uint64_t *vis =
        kRecompute ? nullptr : a.visit + (int64_t)w * a.words_per_plane + visit_word(start, tile);
    const int64_t pix = tg.pix0 + (int64_t)y * tg.W + x;
    const int64_t plane = (int64_t)tg.W * tg.H;
    const float *dimg = a.d_image + 2 * tg.pix0;   // canvas planes from 3 * pix0
    uint32_t nl = 0;
    float Tf = 0.f, g0 = 0.f, g1 = 0.f, g2 = 0.f;
    if (kRecompute) {
        if (wave_on) {
            Staged *my = reinterpret_cast<Staged *>(&wl);
            const Sweep r = fwd_sweep<false, false>(a, my, start, start + len, lx, ly, qx0, qy0,
                                                    valid, lane, [&](uint32_t k, uint64_t bits) {
                                                        if (lane == 0 && k < kVisCap) s_vis[k] = bits;
                                                    });
            nl = valid ? r.last : 0u;
            Tf = valid ? r.T : 0.f;
        }
        wave_lds_sync();
    } else if (valid) {
        nl = a.n_last[pix];
        Tf = a.t_final[pix];
    }
    if (valid) {
        g0 = dimg[pix];
        g1 = dimg[plane + pix];
        g2 = dimg[2 * plane + pix];
    }
    uint32_t top = wave_max_u32(nl);   // wave-uniform
    top = top < len ? top : len;
    const uint32_t min_nl = wave_min_u32(valid ? nl : 0xffffffffu);
    if (lane == 0) s_top[w] = top;
    __syncthreads();
    uint32_t top_block = 0;
    for (int i = 0; i < nwaves; ++i) top_block = max(top_block, s_top[i]);
    const int tab_n = (int)(top_block < (uint32_t)tab_cap ? top_block : (uint32_t)tab_cap);
    for (int i = threadIdx.x; i < kSums * tab_n; i += blockDim.x) {
        const int v = i / tab_n;
        table[v * tab_p + (i - v * tab_n)] = 0.0;
    }
    // the quad's pixels into LDS, and from there into the lanes of the products
    const int q = lane >> 4, j = lane & 15;
    {
        wl.g[0][lane] = g0;
        wl.g[1][lane] = g1;
        wl.g[2][lane] = g2;
        wl.nl[lane] = nl;
        wl.T[lane] = Tf;
        // behind everything: the background
        wl.H[lane] = Tf * fmaf(tg.bg0, g0, fmaf(tg.bg1, g1, tg.bg2 * g2));
    }
    BwdLane L = {{}, {}, vector_f32(a.g_min), vector_f32(a.alpha_max), vector_f32(3.f),
                 vector_f32(9.f)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        L.x[i] = bx + (float)(4 * (q & 1) + i);
        L.y[i] = by + (float)((q >> 1) + 2 * i);
    }
    // the lane's sums of a group: nv of them from v0
    const int v0 = q < 2 ? 3 * q : 3 * q - 1, nv = q & 1 ? 2 : 3;
    __syncthreads();                                       // the table is clear

    // Marked entries, last to first, into the queue of list positions: batch
    // masks 64 at a time (lane l holds that of batch wtop - 1 - l), the ones
    // with entries one by one.
    const uint32_t nb = wave_on ? (uint32_t)(((uint64_t)top + 63) / 64) : 0u;
    uint32_t kbox = nb;                                    // kRecompute: batches to box-test
    uint32_t wtop = 0, wnext = kRecompute && nb > kVisCap ? kVisCap : nb;
    uint64_t words = 0, nz = 0;
    int qn = 0;
    auto push = [&](uint32_t k, uint64_t word) {           // wave-uniform word of batch k
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(word >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)word, 0u));
        const int n = __popcll(word);
        if ((word >> lane) & 1ull) wl.pos[qn + n - 1 - (int)below] = 64 * k + (uint32_t)lane;
        qn += n;
    };
    // only entries of this tile's list can be visited
    auto in_list = [&](uint32_t k) {
        const uint32_t avail = len - 64 * k;
        return avail >= 64 ? ~0ull : ((1ull << avail) - 1ull);
    };
    while (true) {
        while (qn < 64) {
            if (kRecompute && kbox > kVisCap) {
                --kbox;
                const uint32_t p = 64 * kbox + (uint32_t)lane;
                const bool hit = p < len && entry_hit_bwd(a, a.ids[start + p], ox, oy, bx, by);
                push(kbox, __ballot(hit));
                continue;
            }
            if (nz == 0) {
                if (wnext == 0) break;
                wtop = wnext;
                wnext = wtop > 64 ? wtop - 64 : 0;
                words = 0;
                if ((uint32_t)lane < wtop) {
                    const uint32_t k = wtop - 1 - (uint32_t)lane;
                    words = (kRecompute ? s_vis[k] : vis[k]) & in_list(k);
                }
                nz = __ballot(words != 0);
                continue;
            }
            const int i = __builtin_ctzll(nz);
            nz &= nz - 1;
            push(wtop - 1 - (uint32_t)i, lane_u64(words, i));
        }
        if (qn == 0) break;
        const int n = qn < 64 ? qn : 64;
        wave_lds_sync();
        // stage the first n: lane l slot l, the slots past them contribute nothing
        {
            float4 sm = make_float4(0.f, 0.f, 0.f, 0.f), sq = sm, sc = sm;
            float2 mean = make_float2(0.f, 0.f);
            if (lane < n) {
                Staged st;
                float4 shape;
                stage_record(a, a.ids[start + wl.pos[lane]], ox, oy, st, shape, mean);
                sm = st.m;
                sq = st.q;
                sc = st.c;
            }
            wl.rec[0][lane] = sm.x;
            wl.rec[1][lane] = sm.z;
            wl.rec[2][lane] = sm.w;
            wl.rec[3][lane] = sm.y;
            wl.rec[4][lane] = sq.z;
            wl.rec[5][lane] = sq.w;
            wl.rec[6][lane] = sc.x;
            wl.rec[7][lane] = sc.y;
            wl.rec[8][lane] = sc.z;
            wl.rec[9][lane] = mean.x;
            wl.rec[10][lane] = mean.y;
        }
        wave_lds_sync();
        for (int s0 = 0; s0 < n; s0 += kGroup) {
            const int s = s0 + j;
            const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)wl.pos[s0]);
            float E[3];
            bwd_group<kInOrder>(wl, s, q, j == kGroup - 1, first >= min_nl, L, E);
            const bool live = s < n;
            const uint32_t p = live ? wl.pos[s] : 0u;
            if (live && p < (uint32_t)tab_cap) {
                double *row = table + v0 * tab_p + p;
                atomicAdd(row, (double)E[0]);
                atomicAdd(row + tab_p, (double)E[1]);
                if (nv == 3) atomicAdd(row + 2 * tab_p, (double)E[2]);
            }
            if (first >= (uint32_t)tab_cap) {        // some lie past the table
                wave_lds_sync();
                wl.rec[v0][s] = E[0];
                wl.rec[v0 + 1][s] = E[1];
                if (nv == 3) wl.rec[v0 + 2][s] = E[2];
                wave_lds_sync();
                if (q == 0) {                        // the slot's own column, in place
                    uint32_t id = kNoGauss;
                    if (live && p >= (uint32_t)tab_cap) {
                        double S[kSums];
                        float o[kGradPlanes];
#pragma unroll
                        for (int v = 0; v < kSums; ++v) S[v] = (double)wl.rec[v][s];
                        id = a.ids[start + p];
                        planes_of(a, id, S, o);
#pragma unroll
                        for (int v = 0; v < kGradPlanes; ++v) wl.rec[v][s] = o[v];
                    }
                    reinterpret_cast<uint32_t *>(wl.rec[9])[s] = id;
                }
                wave_lds_sync();
                add_grads(a, &wl.rec[0][s0], 64, reinterpret_cast<uint32_t *>(&wl.rec[9][s0]),
                          n - s0 < kGroup ? n - s0 : kGroup, lane);
            }
        }
        wave_lds_sync();
        const uint32_t rest = lane < qn - n ? wl.pos[64 + lane] : 0u;
        wave_lds_sync();
        if (lane < qn - n) wl.pos[lane] = rest;
        qn -= n;
    }
    __syncthreads();
    // the table's moments to the nine planes, 64 positions per wave at a time
    uint32_t *fid = reinterpret_cast<uint32_t *>(wl.rec[9]);
    for (int p0 = 64 * w; p0 < tab_n; p0 += 64 * nwaves) {
        const int p = p0 + lane;
        double S[kSums];
        float o[kGradPlanes];
        bool any = false;
#pragma unroll
        for (int v = 0; v < kSums; ++v) {
            S[v] = p < tab_n ? table[v * tab_p + p] : 0.0;
            any |= S[v] != 0.0;
        }
        uint32_t id = kNoGauss;
        if (any) {
            id = a.ids[start + p];
            planes_of(a, id, S, o);
#pragma unroll
            for (int v = 0; v < kGradPlanes; ++v) wl.rec[v][lane] = o[v];
        }
        fid[lane] = id;
        wave_lds_sync();
        add_grads(a, &wl.rec[0][0], 64, fid, tab_n - p0 < 64 ? tab_n - p0 : 64, lane);
        wave_lds_sync();
    }
}

// Bound by VALU issue: 583 M instructions on the 2048x2048 frame (11.1 M slots), on
// all of the SIMD cycles.  1,480 us in the form of one lane per pixel with a
// 64-lane reduction per slot, float LDS atomics and plane atomics; 1,010-1,050 us in
// this one (2040x1344 with 2,048 closed curves: 867 -> 600-645; 128x128: 101 -> 57, where
// one staging per 64 entries instead of per batch shortens the chain of loads).
// Products on the matrix cores (v_mfma_f32_16x16x4_f32 for u, w, c . g and the
// sums) measured no faster than the first form: FP32 products issue at the
// vector rate there and do not overlap with vector instructions.
template <bool kRecompute, bool kInOrder>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_bwd_tiles(
    TileArgs a) {
    if (a.status[1] & Status::kOverflow) return;         // whole grid
    for_tiles(a, [&](int tile) { bwd_tile<kRecompute, kInOrder>(a, tile); });
}

__global__ void k_zero(float *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0.f;
}

// Sum over the NT lanes of a curve: in all lanes for a whole wave, in the last of 16 or 32
// otherwise.
template <int NT>
__device__ inline float lanes_sum(float v) {
    if (NT >= kWave) return wave_sum(v);
    v += dpp_f32<0x111, 0xF, true>(v);
    v += dpp_f32<0x112, 0xF, true>(v);
    v += dpp_f32<0x114, 0xF, true>(v);
    v += dpp_f32<0x118, 0xF, true>(v);
    if (NT == 32) v += dpp_f32<0x142, 0xA, false>(v);
    return v;
}

// X[r][k1] - X[r][k0] from the samples in double precision, as the sampler has them,
// rounded once; t: the row's place between the boundaries.
__device__ inline float2 chord_between(const CurveView &v, double t, int k0, int k1) {
    double2 first = make_double2(0.0, 0.0), x = first;
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {
        first = x;
        x = boundary_point(v, false, e ? k1 : k0);
        if (v.kind == BZ_CLOSED) {
            const double2 b = boundary_point(v, true, e ? k1 : k0);
            x = make_double2((1.0 - t) * x.x + t * b.x, (1.0 - t) * x.y + t * b.y);
        }
    }
    return make_float2((float)(x.x - first.x), (float)(x.y - first.y));
}

// Stage 2: one workgroup per curve.  Per Gaussian (r, k) the gradients of
// (mean, Q, o, colour) are chained to the sample points of its stencil:
//   Q = R diag(a, b) R^T, a = 1/sx2, b = 1/sy2, (c, s) = v/|v|,
//   sx2 = |X[r][ka]-X[r][kb]|^2/rho^2 + s0, sy2 = |X[ra][k]-X[rb][k]|^2/rho^2 + s0
//   (closed) or w^2 + s0 (open), mean = X[r][k].
// Each Gaussian stores its four stencil terms (mean, along-row, across-row,
// tangent) in LDS; every sample point then gathers the terms that reference
// it (the exact inverse of the stencil's index rules), so no atomics are
// needed and the result is deterministic.  The sample-point gradients then go
// to the control points: X[r][k] = sum_j B_j(t_k) ((1-tau_r) A_{3s+j} + tau_r B_{3s+j}).
// The boundary samples are evaluated in double precision (coordinates of
// thousands of pixels) and only their differences along each boundary and
// from boundary A to B are kept, rounded to float (differences of a pixel):
// a row's differences are blends of those, and the chain itself is float.  Where a row
// turns back on itself its tangent, the difference over two columns, nearly cancels, and
// with the rounding of the chords it is made of so does its direction, in which the
// conic's gradient is turned: below 1% of the chords the direction is the record's
// (kPacked, one load), or the tangent is taken anew from the samples in double precision.
//
// NT threads per curve.  Two launches split the curves by size: those of at
// most kSmallCurve Gaussians (open strokes) run as one-wave workgroups with
// LDS sized for them, the others with kCurveThreads threads; each launch
// skips the other's curves.  Where no curve has more than 32 (16) Gaussians and the
// chip is full, two (four) share a wave: 35,000 strokes of 16 to 32 samples 62 -> 50 us.  lk and lg are the K and Gaussian capacities the
// dynamic LDS is laid out for.
// Eight waves per SIMD (at most 64 VGPRs): the stage waits on
// latency, and at seven it ran 5% slower.  Sharing curves hold theirs in 94 vector
// registers; held to 64 they spill (73 us).
//
// kPacked: d_gauss holds nine floats per Gaussian, and the nine planes are
// written to planes as they are read; rec: the records stage 1 ran on.
template <int NT, bool kPacked>
__global__ __launch_bounds__(NT < kWave ? kWave : NT) __attribute__((amdgpu_waves_per_eu(NT < kWave ? 5 : 8, 8))) void k_bwd_curves(bz_curves c, int lk, int lg, double inv_rho2,
                                                   double s0, const float *__restrict__ d_gauss,
                                                   float *__restrict__ planes,
                                                   const float4 *__restrict__ rec,
                                                   int64_t ng, float *__restrict__ d_ctrl,
                                                   float *__restrict__ d_width,
                                                   float *__restrict__ d_color,
                                                   float *__restrict__ d_opacity) {
    constexpr int kShare = NT < kWave ? kWave / NT : 1;    // curves per wave
    extern __shared__ double2 lds_all[];
    __shared__ float s_taus[kShare][kShare > 1 ? NT : 256];
    __shared__ float s_red[kShare > 1 ? 1 : NT / 64][8];
    __shared__ float s_cps[kShare][2][3 * kMaxSeg + 1][2];
    const int sub = kShare > 1 ? threadIdx.x / NT : 0;
    const int p = blockIdx.x * kShare + sub;
    const int lane = kShare > 1 ? threadIdx.x % NT : threadIdx.x;   // thread of the curve
    if (kShare > 1) {
        if (p >= c.n_curves) return;
    } else {
        const bool small = c.gauss_off[p + 1] - c.gauss_off[p] <= kSmallCurve;
        if (small != (NT == kWave)) return;   // the other launch's curve
    }
    double2 *const lds_xy = reinterpret_cast<double2 *>(
        reinterpret_cast<char *>(lds_all) + sub * (stage2_terms_offset(lk) + 4 * 8 * lg));
    float *const s_tau = s_taus[sub];
    float (*const s_cp)[3 * kMaxSeg + 1][2] = s_cps[sub];
    CurveView v = load_curve_view(c, p);
    stage_tau(v, s_tau, lane, NT);
    // [K] column differences of the boundary samples: DA[k] = XA[k+1] - XA[k],
    // DB[k] likewise, and W[k] = XB[k] - XA[k] (closed), in the boundary
    // samples' space (2 x double2 per column)
    float2 *DA = reinterpret_cast<float2 *>(lds_xy);
    float2 *DB = DA + lk;
    float2 *Wd = DB + lk;
    float4 *Bw = reinterpret_cast<float4 *>(lds_xy + 2 * lk);          // [K] Bernstein weights
    int *Bs = reinterpret_cast<int *>(Bw + lk);                        // [K] segment of column k
    float2 *Tm = reinterpret_cast<float2 *>(reinterpret_cast<char *>(lds_xy) +
                                            stage2_terms_offset(lk));  // mean term, then Xbar
    float2 *Tf = Tm + lg;                                              // along-row term
    float2 *Th = Tf + lg;                                              // across-row term
    float2 *Tv = Th + lg;                                              // tangent term
    float2 *Xbar = Tm;                                                 // [rows*K]
    const bool closed = v.kind == BZ_CLOSED;
    // The boundary samples in double precision, one per thread, in the space
    // of the terms (written only after the next barrier; 32 K <= 32 lg
    // bytes), and each column's segment and Bernstein weights beside them;
    // then the differences, rounded once.
    {
        double2 *P = reinterpret_cast<double2 *>(Tm);    // [A's K][B's K]
        const int nb = closed ? 2 : 1;
        for (int i = lane; i < (nb + 1) * v.K; i += NT) {
            if (i < nb * v.K) {
                const bool bb = i >= v.K;
                P[i] = boundary_point(v, bb, bb ? i - v.K : i);
            } else {
                const int k = i - nb * v.K;
                int s;
                double t, B[4];
                column_param(k, v.K, v.S, s, t);
                bernstein3(t, B);
                Bw[k] = make_float4((float)B[0], (float)B[1], (float)B[2], (float)B[3]);
                Bs[k] = s;
            }
        }
        __syncthreads();
        for (int k = lane; k < v.K; k += NT) {
            const double2 a0 = P[k], a1 = k + 1 < v.K ? P[k + 1] : a0;
            DA[k] = make_float2((float)(a1.x - a0.x), (float)(a1.y - a0.y));
            if (closed) {
                const double2 b0 = P[v.K + k], b1 = k + 1 < v.K ? P[v.K + k + 1] : b0;
                DB[k] = make_float2((float)(b1.x - b0.x), (float)(b1.y - b0.y));
                Wd[k] = make_float2((float)(b0.x - a0.x), (float)(b0.y - a0.y));
            }
        }
    }
    const int n = v.rows * v.K;
    __syncthreads();

    float wbar = 0.f, cb0 = 0.f, cb1 = 0.f, cb2 = 0.f;
    float ob[kMaxSeg] = {0.f, 0.f, 0.f, 0.f};
    const float rho2f = (float)inv_rho2;
    const int K = v.K, R1 = v.R + 1;
    // (r, k) of idx = lane + i*NT advance by (NT / K, NT % K) per pass.
    const int rstep = NT / K, kstep = NT - rstep * K;
    const int r0 = lane / K, k0 = lane - r0 * K;
    for (int idx = lane, r = r0, k = k0; idx < n; idx += NT) {
        float dg[kGradPlanes];
        const auto load = [&] {
#pragma unroll
            for (int q = 0; q < kGradPlanes; ++q)
                dg[q] = d_gauss[kPacked ? kGradPlanes * (v.g0 + idx) + q : q * ng + v.g0 + idx];
        };
        if (kPacked) load();
        // stencil (Eq. sigma with nearest-neighbour ends, Eq. rotation).  Row
        // r's samples are (1 - tau_r) XA + tau_r XB, so its differences along
        // the row are the same blend of DA and DB, and across rows
        // (tau_ra - tau_rb) W.
        const int kb = k < K - 1 ? k : K - 2;              // ka = kb + 1
        const int km = k > 0 ? k - 1 : 0;                  // kp = km + 1 or km + 2
        const bool two = k > 0 && k < K - 1;
        const float tr = closed ? v.tau[r] : 0.f, t1 = 1.f - tr;
        float dax = DA[kb].x, day = DA[kb].y;
        float vx = DA[km].x, vy = DA[km].y;
        float chords = fabsf(vx) + fabsf(vy);
        if (two) {
            const float2 a1 = DA[km + 1];
            vx += a1.x;
            vy += a1.y;
            chords += fabsf(a1.x) + fabsf(a1.y);
        }
        if (closed) {
            float bx = DB[km].x, by = DB[km].y;
            float chords_b = fabsf(bx) + fabsf(by);
            if (two) {
                const float2 b1 = DB[km + 1];
                bx += b1.x;
                by += b1.y;
                chords_b += fabsf(b1.x) + fabsf(b1.y);
            }
            chords = fmaf(tr, chords_b, t1 * chords);
            vx = fmaf(tr, bx, t1 * vx);
            vy = fmaf(tr, by, t1 * vy);
            dax = fmaf(tr, DB[kb].x, t1 * dax);
            day = fmaf(tr, DB[kb].y, t1 * day);
        }
        float nv2 = vx * vx + vy * vy;
        const bool turns = nv2 < 1e-4f * chords * chords;
        if (!kPacked) {
            if (turns) {
                const float2 chord = chord_between(v, (double)tr, km, km + (two ? 2 : 1));
                vx = chord.x;
                vy = chord.y;
                nv2 = vx * vx + vy * vy;
            }
            load();                              // not held over the branch above
        }
        float dyx = 0.f, dyy = 0.f, sy2;
        if (closed) {
            const int ra = r < R1 ? r + 1 : R1, rb = r < R1 ? r : R1 - 1;
            const float dt = v.tau[ra] - v.tau[rb];
            dyx = dt * Wd[k].x;
            dyy = dt * Wd[k].y;
            sy2 = (dyx * dyx + dyy * dyy) * rho2f + (float)s0;
        } else {
            sy2 = v.width * v.width + (float)s0;
        }
        const float sx2 = (dax * dax + day * day) * rho2f + (float)s0;
        const float inv_nv = nv2 > 0.f ? __frsqrt_rn(nv2) : 0.f;
        float cs = nv2 > 0.f ? vx * inv_nv : 1.f, sn = nv2 > 0.f ? vy * inv_nv : 0.f;
        if (kPacked && turns) {
            const float4 e = rec[3 * (v.g0 + idx) + 1];
            const float e2 = fmaf(e.x, e.x, e.y * e.y);
            if (e2 > 0.f && e2 < 3.0e38f) {                // a Gaussian in no list may have any
                cs = e.x * __frsqrt_rn(e2);
                sn = e.y * __frsqrt_rn(e2);
            }
        }
        const float ia = __builtin_amdgcn_rcpf(sx2), ib = __builtin_amdgcn_rcpf(sy2);
        // the conic's gradient in the principal frame: along, across and mixed
        float abar, bbar, mixed;
        if (kPacked) {
            abar = dg[2];
            mixed = dg[3];
            bbar = dg[4];
            // abar may be hundreds of times bbar, and the way back takes bbar from
            // differences of terms of its size: in double, what is lost is the planes'
            // rounding alone
            const double c = cs, s = sn, d = (double)abar - bbar;
            const double c2 = c * c, s2 = s * s, m = c * s * mixed;
            dg[2] = (float)(c2 * d + (bbar - m));
            dg[3] = (float)(2.0 * c * s * d + (c2 - s2) * mixed);
            dg[4] = (float)(s2 * d + (bbar + m));
#pragma unroll
            for (int q = 0; q < kGradPlanes; ++q) planes[q * ng + v.g0 + idx] = dg[q];
        } else {
            const double qxx = dg[2], qxy = dg[3], qyy = dg[4], c = cs, s = sn;
            abar = (float)(qxx * c * c + qxy * c * s + qyy * s * s);
            bbar = (float)(qxx * s * s - qxy * c * s + qyy * c * c);
            mixed = (float)(2.0 * c * s * (qyy - qxx) + (c * c - s * s) * qxy);
        }
        const float f = 2.f * (-abar * ia * ia) * rho2f;
        const float sy2bar = -bbar * ib * ib;
        Tm[idx] = make_float2(dg[0], dg[1]);
        Tf[idx] = make_float2(f * dax, f * day);
        if (closed) {
            const float h = 2.f * sy2bar * rho2f;
            Th[idx] = make_float2(h * dyx, h * dyy);
        } else {
            wbar += 2.f * v.width * sy2bar;
        }
        if (nv2 > 0.f) {
            // the tangent's gradient across itself: turning it mixes the two scales
            const float h = (ia - ib) * mixed * inv_nv;
            Tv[idx] = make_float2(-sn * h, cs * h);
        } else {
            Tv[idx] = make_float2(0.f, 0.f);
        }
        const int slot = v.nopa == v.S ? Bs[k] : 0;
#pragma unroll
        for (int q = 0; q < kMaxSeg; ++q)
            if (q == slot) ob[q] += dg[5];
        cb0 += dg[6];
        cb1 += dg[7];
        cb2 += dg[8];
        k += kstep;
        r += rstep;
        if (k >= K) { k -= K; ++r; }
    }
    __syncthreads();
    // Gather: the terms each sample point (r, k) receives.
    //  along  +Tf(j) where ka(j) = k: j = k-1 (k >= 1), and j = K-1 when k = K-1
    //         -Tf(j) where kb(j) = k: j = k (k < K-1), and j = K-1 when k = K-2
    //  tangent+Tv(j) where kp(j) = k: j = k-1 (k >= 1), and j = K-1 when k = K-1
    //         -Tv(j) where km(j) = k: j = k+1 (k < K-1), and j = 0 when k = 0
    //  across +Th(i) where ra(i) = r: i = r-1 (r >= 1), and i = R+1 when r = R+1
    //         -Th(i) where rb(i) = r: i = r (r <= R), and i = R+1 when r = R
    // Xbar overwrites Tm in place: a point reads only its own mean term.
    for (int idx = lane, r = r0, k = k0; idx < n; idx += NT) {
        const int row = idx - k;
        const float2 x = Tm[idx];
        float ax = 0.f, ay = 0.f;
        if (k >= 1) { ax += Tf[row + k - 1].x + Tv[row + k - 1].x; ay += Tf[row + k - 1].y + Tv[row + k - 1].y; }
        if (k == K - 1) { ax += Tf[row + K - 1].x + Tv[row + K - 1].x; ay += Tf[row + K - 1].y + Tv[row + K - 1].y; }
        if (k < K - 1) { ax -= Tf[row + k].x + Tv[row + k + 1].x; ay -= Tf[row + k].y + Tv[row + k + 1].y; }
        if (k == K - 2) { ax -= Tf[row + K - 1].x; ay -= Tf[row + K - 1].y; }
        if (k == 0) { ax -= Tv[row].x; ay -= Tv[row].y; }
        if (closed) {
            if (r >= 1) { ax += Th[idx - K].x; ay += Th[idx - K].y; }
            if (r == R1) { ax += Th[idx].x; ay += Th[idx].y; }
            if (r <= R1 - 1) { ax -= Th[idx].x; ay -= Th[idx].y; }
            if (r == R1 - 1) { ax -= Th[idx + K].x; ay -= Th[idx + K].y; }
        }
        Xbar[idx] = make_float2(x.x + ax, x.y + ay);
        k += kstep;
        r += rstep;
        if (k >= K) { k -= K; ++r; }
    }

    // per-curve sums: wave (or part of one) reduction, then across the workgroup's waves
    wbar = lanes_sum<NT>(wbar);
    cb0 = lanes_sum<NT>(cb0);
    cb1 = lanes_sum<NT>(cb1);
    cb2 = lanes_sum<NT>(cb2);
#pragma unroll
    for (int q = 0; q < kMaxSeg; ++q) ob[q] = lanes_sum<NT>(ob[q]);
    if (kShare == 1 && (lane & 63) == 0) {
        float *sr = s_red[lane >> 6];
        sr[0] = wbar; sr[1] = cb0; sr[2] = cb1; sr[3] = cb2;
#pragma unroll
        for (int q = 0; q < kMaxSeg; ++q) sr[4 + q] = ob[q];
    }
    __syncthreads();
    if (lane == (kShare > 1 ? NT - 1 : 0)) {
        for (int wv = 1; wv < NT / 64; ++wv) {
            wbar += s_red[wv][0]; cb0 += s_red[wv][1]; cb1 += s_red[wv][2]; cb2 += s_red[wv][3];
#pragma unroll
            for (int q = 0; q < kMaxSeg; ++q) ob[q] += s_red[wv][4 + q];
        }
        d_width[v.id] = closed ? 0.f : wbar;
        d_color[3 * v.id] = cb0;
        d_color[3 * v.id + 1] = cb1;
        d_color[3 * v.id + 2] = cb2;
        float *dop = d_opacity + c.opa_off[v.id];
#pragma unroll
        for (int q = 0; q < kMaxSeg; ++q)
            if (q < v.nopa) dop[q] = ob[q];
    }

    // Control points, in two deterministic steps.  (1) Thread (k, coord) sums
    // column k of Xbar over the rows three ways: all rows (open curves and the
    // endpoints a closed curve's boundaries share), weighted by 1 - tau_r (A's
    // interior points) and by tau_r (B's interior points); the sums go to LDS
    // over Tf..Tv (dead by now; 24 K bytes fit in their 24 rows*K).  (2) Thread
    // (point jj, coord, boundary) adds B_{jj - 3 s_k}(t_k) times those sums
    // over the columns k in order.
    const int m = 3 * v.S;
    float *colsum = reinterpret_cast<float *>(Tf);      // [K][coord][3]
    __syncthreads();   // every Xbar written, every T* read
    for (int t = lane; t < 2 * K; t += NT) {
        const int coord = t & 1, kk = t >> 1;
        float sall = 0.f, sa = 0.f, sb = 0.f;
        for (int rr = 0; rr < v.rows; ++rr) {
            const float2 xb2 = Xbar[rr * K + kk];
            const float xb = coord ? xb2.y : xb2.x;
            const float tr = closed ? v.tau[rr] : 0.f;
            sall += xb;
            sa = fmaf(1.f - tr, xb, sa);
            sb = fmaf(tr, xb, sb);
        }
        float *o = colsum + 3 * t;
        o[0] = sall;
        o[1] = sa;
        o[2] = sb;
    }
    __syncthreads();
    for (int t = lane; t < 4 * (m + 1); t += NT) {
        const int coord = t & 1, which = (t >> 1) & 1, jj = t >> 2;
        // which 1 (B's interior points) exists only for closed curves
        if (which == 1 && (!closed || jj == 0 || jj == m)) continue;
        const int pick = !closed || jj == 0 || jj == m ? 0 : 1 + which;
        float sum = 0.f;
        for (int kk = 0; kk < K; ++kk) {
            const int i = jj - 3 * Bs[kk];
            if (i < 0 || i > 3) continue;
            const float4 B = Bw[kk];
            const float w = i == 0 ? B.x : i == 1 ? B.y : i == 2 ? B.z : B.w;
            sum = fmaf(w, colsum[3 * (2 * kk + coord) + pick], sum);
        }
        s_cp[which][jj][coord] = sum;
    }
    __syncthreads();
    const int nstore = closed ? 2 * m : m + 1;
    float *out = d_ctrl + 2 * (int64_t)c.ctrl_off[v.id];
    for (int t = lane; t < 2 * nstore; t += NT) {
        const int coord = t & 1, j = t >> 1;
        const int which = j <= m ? 0 : 1;       // A (or open) points, then B's interior
        const int jj = j <= m ? j : j - m;
        out[t] = s_cp[which][jj][coord];
    }
}

__global__ void k_loss_zero(float *loss) {
    if (threadIdx.x == 0) loss[0] = 0.f;
}

// kGrad: also writes the gradient.  status (may be null): nothing is done from
// max_pairs pairs on, where the forward has added up the loss.
template <bool kGrad>
__global__ __launch_bounds__(256) void k_l2(const float *__restrict__ img,
                                            const float *__restrict__ tgt, int64_t n, float scale,
                                            float *__restrict__ d, float *loss,
                                            const int64_t *status, int64_t max_pairs) {
    if (status && status[0] >= max_pairs) return;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    float acc = 0.f;
    // four elements per load where all three arrays are 16-byte aligned
    const bool vec = ((reinterpret_cast<uintptr_t>(img) | reinterpret_cast<uintptr_t>(tgt) |
                       reinterpret_cast<uintptr_t>(d)) & 15) == 0;
    const int64_t n4 = vec ? n / 4 : 0;
    for (int64_t i = t0; i < n4; i += stride) {
        const float4 a = reinterpret_cast<const float4 *>(img)[i];
        const float4 b = reinterpret_cast<const float4 *>(tgt)[i];
        const float4 e = make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
        if (kGrad)
            reinterpret_cast<float4 *>(d)[i] = make_float4(scale * e.x, scale * e.y, scale * e.z,
                                                           scale * e.w);
        acc = fmaf(e.x, e.x, fmaf(e.y, e.y, fmaf(e.z, e.z, fmaf(e.w, e.w, acc))));
    }
    for (int64_t i = 4 * n4 + t0; i < n; i += stride) {
        const float e = img[i] - tgt[i];
        if (kGrad) d[i] = scale * e;
        acc = fmaf(e, e, acc);
    }
    if (loss) {
        __shared__ float s_part[4];
        acc = wave_sum(acc);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(loss, s_part[0] + s_part[1] + s_part[2] + s_part[3]);
    }
}

__global__ void k_counter_reset(uint32_t *counter) {
    if (threadIdx.x == 0) counter[0] = 0u;
}

// Workgroups of a persistent launch: as many as are resident on the device at
// once (occupancy of this kernel and block shape x compute units), at most
// one per tile.  Host queries only (nothing is enqueued), so the launch can be
// captured in a graph.
int persistent_grid(const void *kernel, int threads, size_t lds, int n_tiles) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, lds) != hipSuccess)
        return n_tiles;
    const int64_t blocks = (int64_t)(cus > 0 ? cus : 1) * (per > 0 ? per : 1);
    return blocks < n_tiles ? (int)blocks : n_tiles;
}

// Launch a blend kernel over all tiles: one workgroup per tile, or persistent
// workgroups behind a counter that is cleared first (by a kernel, so that the
// sequence can be captured in a graph).
template <typename K>
void launch_tiles(K kernel, TileArgs &a, const bz_bins &b, const bz_opts &o, int which,
                  int threads, size_t lds, hipStream_t s) {
    if (o.persistent && a.n_tiles > 0) {
        uint32_t *counters = (uint32_t *)b.workspace;     // BinLayout::off_counters == 0
        a.counter = counters + which;
        hipLaunchKernelGGL(k_counter_reset, dim3(1), dim3(64), 0, s, a.counter);
        int grid = persistent_grid(reinterpret_cast<const void *>(kernel), threads, lds,
                                   a.n_tiles);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, s, a);
    } else {
        a.counter = nullptr;
        hipLaunchKernelGGL(kernel, dim3(8 * a.xcd_run * cdiv(a.n_tiles, 8 * a.xcd_run)), dim3(threads), lds, s, a);
    }
}

TileArgs tile_args(const float *rec, const bz_bins &b, const bz_opts &o) {
    TileArgs a = {};
    a.rec = (const float4 *)rec;
    a.ids = b.ids;
    a.ranges = b.ranges;
    a.status = b.status;
    a.W = o.width;
    a.H = o.height;
    if (o.batch) {
        a.canvas = o.batch->canvas;
        a.n_canvas = o.batch->n_canvas;
    }
    a.tile_w = o.tile_w;
    a.tile_h = o.tile_h;
    a.tiles_x = (int)tiles_x(o);
    a.n_tiles = (int)num_tiles(o);
    const int64_t run = a.n_tiles / 64;
    a.xcd_run = (int)(run < 1 ? 1 : run > kXcdRun ? kXcdRun : run);
    a.quads_x = o.tile_w / kQuad;
    a.bg0 = o.bg[0];
    a.bg1 = o.bg[1];
    a.bg2 = o.bg[2];
    a.g_min = o.g_min;
    a.alpha_max = o.alpha_max;
    a.t_min = o.t_min;
    a.inv_1mg = 1.0f / (1.0f - o.g_min);
    a.box_thr = 2.0f * (-logf(o.g_min)) * kCullSlackQuad;
    a.words_per_plane = visit_words_per_plane(o, b.cap_pairs);
    return a;
}

}  // namespace

// Workgroups of an elementwise pass that ends in one atomic each on a single
// word: more than ~256 and those same-address atomics, not HBM, set the time (at
// 2048x2048: 27 us with 256, 33 with 1024, 62 with 4096).
static int64_t l2_blocks(int64_t n) {
    const int64_t blocks = cdiv(n, 4 * 256);
    return blocks > 256 ? 256 : blocks;
}

// Who sums the loss.  The forward's blocks add theirs with one atomic each, 13
// ns one after another on the one word: 140 us at 10,752 tiles, hidden under a
// forward that takes longer (2,048 closed curves at 2040x1344, 257 pairs per tile:
// 265 us, 287 with the sum as a pass of its own) and all of a forward that does
// not (2,048 strokes, 25 pairs per tile: 144 us, 57 with the pass).  Up to
// kLossTiles tiles (27 us of atomics) it is always the blocks; above, the pass
// where there are fewer than kLossPairs pairs per tile, which only the device
// knows.
constexpr int kLossTiles = 2048;
constexpr int64_t kLossPairs = 128;

hipError_t launch_fwd(const float *rec, const bz_bins &b, const bz_opts &o, float *image,
                      const bz_pixstate *st, const L2Out *l2, hipStream_t s) {
    TileArgs a = tile_args(rec, b, o);
    a.image = image;
    int threads = o.tile_w * o.tile_h;
    size_t lds = sizeof(Staged) * (size_t)threads;
    if (l2) {
        a.l2_target = l2->target;
        a.l2_grad = l2->d_image;
        a.l2_loss = l2->loss;
        a.l2_scale = l2->scale;
        a.l2_min_pairs = a.n_tiles > kLossTiles ? kLossPairs * (int64_t)a.n_tiles : 0;
        if (l2->loss && !l2->cleared) hipLaunchKernelGGL(k_loss_zero, dim3(1), dim3(64), 0, s, l2->loss);
    }
    if (st) {
        a.t_final = st->t_final;
        a.n_last = st->n_last;
        a.n_contrib = st->n_contrib;
        a.visit = st->visit;
    }
    const bool count = st && st->n_contrib;
    if (l2) {
        if (!st)
            launch_tiles(k_fwd_l2<false, false>, a, b, o, 0, threads, lds, s);
        else if (count)
            launch_tiles(k_fwd_l2<true, true>, a, b, o, 0, threads, lds, s);
        else
            launch_tiles(k_fwd_l2<true, false>, a, b, o, 0, threads, lds, s);
        if (l2->loss && a.l2_min_pairs > 0) {
            const int64_t n = 3 * num_pixels(o);
            hipLaunchKernelGGL(k_l2<false>, dim3(l2_blocks(n)), dim3(256), 0, s, image, l2->target,
                               n, 0.f, (float *)nullptr, l2->loss, b.status, a.l2_min_pairs);
        }
    } else {
        if (!st)
            launch_tiles(k_fwd<false, false>, a, b, o, 0, threads, lds, s);
        else if (count)
            launch_tiles(k_fwd<true, true>, a, b, o, 0, threads, lds, s);
        else
            launch_tiles(k_fwd<true, false>, a, b, o, 0, threads, lds, s);
    }
    return hipGetLastError();
}

// Sum-table positions of a backward block whose batch masks take vis_bytes of
// LDS (0 for the stored blend state): kTableCap less those bytes, in whole
// multiples of 16 positions, at least 64.
int table_cap(size_t vis_bytes) {
    const int64_t per16 = (int64_t)(sizeof(double) * kSums * 16);
    const int64_t cut = ((int64_t)vis_bytes + per16 - 1) / per16 * 16;
    return kTableCap - cut < 64 ? 64 : (int)(kTableCap - cut);
}

// Do 16 factors 1 / (1 - alpha) at the clamp stay below 2^126?  alpha_max up to 0.9957;
// above, the products are taken in order: backward 98 -> 117 us on 512x512 with 2,048
// strokes, 332 -> 390 on 1024x1024 with 2,000 curves (one lane per pixel and slot by slot
// they were 166 and 451).
static bool factors_fit(float alpha_max) {
    float p = 1.f - alpha_max;
    for (int i = 0; i < 4; ++i) p *= p;
    return p >= 1.1754944e-38f;
}

hipError_t launch_bwd_gauss(const float *rec, int64_t n_gauss, const bz_bins &b,
                            const bz_opts &o, const float *d_image, const bz_pixstate *st,
                            float *d_gauss, bool packed, hipStream_t s, bool cleared) {
    int64_t nz = (int64_t)kGradPlanes * n_gauss;
    if (nz > 0 && !cleared) {
        int64_t blocks = cdiv(nz, 256);
        if (blocks > 16384) blocks = 16384;
        hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, d_gauss, nz);
    }
    TileArgs a = tile_args(rec, b, o);
    a.d_image = d_image;
    a.d_gauss = d_gauss;
    a.packed = packed;
    a.n_gauss = n_gauss;
    int threads = o.tile_w * o.tile_h;
    const size_t vis = st ? 0 : sizeof(uint64_t) * kVisCap * (size_t)(threads / 64);
    a.tab_cap = table_cap(vis);
    size_t lds = sizeof(BwdWave) * (size_t)(threads / 64) + vis +
                 sizeof(double) * kSums * (size_t)(a.tab_cap + kTabPad);
    if (st) {
        a.t_final = st->t_final;
        a.n_last = st->n_last;
        a.visit = st->visit;
    }
    if (factors_fit(o.alpha_max)) {
        if (st) launch_tiles(k_bwd_tiles<false, false>, a, b, o, 1, threads, lds, s);
        else launch_tiles(k_bwd_tiles<true, false>, a, b, o, 1, threads, lds, s);
    } else {
        if (st) launch_tiles(k_bwd_tiles<false, true>, a, b, o, 1, threads, lds, s);
        else launch_tiles(k_bwd_tiles<true, true>, a, b, o, 1, threads, lds, s);
    }
    return hipGetLastError();
}

// Curves from which short ones share waves: four waves per SIMD without sharing.  2,048
// curves of 32 samples and one segment 14.0 -> 12.0 us, but of 24 and three 11.7 ->
// 12.9, where the longest chain counts, not the number of waves.
constexpr int kShareCurves = 4096;

template <bool kPacked>
void launch_curves(const bz_curves &c, const bz_opts &o, const float *rec_f, const float *d_gauss,
                   float *planes, const bz_grads &gr, hipStream_t s) {
    const float4 *rec = reinterpret_cast<const float4 *>(rec_f);
    const double rho = (double)o.rho, inv_rho2 = 1.0 / (rho * rho), s0 = (double)o.sigma0_sq;
    if (c.max_gauss_per_curve > kSmallCurve) {
        const size_t lds = stage2_lds_bytes(c.max_k, c.max_gauss_per_curve);
        hipLaunchKernelGGL((k_bwd_curves<kCurveThreads, kPacked>), dim3(c.n_curves),
                           dim3(kCurveThreads), lds, s, c, c.max_k, c.max_gauss_per_curve, inv_rho2,
                           s0, d_gauss, planes, rec, c.n_gauss, gr.d_ctrl, gr.d_width, gr.d_color,
                           gr.d_opacity);
    }
    if (c.max_gauss_per_curve <= 32 && c.n_curves >= kShareCurves) {
        // K is at most the Gaussian count, however loose a bound max_k is
        const int share = c.max_gauss_per_curve <= 16 ? 4 : 2;
        const int lk = c.max_k < c.max_gauss_per_curve ? c.max_k : c.max_gauss_per_curve;
        const int64_t lds = share * stage2_lds_bytes(lk, c.max_gauss_per_curve);
        hipLaunchKernelGGL((share == 4 ? k_bwd_curves<16, kPacked> : k_bwd_curves<32, kPacked>),
                           dim3((c.n_curves + share - 1) / share), dim3(kWave), lds, s, c, lk,
                           c.max_gauss_per_curve, inv_rho2, s0, d_gauss, planes, rec, c.n_gauss,
                           gr.d_ctrl, gr.d_width, gr.d_color, gr.d_opacity);
        return;
    }
    // a small curve has K <= its Gaussian count <= kSmallCurve
    const int lk = c.max_k < kSmallCurve ? c.max_k : kSmallCurve;
    const int lg = c.max_gauss_per_curve < kSmallCurve ? c.max_gauss_per_curve : kSmallCurve;
    hipLaunchKernelGGL((k_bwd_curves<kWave, kPacked>), dim3(c.n_curves), dim3(kWave),
                       stage2_lds_bytes(lk, lg), s, c, lk, lg, inv_rho2, s0, d_gauss, planes, rec,
                       c.n_gauss, gr.d_ctrl, gr.d_width, gr.d_color, gr.d_opacity);
}

hipError_t launch_bwd_curves(const bz_curves &c, const bz_opts &o, const float *rec,
                             const float *d_gauss, float *planes, const bz_grads &gr,
                             hipStream_t s) {
    if (c.n_curves == 0) return hipSuccess;
    if (planes)
        launch_curves<true>(c, o, rec, d_gauss, planes, gr, s);
    else
        launch_curves<false>(c, o, nullptr, d_gauss, nullptr, gr, s);
    return hipGetLastError();
}

hipError_t launch_l2(const float *image, const float *target, int64_t n, float scale,
                     float *d_image, float *loss, hipStream_t s) {
    if (loss) hipLaunchKernelGGL(k_loss_zero, dim3(1), dim3(64), 0, s, loss);
    if (n > 0) {
        hipLaunchKernelGGL(k_l2<true>, dim3(l2_blocks(n)), dim3(256), 0, s, image, target, n, scale,
                           d_image, loss, (const int64_t *)nullptr, (int64_t)0);
    }
    return hipGetLastError();
}

}  // namespace bz
