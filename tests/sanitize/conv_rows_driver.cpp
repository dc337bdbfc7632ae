// Every slice that the vector convolution kernel reads, replayed on the host from the
// kernel's own index arithmetic (csrc/cnn_rows.h).  Arguments: n h w c k r stride pad.
// For each pixel, class and slice of 8 channels: an accepted read lies inside the
// operand and is the one the convolution's definition gives, and a refused one is
// padding, a slice past K or a row past the last image.
#include <stdio.h>
#include <stdlib.h>

#define __host__
#define __device__
#include "cnn_rows.h"

using namespace bz;

template <int MODE>
static long replay(const Shape &S, int classes, long *reads) {
    GemmArgs g = {};
    g.S = S;
    g.K = S.r * S.r * S.c;
    const long size = MODE == kFwd ? (long)S.n * S.h * S.w * S.c : (long)S.n * S.ho * S.wo * S.k;
    const int per = MODE == kFwd ? S.c : S.k;
    const Divisor image = conv_image<MODE>(S), line = conv_line<MODE>(S);
    long bad = 0;
    for (int z = 0; z < classes; ++z) {
        if (MODE == kBwdData) set_class(g, z);
        const ConvClass cls = {0, conv_steps(g.K), g.cy, g.cx};
        for (int i = 0; i < 4 * cls.steps; ++i) {
            const ConvTab e = conv_tab<MODE>(g, 8 * i);
            const int k = 8 * i, tap = k / per, ch = k % per;
            const int a = MODE == kFwd ? tap / S.r : g.ky0 + tap / g.nkx * S.s;
            const int b = MODE == kFwd ? tap % S.r : g.kx0 + tap % g.nkx * S.s;
            for (int tile = 0; tile < conv_tiles(S, image); ++tile)
                for (int j = 0; j < 16; ++j) {
                    const ConvRow r = conv_row<MODE>(g, image, line, tile, j);
                    const bool in = conv_reads<MODE>(S, r, e);
                    const long at = (long)r.base + e.off;
                    *reads += in;
                    if (in && (at < 0 || at + 8 > size)) {
                        ++bad;                  // outside the operand
                        continue;
                    }
                    // the definition, for the pixel the sums belong to
                    const long out = conv_out<MODE>(g, r, tile, j, cls);
                    long want = -1;
                    if (MODE == kFwd && out >= 0 && out < (long)S.n * S.ho * S.wo) {
                        const long img = out / (S.ho * S.wo), p = out % (S.ho * S.wo);
                        const long y = p / S.wo * S.s - S.p + a, x = p % S.wo * S.s - S.p + b;
                        if (k < g.K && y >= 0 && y < S.h && x >= 0 && x < S.w)
                            want = ((img * S.h + y) * S.w + x) * S.c + ch;
                    } else if (MODE == kBwdData && out >= 0) {
                        const long img = out / (S.h * S.w), p = out % (S.h * S.w);
                        const long y = p / S.w + S.p - a, x = p % S.w + S.p - b;
                        if (k < g.K && y >= 0 && x >= 0 && y / S.s < S.ho && x / S.s < S.wo)
                            want = ((img * S.ho + y / S.s) * S.wo + x / S.s) * S.k + ch;
                    } else {
                        continue;               // no pixel: any slice inside will do
                    }
                    bad += (in ? at : -1) != want;
                }
        }
    }
    return bad;
}

// The lanes' first 16-byte pieces in every block of 16 nb output channels of n: pixel and
// piece inside the tile (the sanitizer sees a division by zero).
template <int MODE>
static long pieces(int n, int nb) {
    long bad = 0;
    for (int n0 = 0; n0 < n; n0 += 16 * nb) {
        const int nc = n - n0 < 16 * nb ? n - n0 : 16 * nb;
        const int per = conv_pieces<MODE>(nc);
        for (int lane = 0; lane < 64; ++lane)
            bad += lane / per * per + lane % per != lane;
        if (nc * (MODE == kFwd ? 2 : 4) % 16 == 0)
            bad += per * 16 != nc * (MODE == kFwd ? 2 : 4);
    }
    return bad;
}

int main(int argc, char **argv) {
    if (argc != 9) return 2;
    int v[8];
    for (int i = 0; i < 8; ++i) v[i] = atoi(argv[1 + i]);
    Shape S = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], 0, 0};
    S.ho = (S.h + 2 * S.p - S.r) / S.s + 1;
    S.wo = (S.w + 2 * S.p - S.r) / S.s + 1;
    long fwd = 0, bwd = 0, bad_bwd = 0;
    const long bad_fwd = replay<kFwd>(S, 1, &fwd);
    if (S.k % 8 == 0) bad_bwd = replay<kBwdData>(S, S.s * S.s, &bwd);
    for (int nb = 1; nb <= 4; nb += 3) {
        bad_bwd += pieces<kBwdData>(S.c, nb);
        if (pieces<kFwd>(S.k, nb)) return 3;
    }
    printf("forward: %ld reads, %ld wrong; input gradient: %ld reads, %ld wrong\n", fwd, bad_fwd, bwd,
           bad_bwd);
    return bad_fwd || bad_bwd;
}
