// Enumerates the addresses k_direct_conv asks for (csrc/wq_direct_walk.h) over layer shapes, wave tiles
// and slice counts, and reports every access that leaves its buffer.  Exit status: 0 = none.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "wq_direct_walk.h"

static long checked = 0, bad = 0;

static void inside(const char *what, unsigned scalar, unsigned lane, unsigned width, unsigned bytes, const char *layer) {
    ++checked;
    // the scalar part alone must not pass the end either: the range check subtracts it from the size
    if ((unsigned long)scalar + lane + width <= bytes && scalar <= bytes) return;
    if (++bad <= 20) printf("%s: scalar %u + lane %u + %u > %u  (%s)\n", what, scalar, lane, width, bytes, layer);
}

// an operand or scale of pixel `p`, or of none: whatever is not masked must lie inside the data itself,
// margins excluded, and be the pixel the tap asks for
static void pixel(const char *what, unsigned scalar, unsigned lane, unsigned width, unsigned bytes, unsigned margin,
                  bool wanted, unsigned long want, const char *layer) {
    ++checked;
    if (lane >> 31) {
        if (!wanted && scalar <= bytes) return;
    } else if (wanted && scalar <= bytes && (unsigned long)scalar + lane == want + margin &&
               want + width <= bytes - 2ul * margin) {
        return;
    }
    if (++bad <= 20) printf("%s: scalar %u lane %#x wanted %d at %lu, buffer %u  (%s)\n", what, scalar, lane, wanted, want, bytes, layer);
}

template <int KSTEP, bool W4, bool T9>
static void layer(int P, int H, int W, int Cin, int Cout_pad, int g, wq_direct_tile t) {
    using Walk = wq_direct_walk<KSTEP, W4, T9>;
    int log2g = 0;
    while ((1 << log2g) < g) ++log2g;
    const int groups = Cin / g, ob = Cout_pad / 16, G = (T9 ? 9 : 1) * groups;
    const int nOt = (ob + t.no * t.wo - 1) / (t.no * t.wo);
    const unsigned kbW = KSTEP / 4 / (W4 ? 2 : 1);
    char name[160];
    snprintf(name, sizeof name, "P %d W %d %d->%d g%d taps %d w%d tile %dx%d slices %d wo %d wt %d", P, W, Cin, Cout_pad, g,
             T9 ? 9 : 1, W4 ? 4 : 8, t.no, t.nb, t.slices, t.wo, t.wt);
    long steps = 0;
    for (int ks = 0; ks < t.slices; ++ks) {
        Walk at(P, W, Cin, Cout_pad, log2g, ks, t.slices);
        steps += at.steps;
        for (int s = 0; s < at.steps + 7; ++s) {   // the requests past the end repeat the last one
            for (int ob0 = 0; ob0 < nOt * t.no * t.wo; ob0 += t.no)
                for (int e = 0; e < t.no; ++e) {
                    const unsigned o = wq_direct_block(ob0, e, Cout_pad);
                    if (ob0 + e < ob && o != (unsigned)(ob0 + e)) ++bad;
                    inside("weights", at.weights(o), Walk::lane_w(63), kbW, Walk::bytes_w(Cout_pad, Cin), name);
                    inside("weight scales", at.weight_scales(o), Walk::lane_sw(63), 4, Walk::bytes_sw(Cout_pad, groups), name);
                }
            if (t.no == 1 && t.wo == 1 && P <= 400 && s < at.steps) {   // (neither depends on the channel tile)
                const int s0 = (ks * G / t.slices) * (g / KSTEP) + s, tap = s0 / (Cin / KSTEP), kstep = s0 % (Cin / KSTEP);
                for (int p = 0; p < (P + 63) / 64 * 64; ++p) {
                    const int dv = T9 ? tap % 3 - 1 : 0, du = T9 ? tap / 3 - 1 : 0, ww = p % W + dv, hh = p / W % H + du;
                    const bool in = p < P && (!T9 || (ww >= 0 && ww < W && hh >= 0 && hh < H));
                    const unsigned long q = (unsigned long)p + du * W + dv;
                    // (every other row block's mask lies in the upper half, next to another one's)
                    const int half = p / 16 % 2;
                    const unsigned out = Walk::outside(p, H, W) << (16 * half) | 0x1ffu << (16 - 16 * half);
                    for (int quarter = 0; quarter < 4; ++quarter)
                        pixel("codes", at.oX, at.masked(p < P ? Walk::lane_x(quarter, p, P) : 1u << 31, out, half), KSTEP / 4,
                              Walk::bytes_x(P, W, Cin), Walk::back(W) * (KSTEP / 4), in,
                              ((kstep * 4ul + quarter) * P + q) * (KSTEP / 4), name);
                    pixel("scales", at.oSX, at.masked(p < P ? Walk::lane_sx(p) : 1u << 31, Walk::outside(p, H, W)), 4, Walk::bytes_sx(P, W, groups),
                          Walk::back(W) * 4, in, ((unsigned long)(kstep * KSTEP / g) * P + q) * 4, name);
                }
            }
            at.advance();
        }
    }
    if (steps != (long)G * (g / KSTEP) && ++bad) printf("slices do not add up: %s\n", name);
}

template <int KSTEP>
static void shapes(int g) {
    static const int couts[] = {32, 64, 96, 160, 224}, cins[] = {1, 2, 5, 9}, pixels[][3] = {{1, 1, 1}, {7, 1, 7}, {40, 5, 8}, {35, 7, 5}, {66, 2, 11}, {200, 1, 200}, {90, 90, 1}, {10000, 100, 100}};
    static const int tiles[][2] = {{1, 1}, {1, 4}, {2, 4}, {4, 4}}, sl[] = {1, 2, 3, 4, 8, 9, 16};
    for (int c : couts)
        for (int n : cins)
            for (auto &p : pixels) {
                const int P = p[0], H = p[1], W = p[2], Cin = n * g;
                for (int taps = 1; taps <= 9; taps += 8) {
                    wq_direct_tile own = wq_direct_choose_tile(P, c, taps, n, g, KSTEP, 0);
                    for (int k = -1; k < 4 * 7 * 2; ++k) {
                        wq_direct_tile t = own;
                        if (k >= 0) {
                            t = {tiles[k % 4][0], tiles[k % 4][1], sl[k / 4 % 7], 1 + k / 28, 1 + k / 28};
                            if (t.slices > taps * n) continue;
                        }
                        if (taps == 1) layer<KSTEP, false, false>(P, 1, 1, Cin, c, g, t), layer<KSTEP, true, false>(P, 1, 1, Cin, c, g, t);
                        else layer<KSTEP, false, true>(P, H, W, Cin, c, g, t), layer<KSTEP, true, true>(P, H, W, Cin, c, g, t);
                    }
                }
            }
}

// a workgroup's tiles do not lie past the channels where the channels of one tile are all there are
static void narrow() {
    for (int P = 1; P < 500000; P += 1 + P / 7)
        for (int c = 32; c <= 160; c += 32)
            for (int groups : {1, 3, 9, 40})
                for (int taps : {1, 9}) {
                    const wq_direct_tile t = wq_direct_choose_tile(P, c, taps, groups, 64, 64, 0);
                    ++checked;
                    if (((t.no > 1 && t.no * 8 >= c) || (t.wo > 1 && t.no * 16 >= c)) && ++bad <= 20)
                        printf("P %d outputs %d: tile of %d blocks, %d in a workgroup\n", P, c, t.no, t.wo);
                }
}

int main() {
    narrow();
    shapes<32>(32);
    shapes<64>(64);
    shapes<64>(128);
    shapes<64>(512);
    printf("%ld accesses, %ld outside\n", checked, bad);
    return bad != 0;
}
