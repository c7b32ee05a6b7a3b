// How k_direct_conv (wq_direct.hip) cuts a layer into wave tiles, and the addresses a wave walks.
// Plain integer arithmetic without device code, so that a CPU test can enumerate every access of a
// launch against the buffers' sizes.
#pragma once

#ifdef __HIP__
#define WQ_HD __host__ __device__ __forceinline__
#else
#define WQ_HD inline
#endif

// The kernel instance and its launch shape: 16-row blocks per wave along channels and pixels, waves per
// workgroup that split a wave tile's reduction, wave tiles per workgroup along channels and pixels.
struct wq_direct_tile {
    int no, nb, slices, wo, wt;
};

// Wave tile (16-row blocks along channels x pixels) and how many waves share its reduction.  A big
// tile moves fewer operand bytes per product; but a CU takes only 8 waves of it, and a launch is as
// slow as the CU with the most of them.  Measured over layers from 5 to 9792 pixels and 32 to 5120
// channels; n44 = the tiles of 64 x 64:
//   n44 >= 1500      64 x 64; from 3000 on enough waves without sharing a reduction at all (four tiles in
//                    a workgroup, so that its stores and loads stay together)
//   n44 >= 150 (171) 64 x 64 and 4 slices, except 3x3 layers below 640 tiles: there the nine-fold
//                    reduction makes a tile of work so big that 32 x 64 fills the last round better
//                    (2 x 32^2 pixels, 640 -> 640: 26.5 against 29.8 us)
//   n44 >= 40        32 x 64, 8 slices; 3x3 layers of more than six groups up to 170 tiles too, whose four
//                    slices would be longer chains of fp32 additions than nine taps on their own
//                    (2x16x16 1280->1280: relative error 1.29e-7 with 4 slices, 9.3e-8 with 8, 36.3 and
//                    40.1 us; 3x20x19 128->544 g 128, nine groups in all, takes four: 12.1, 16.1 us)
//   fewer            16 x 16 (as long as those are few too), else 16 x 64, 8 slices: latency rules,
//                    every wave should have only a handful of K-steps
//   up to 9 groups   of a linear layer, from 150 tiles: two slices, 32 x 64 below 600 (354x768->3936 g 128
//                    11.2 us, 64 x 64 in four 13.2; 3224x1024->384 g 256 14.1, 15.9), 64 x 64 below 900
//                    (1746x1792->2016 g 256 23.4, 27.9; 32 x 64 28.3); then one, 32 x 64 below 1500
//                    (1817x512->3264 g 128 15.8, 24.4; 64 x 64 17.7), 64 x 64 from there (2356x320->3040
//                    14.9, in two 18.6; 32 x 64 15.6) and for groups of 256 (2681x1536->2067 34.4, 37.6)
//   up to 3 groups   one chain rounds less often than slices and their sum would, so the waves come from
//                    smaller tiles instead: 16 x 16 below 90 tiles (340x192->672 6.3 us, 32 x 64 7.7;
//                    5538x192->64 7.1, 8.3), 16 x 64 below 300 (2699x384->384 9.9, 64 x 64 12.5, 11.1 in four
//                    slices; 2512x512->256 9.3, 12.5), 32 x 64 below 1500 (3516x128->704 9.2, 10.4;
//                    6618x512->832 17.9, 18.5; from there 5441x256->1440 16.9, 16.3).  Three waves with a
//                    long group each, whose fp64 sum rounds as often, where 16 x 16 tiles are few
//                    (223x768->96 g 256 6.7, one chain 7.6)
// No tile is wider than the layer's padded channels, and a workgroup's tiles lie along the pixels where
// one covers all channels: a wave that has no channels of its own costs as much as one that has (us at
// 64 x 64 tiles and 2 x 2 of them in a workgroup, and so: 640^2 pixels 128->24 183, 87; 448^2 64->64 59,
// 41; 50000x640->16 38.6, 32.7).
// `splits`: the slices asked for by a caller, 0 for the choice above.
inline wq_direct_tile wq_direct_choose_tile(int P, int Cout_pad, int taps, int groups, int g, int kstep, int splits) {
    const long ob = Cout_pad / 16, pb = (P + 15) / 16, G = (long)taps * groups;
    const long n44 = ((ob + 3) / 4) * ((pb + 3) / 4);
    wq_direct_tile t = {1, 4, 1, 1, 1};
    if (pb == 1 || (n44 < 40 && ob * pb <= 512)) {
        t.nb = 1;
        t.slices = 8;
        while (t.slices > 4 && ob * pb * t.slices > 2048) t.slices /= 2;
    } else if (n44 < 40) {
        t.slices = 8;
    } else if (n44 < (taps == 9 && groups > 6 ? 171 : 150)) {
        t.no = 2; t.slices = 8;
    } else if (taps == 9 && n44 < 640) {
        t.no = 2;
        t.slices = ((ob + 1) / 2) * ((pb + 3) / 4) > 1024 ? 2 : 4;
    } else if (n44 < 3000 && taps == 1 && G < 10) {
        t.no = n44 < 600 || (n44 >= 900 && n44 < 1500 && g < 256) ? 2 : 4;
        t.slices = n44 < 900 ? 2 : 1;
    } else if (n44 < 1500) {
        t.no = 4; t.slices = 4;
    } else if (n44 < 3000) {
        t.no = 4; t.slices = 2; t.wt = 2;
    } else {
        t.no = 4; t.wo = t.wt = 2;
    }
    if (G < 4 && n44 < 1500 && pb > 1) {
        t.no = n44 < 300 ? 1 : 2;
        t.nb = n44 < 90 ? 1 : 4;
    }
    if (ob <= t.no / 2) t.no /= 2;   // (ob is even, and 2 or more)
    if (t.wo == 2 && ob <= t.no) {
        t.wo = 1; t.wt = 4;
    }
    if (splits > 0) {
        t.slices = splits;
        t.wo = t.wt = 1;
        if (t.slices > 8) t.no = 1;   // the larger tiles' registers allow 8 waves per workgroup
    } else {
        // two K-steps each at least, and a whole group (3x2048->510 g 512 in 8 slices of its four groups 8.3,
        // in four 7.2; 445x2560->128 g 512, five groups, 10.6, 10.1)
        while (t.slices > 1 && (G * g < 2L * kstep * t.slices || t.slices > G)) t.slices /= 2;
        if (G < 4) t.slices = G == 3 && g >= 128 && t.nb == 1 && ob * pb <= 512 ? 3 : 1;
    }
    return t;
}

// The loader's cursor over one slice of a wave tile's reduction: whole groups of the flat sequence
// tap-major, then channels.  Scalar byte offsets into the four buffers; the per-lane parts are below.
template <int KSTEP, bool W4, bool T9>
struct wq_direct_walk {
    static constexpr unsigned KB = KSTEP / 4, BLK = 16 * KSTEP;
    int W, groups, cpg, steps;   // steps: K-steps of the slice
    int t, gam, k, left, col;    // filter tap, group, K-step in the group, K-steps not yet requested, tap's window column
    unsigned blkW, jumpW, stepX, stepSX, stepSW;
    unsigned oW, oSW, shift, oX, oSX;   // shift: pixels from the pixel buffer's start, = back + the tap's shift

    // the pixel buffers start the largest backward shift of a filter tap (a row and a pixel) early, so
    // that shifts are non-negative scalar offsets, and end the largest forward shift late, so that those
    // do not pass the end; nothing is loaded from either margin (see masked)
    static WQ_HD int back(int W) { return T9 ? W + 1 : 0; }
    // which of the 9 window positions of a pixel lie outside the image
    static WQ_HD unsigned outside(unsigned p, unsigned H, unsigned W) {
        if (!T9) return 0;
        const unsigned ww = p % W, hh = (p / W) % H;
        return (hh == 0 ? 0x007u : 0u) | (hh == H - 1 ? 0x1c0u : 0u) | (ww == 0 ? 0x049u : 0u) | (ww == W - 1 ? 0x124u : 0u);
    }
    // a lane's offset at the current tap: bit 31, past the end of every buffer, where the window position
    // lies outside the image (`out`: the positions of two pixels, 16 bits each)
    WQ_HD unsigned masked(unsigned lane, unsigned out, int half = 0) const {
        return T9 ? lane | ((out << (31 - 16 * half - t)) & 0x80000000u) : lane;
    }
    // lane parts
    static WQ_HD unsigned lane_x(int quarter, int p, int P) { return ((unsigned)quarter * (unsigned)P + (unsigned)p) * KB; }
    static WQ_HD unsigned lane_sx(int p) { return (unsigned)p * 4u; }
    static WQ_HD unsigned lane_w(int lane) { return ((unsigned)lane * KB) >> (W4 ? 1 : 0); }
    static WQ_HD unsigned lane_sw(int lane) { return (unsigned)(4 * (lane >> 4) + (lane & 3)) * 4u; }
    // buffer sizes
    static WQ_HD unsigned bytes_x(int P, int W, int Cin) { return (unsigned)P * (unsigned)Cin + 2u * (unsigned)back(W) * KB; }
    static WQ_HD unsigned bytes_sx(int P, int W, int groups) {
        return ((unsigned)P * (unsigned)groups + 2u * (unsigned)back(W)) * 4u;
    }
    static WQ_HD unsigned bytes_w(int Cout_pad, int Cin) {
        return ((T9 ? 9u : 1u) * (unsigned)Cout_pad * (unsigned)Cin) >> (W4 ? 1 : 0);
    }
    static WQ_HD unsigned bytes_sw(int Cout_pad, int groups) {
        return (T9 ? 9u : 1u) * (unsigned)groups * (unsigned)Cout_pad * 4u;
    }

    WQ_HD wq_direct_walk(int P, int W_, int Cin, int Cout_pad, int log2g, int ks, int slices) {
        W = W_;
        groups = Cin >> log2g;
        cpg = (1 << log2g) / KSTEP;
        const int G = (T9 ? 9 : 1) * groups, g_beg = ks * G / slices, g_end = (ks + 1) * G / slices;
        steps = left = (g_end - g_beg) * cpg;
        t = g_beg / groups;
        gam = g_beg - t * groups;
        k = 0;
        blkW = 16u * (unsigned)Cin;
        jumpW = (unsigned)Cout_pad * (unsigned)Cin - blkW;   // next tap's plane
        stepX = 4u * (unsigned)P * KB;
        stepSX = (unsigned)P * 4u;
        stepSW = (unsigned)Cout_pad * 4u;
        oW = (unsigned)t * (unsigned)Cout_pad * (unsigned)Cin + (unsigned)(gam * cpg) * BLK;
        oSW = (unsigned)g_beg * stepSW;
        col = T9 ? t % 3 : 0;
        shift = T9 ? (unsigned)((t / 3) * W + col) : 0u;
        oX = (unsigned)(gam * cpg) * stepX + shift * KB;
        oSX = (unsigned)gam * stepSX + shift * 4u;
    }

    // offsets of the 16-channel block `ob`
    WQ_HD unsigned weights(unsigned ob) const { return (oW + ob * blkW) >> (W4 ? 1 : 0); }
    WQ_HD unsigned weight_scales(unsigned ob) const { return oSW + ob * 64u; }

    // branch-free scalar bookkeeping (a branch here would let the compiler sink the dequantization of
    // all steps in flight to the end of the round, with their sums in registers); stops at the last K-step
    WQ_HD void advance() {
        const bool go = --left > 0;
        k += go ? 1 : 0;
        const bool ng = go && k == cpg;
        k = ng ? 0 : k;
        gam += ng ? 1 : 0;
        const bool nt = T9 && gam == groups;
        gam = nt ? 0 : gam;
        oW += (go ? BLK : 0u) + (nt ? jumpW : 0u);
        oSW += ng ? stepSW : 0u;
        oX += go ? stepX : 0u;
        oSX += ng ? stepSX : 0u;
        if constexpr (T9) {
            t += nt ? 1 : 0;
            const unsigned d = col == 2 ? (unsigned)(W - 2) : 1u;
            shift += nt ? d : 0u;
            col = nt ? (col == 2 ? 0 : col + 1) : col;
            oX = nt ? shift * KB : oX;
            oSX = nt ? shift * 4u : oSX;
        }
    }
};

// The 16-channel blocks of a wave tile that starts at block ob0.  A tile may end past the padded
// channels (a multiple of 32, where a tile has up to 64): such a block reads the last one again and
// is not stored, so that no offset passes the end of the weights.
WQ_HD unsigned wq_direct_block(int ob0, int e, int Cout_pad) {
    const int last = Cout_pad / 16 - 1;
    return (unsigned)(ob0 + e < last ? ob0 + e : last);
}
