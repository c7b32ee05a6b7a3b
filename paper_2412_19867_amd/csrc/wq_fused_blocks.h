// Which block of tiles and of output channels a workgroup of the fused kernel (k_contract_output) works on.
// Plain integer arithmetic without device code, so that a CPU test can enumerate every launch.
#pragma once

#ifdef __HIP__
#define WQ_HD __host__ __device__ __forceinline__
#else
#define WQ_HD inline
#endif

// How the fused kernel's workgroups are shared out to the eight XCDs: 0 = every 8th block of output
// channels each, 1 = every 8th block of tiles (whichever operand is larger), 2 = every 4th block of tiles
// and one half of the channels: where all taps' weights would fill an XCD's 4 MB L2 on their own, half of
// them stays resident next to the streaming activations.  nOB: blocks of output channels.
inline int wq_fused_xcd_mode(int T_pad, int Cout_pad, int Cin, int n, int nOB) {
    const long wbytes = (long)Cout_pad * Cin, xbytes = (long)T_pad * Cin, wall = wbytes * n * n;
    if (wbytes >= xbytes) return 0;
    return wall > (5L << 19) && wall <= (8L << 20) && nOB >= 2 ? 2 : 1;
}

// A launch's blocks (nTB of tiles x nOB of channels) and their order.  band: how many blocks of the operand that
// the XCDs do not share out pass before an XCD's own blocks change.
struct wq_fused_blocks {
    int nTB, nOB, mode, band;
};

// nt, no: 16-row blocks of tiles and of channels per workgroup
inline wq_fused_blocks wq_fused_launch_blocks(int T_pad, int Cout_pad, int Cin, int n, int nt, int no) {
    wq_fused_blocks b;
    b.nTB = T_pad / (16 * nt);
    b.nOB = Cout_pad / (16 * no);
    b.mode = wq_fused_xcd_mode(T_pad, Cout_pad, Cin, n, b.nOB);
    // all blocks where they fit an XCD's 4 MB L2 (all taps of them), otherwise bands of 1 MB
    const long bytes = (long)n * n * Cin * 16 * (b.mode == 0 ? nt : no);
    const int others = b.mode == 0 ? b.nTB : b.nOB, fit = (int)((1L << 20) / bytes);
    b.band = others * bytes <= (4L << 20) ? others : fit > 1 ? fit : 1;
    return b;
}

inline unsigned wq_fused_grid(const wq_fused_blocks &b) {
    if (b.mode == 2) return (unsigned)(((b.nTB + 3) / 4) * ((b.nOB + 1) / 2) * 8);
    const int split = b.mode == 0 ? b.nOB : b.nTB, other = b.mode == 0 ? b.nTB : b.nOB;
    return (unsigned)(((split + 7) / 8) * 8 * other);
}

// the blocks of workgroup `id`; past the last ones (tb >= nTB or ob >= nOB) it has none
WQ_HD void wq_fused_block(const wq_fused_blocks &b, int id, int &tb, int &ob) {
    const int xcd = id & 7, s = id >> 3;
    if (b.mode != 2) {
        // in bands of the other operand's blocks: all of the XCD's own blocks pass a band while it is in the L2
        const bool channels = b.mode == 0;
        const int others = channels ? b.nTB : b.nOB, own = ((channels ? b.nOB : b.nTB) + 7) >> 3;
        const int first = s / (own * b.band) * b.band, r = s - first * own;
        const int width = b.band < others - first ? b.band : others - first;
        const int mine8 = (r / width) * 8 + xcd, other = first + r % width;
        ob = channels ? mine8 : other;
        tb = channels ? other : mine8;
    } else {   // 4 parts of the tiles x 2 halves of the channels
        const int hob = (b.nOB + 1) >> 1;
        tb = (s / hob) * 4 + (xcd >> 1);
        ob = (xcd & 1) * hob + s % hob;
    }
}
