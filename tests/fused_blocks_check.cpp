// Enumerates the workgroups of a launch of the fused kernel (csrc/wq_fused_blocks.h).
//   no arguments: over layer shapes and workgroup tiles, every block of tiles and channels once.  Exit status: 0 = so.
//   T_pad Cout_pad Cin n nt no: prints how that launch is cut: mode band width-of-the-last-band
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "wq_fused_blocks.h"

static long launches[3][3], bad = 0;   // by mode; bands: none, even, the last one narrower

static int last_band(const wq_fused_blocks &b) {
    const int others = b.mode == 0 ? b.nTB : b.nOB;
    return b.mode == 2 || others % b.band == 0 ? b.band : others % b.band;
}

static void launch(int T_pad, int Cout_pad, int Cin, int n, int nt, int no) {
    const wq_fused_blocks b = wq_fused_launch_blocks(T_pad, Cout_pad, Cin, n, nt, no);
    std::vector<int> times((size_t)b.nTB * b.nOB);
    const unsigned grid = wq_fused_grid(b);
    bool ok = b.nTB * 16 * nt == T_pad && b.nOB * 16 * no == Cout_pad && b.band >= 1;
    for (unsigned id = 0; id < grid && ok; ++id) {
        int tb = -1, ob = -1;
        wq_fused_block(b, (int)id, tb, ob);
        if (tb < 0 || ob < 0) ok = false;
        else if (tb < b.nTB && ob < b.nOB) ++times[(size_t)tb * b.nOB + ob];
    }
    for (int t : times) ok = ok && t == 1;
    const int others = b.mode == 0 ? b.nTB : b.nOB;
    ++launches[b.mode][b.mode == 2 || b.band == others ? 0 : last_band(b) == b.band ? 1 : 2];
    if (!ok && ++bad <= 20) printf("T_pad %d Cout_pad %d Cin %d n %d tile %dx%d: mode %d band %d\n", T_pad, Cout_pad, Cin, n, nt, no, b.mode, b.band);
}

int main(int argc, char **argv) {
    if (argc == 7) {
        int v[6];
        for (int i = 0; i < 6; ++i) v[i] = atoi(argv[i + 1]);
        const wq_fused_blocks b = wq_fused_launch_blocks(v[0], v[1], v[2], v[3], v[4], v[5]);
        printf("%d %d %d\n", b.mode, b.band, last_band(b));
        return 0;
    }
    const int tiles[] = {32, 64, 96, 160, 224, 320, 480, 608, 1184, 1248, 2048, 4704, 10016}, chans[] = {32, 64, 96, 160, 288, 320, 448, 640, 928, 1184, 1280, 2560};
    const int cins[] = {32, 64, 96, 128, 192, 256, 320, 512, 704, 960, 1280, 2560};
    for (int n : {4, 6, 8})
        for (int T_pad : tiles)
            for (int Cout_pad : chans)
                for (int Cin : cins) {
                    launch(T_pad, Cout_pad, Cin, n, 1, 1);
                    launch(T_pad, Cout_pad, Cin, n, 2, 1);
                    launch(T_pad, Cout_pad, Cin, n, 2, 2);
                }
    for (int m = 0; m < 3; ++m)
        for (int k = 0; k < (m == 2 ? 1 : 3); ++k)
            if (!launches[m][k]) ++bad, printf("no launch of mode %d with bands of kind %d\n", m, k);
    printf("%ld faults\n", bad);
    return bad != 0;
}
