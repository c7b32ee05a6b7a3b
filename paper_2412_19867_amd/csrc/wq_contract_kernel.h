// Stages 2+3 for gfx950: the Winograd-domain contraction as int8 MFMA GEMMs
// with per-group dequantization, and the output transform y = A^T Y A + bias
// fused behind it, so the n*n fp32 Winograd-domain planes never reach memory.
//
// Work decomposition
//   workgroup  = one (16*NT tiles) x (16*NO output channels) block, ALL n*n taps;
//   wave       = (tap row i, K slice ks): taps i*n .. i*n+n-1 over 1/KS of the
//                input channels (whole quantization groups);  n*KS waves.
// A wave walks a flat sequence of K-steps (tap-major, then channels):
//   int32 block  = MFMA(Wq block, Xq block)       exact, fresh per group
//   M           += float(block) * (sW[o] * sX[tile])     at the end of each group
// A operand = 16 output channels, B operand = 16 tiles.  Both tensors are stored
// in the blocked operand order (include/wq.h), so one K-step of one 16-row block
// is 16*KSTEP contiguous bytes and every lane fetches KB bytes at lane*KB; the
// exact integer sum does not depend on how the instruction orders K as long as
// A and B use the same order, which they do.  Operands and scales are fetched D
// K-steps ahead into registers with buffer loads whose running offsets are
// scalar.  At the end of a tap the wave folds M into R[b] += A^T[b][j] * M (its
// share of row i of Y A); after its n taps R goes through LDS and the workgroup
// finishes Y[a][b] = sum_i A^T[a][i] (sum_ks R_{i,ks}[b]), adds bias and stores
// NHWC with the ragged right/bottom edge masked.
//
// What bounds it: a 1 KiB operand load costs the CU's load path 17 cycles, one of a word per lane 8, and a SIMD
// issues a block's 12 dequantization instructions and its MFMA in 46 (the two do not overlap).  With NT x NO
// blocks of operands per wave the load path takes 17 (NT + NO) / (NT NO) cycles of a CU per block, 34 with one
// and 17 with four, against 11.5 of its four SIMDs.
//
// A wave waits for nothing but its own loads, so what counts is that the compiler can count them:
// the request of the K-step D ahead is unconditional, a walk is whole rounds of n K-steps, and the request
// is placed between the MFMAs and the dequantization, which covers their latency.  The last
// round is written out without the requests past its end: a walk has only (m + 2) Cin / K-step steps, so those
// would cost up to a half more (whole forward with and without: 29x43x43 64->992 F(2,3), one
// round, 201, 130 us; 8x78x78 192->512 F(2,3) 168, 135).
//
// Scales of groups of one K-step: a round's scales of n groups come in one load per tensor straight into LDS
// that is the wave's own (no barrier: the wave's count of loads in flight says when they are there), a round
// ahead, and reach the lanes as broadcast LDS reads, which cost neither the load path nor the vector ALU
// anything.  (One word per lane, load and K-step, spread by DPP, took two of five loads, and one DPP
// instruction in twelve keeps the SIMD from issuing for two waves at once: 2.9 -> 4.4 cycles an instruction.)
// This kernel alone under a trace, with that form and now, one, two and four blocks: 2x128x128 320->320 F(4,3)
// 54.4, 48.2, 51.2 -> 53.7, 46.5, 44.5 us (46 with plain stores of y, in a chain of such layers); 32x56x56 64->64
// F(6,3) 18.3, 16.3, 16.6 -> 18.0, 16.7, 14.9; 1x32x32 64->64 F(4,3), one block, 5.3 -> 5.2.  Longer groups keep the
// DPP form.
//
// Workgroups are numbered so that the eight XCDs (which receive consecutive
// workgroup ids round-robin and have private L2s) each own a slice of the
// larger operand: with xcd_mode 0 an XCD owns every 8th block of output
// channels (weights stay in its L2), with xcd_mode 1 every 8th block of tiles,
// with xcd_mode 2 every 4th block of tiles and one half of the channels.  Where the other operand does not fit
// that L2 it passes in bands of 1 MB (all of the XCD's own blocks meet a band before the next comes).  Whole forward
// without and with, one, two and four blocks: 5x64x64 448->992 F(4,3) 217, 140, 131 -> 143, 125, 102 us; 5x96x96 448->992
// F(6,3) 388, 244, 232 -> 267, 212, 180; 2x96x96 512->640 152, 114, 100 -> 107, 99, 88.
#pragma once

#include <type_traits>

#include "wq_device.h"
#include "wq_internal.h"

namespace {   // every including file instantiates its own tile size; nothing here is exported

// K-steps in flight of a wave, a divisor of the taps of a row.  Two with four blocks per wave, and with two of
// F(6,3) at K 64: two workgroups then fit a CU where the registers of more in flight leave one.
template <int M, int NT, int NO, bool K64 = true>
constexpr int kDepth = NT * NO == 4 || (M == 6 && NT * NO == 2 && K64) ? 2 : (M == 4 ? 3 : 4);

// the instances that Args::plain_y is for
template <int M, int NT, int NO>
constexpr bool kPlainY = M == 4 && NT == 2 && NO == 2;

struct Args {
    wq_xf xf;
    const int8_t *Xq;
    const float *sX;
    const int8_t *Wq;
    const float *sW;
    const float *bias;
    float *y;
    wq_dump dump;   // debug calls: where to store the int32 group sums (P == nullptr otherwise)
    int H, W, Cin, Cout, TH, TW, T, T_pad, Cout_pad, log2g;
    wq_fused_blocks blocks;
    // Store y with plain instead of streaming stores: the next layer's input kernel finds 32 to 56 MB in the caches.
    // Whole forward with four blocks, streaming and plain, in a chain of such layers and on other buffers each time:
    // 24 MB (2x96x96 320->320) 40.4, 39.4 and 38.2, 39.1 us; 42 MB (2x128x128) 64.0, 61.3 and 59.6, 60.4; 55 MB
    // (2x128x104 512->512) 97.8, 93.7 and 91.0, 91.9; 63 MB (3x128x128 320->320) 85.7, 83.2 and 78.7, 86.1; 126 MB
    // 159, 168 and 157, 162.
    int plain_y;
    int dense_rows;   // see wq_plan
};

template <bool K64, int NT, int NO>
struct Stage {
    v4i a[NO], b[NT];   // K64: 16 operand bytes per lane; otherwise .xy only
    float sw[NO];       // longer groups: weight scale of channel 4 q + lane % 4 of each sub-block
    float sx;           // and activation scale of tile lane % (16 NT)
};

template <int M, bool K64, bool CPG1, bool WIDE, bool ATSP, bool DUMP, int NT, int NO, int KS, int D, bool ONE>
__global__ __launch_bounds__(64 * (M + 2) * KS) void k_contract_output(const Args a) {
    constexpr int n = M + 2;
    static_assert(n % D == 0, "a tap row is a whole number of rounds of the ring");
    // an int32 block that starts at kMagic converts by a subtraction (groups of one K-step: |sum| < 2^21)
    constexpr bool MAGIC = CPG1;
    constexpr int KSTEP = K64 ? 64 : 32;   // K per MFMA
    constexpr int KB = KSTEP / 4;          // operand bytes per lane per MFMA
    constexpr int NW = n * KS;             // waves
    constexpr int RS = 16 * NO + 4;              // floats per tile row of the exchange (the channels + pad)
    constexpr int RSW = 16 * RS;                 // floats of one wave's column
    // output columns per LDS pass: all M, or half of them (with two channel blocks their stores then fill
    // lines of 128 bytes)
    constexpr int BP = ONE ? M : M / 2;
    constexpr int SLOT = 2048;                   // bytes of a wave's scales of one round: 1 KiB per tensor
    static_assert(n * 16 * (NO > NT ? NO : NT) * 4 <= 1024, "a round's scales are one wave-wide load per tensor");
    constexpr int LDS_BYTES = NW * (BP * RSW * 4 > 2 * SLOT || !CPG1 ? BP * RSW * 4 : 2 * SLOT);
    // the scales of the rounds in flight while the walk lasts, then the exchange of the row sums
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    float *const Rs = reinterpret_cast<float *>(lds);

    // ---- which block (uniform) ----
    int tb, ob;
    wq_fused_block(a.blocks, blockIdx.x, tb, ob);
    if (tb >= a.blocks.nTB || ob >= a.blocks.nOB) return;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = w % n, ks = w / n;   // tap row, K slice (uniform)
    const int tau0 = tb * 16 * NT, o0 = ob * 16 * NO;
    const int Cin = a.Cin, Cout_pad = a.Cout_pad, T_pad = a.T_pad;
    const int groups = Cin >> a.log2g;
    const int gps = groups / KS;                 // groups per K slice
    const int cps = (Cin / KSTEP) / KS;          // K-steps per tap for this wave
    const int cpg_mask = ((1 << a.log2g) / KSTEP) - 1;

    const unsigned n2 = n * n;
    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t *>(a.Wq), 0, (int)(n2 * (unsigned)Cout_pad * (unsigned)Cin), kBufFlags);
    const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t *>(a.Xq), 0, (int)(n2 * (unsigned)T_pad * (unsigned)Cin), kBufFlags);
    const __amdgpu_buffer_rsrc_t rSW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.sW), 0, (int)(n2 * (unsigned)groups * (unsigned)Cout_pad * 4u),
        kBufFlags);
    const __amdgpu_buffer_rsrc_t rSX = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.sX), 0, (int)(n2 * (unsigned)T_pad * (unsigned)groups * 4u),
        kBufFlags);
    // per-lane byte offsets inside a tap plane (sub-block 0); the tap/K position is scalar
    const int vW = o0 * Cin + lane * KB;
    const int vX = tau0 * Cin + lane * KB;
    const int vSW = (o0 + 4 * q + (lane & 3)) * 4;          // sW [tap][group][Cout_pad]
    const int vSX = ((tau0 >> 4) + ((lane >> 4) & (NT - 1))) * groups * 64 + l16 * 4;   // sX [tap][16-tile block][group][16]
    const unsigned planeW = (unsigned)Cout_pad * Cin, planeX = (unsigned)T_pad * Cin;
    const unsigned planeSW = (unsigned)groups * Cout_pad * 4, planeSX = (unsigned)T_pad * groups * 4;
    constexpr unsigned stepOp = 16 * KSTEP;                 // bytes of one K-step of a 16-row block
    const unsigned stepSW = (unsigned)Cout_pad * 4;
    // scalar running offsets of the loader, and what to add when it wraps to the next tap
    const unsigned t0 = (unsigned)(i * n);
    unsigned oW = t0 * planeW + (unsigned)(ks * cps) * stepOp;
    unsigned oX = t0 * planeX + (unsigned)(ks * cps) * stepOp;
    unsigned oSW = t0 * planeSW + (unsigned)(ks * gps) * stepSW;
    unsigned oSX = t0 * planeSX + (unsigned)(ks * gps) * 64u;
    const unsigned dW = planeW - (unsigned)cps * stepOp, dX = planeX - (unsigned)cps * stepOp;
    const unsigned dSW = planeSW - (unsigned)gps * stepSW, dSX = planeSX - (unsigned)gps * 64u;
    int k_ld = 0, kg_ld = 0;

    auto load_stage = [&](Stage<K64, NT, NO> &s) {
#pragma unroll
        for (int no = 0; no < NO; ++no) {
            if constexpr (K64) {
                s.a[no] = __builtin_amdgcn_raw_buffer_load_b128(rW, vW + no * 16 * Cin, oW, 0);
            } else {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rW, vW + no * 16 * Cin, oW, 0);
                s.a[no] = v4i{t.x, t.y, 0, 0};
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (K64) {
                s.b[nt] = __builtin_amdgcn_raw_buffer_load_b128(rX, vX + nt * 16 * Cin, oX, 0);
            } else {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rX, vX + nt * 16 * Cin, oX, 0);
                s.b[nt] = v4i{t.x, t.y, 0, 0};
            }
        }
        if constexpr (!CPG1) {
#pragma unroll
            for (int no = 0; no < NO; ++no)
                s.sw[no] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rSW, vSW, oSW + 64u * no, 0));
            s.sx = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rSX, vSX, oSX, 0));
        }
        // branch-free scalar bookkeeping
        ++k_ld;
        ++kg_ld;
        const bool next_group = (kg_ld & cpg_mask) == 0, next_tap = k_ld == cps;
        k_ld = next_tap ? 0 : k_ld;
        oW += stepOp + (next_tap ? dW : 0u);
        oX += stepOp + (next_tap ? dX : 0u);
        if constexpr (!CPG1) {
            oSW += (next_group ? stepSW : 0u) + (next_tap ? dSW : 0u);
            oSX += (next_group ? 64u : 0u) + (next_tap ? dSX : 0u);
        }
    };

    // ---- scales of groups of one K-step: n groups of the walk a round, loaded into the wave's own LDS ----
    // One load per tensor and round; lane l fetches four channels (tiles) of the round's group l / (4 NO)
    // (l / (4 NT)).  `at`: that group's position in its tap, `off`: its byte offset.
    char *const mine = lds + w * (2 * SLOT);
    struct ScaleWalk {
        int at;
        unsigned off;
    };
    auto scale_walk = [&](int gl, unsigned lane_off, unsigned base, unsigned plane, unsigned step) {
        ScaleWalk c;
        const int tap = gl / gps;
        c.at = gl - tap * gps;
        c.off = gl < n ? base + (unsigned)tap * plane + (unsigned)c.at * step + lane_off : kPastEnd;
        return c;
    };
    ScaleWalk cW = {}, cX = {};
    const int skip_taps = n / gps, skip_groups = n - skip_taps * gps;   // n groups further on
    if constexpr (CPG1) {
        cW = scale_walk(lane / (4 * NO), (unsigned)(o0 + 4 * (lane % (4 * NO))) * 4u, oSW, planeSW, stepSW);
        const int tile = 4 * (lane % (4 * NT));   // sX [tap][16-tile block][group][16]
        cX = scale_walk(lane / (4 * NT), (unsigned)(((tau0 + tile) >> 4) * groups * 64 + (tile & 15) * 4), oSX, planeSX, 64u);
    }
    auto load_scales = [&](int slot) {
        lds_load16(rSW, mine + slot * SLOT, cW.off, 0);
        lds_load16(rSX, mine + slot * SLOT + 1024, cX.off, 0);
        auto advance = [&](ScaleWalk &c, unsigned plane, unsigned step) {   // (past its last tap a wave loads what it never reads)
            c.at += skip_groups;
            const bool wrap = c.at >= gps;
            c.at -= wrap ? gps : 0;
            c.off += (unsigned)skip_taps * plane + (unsigned)skip_groups * step + (wrap ? plane - (unsigned)gps * step : 0u);
        };
        advance(cW, planeSW, stepSW);
        advance(cX, planeSX, 64u);
    };

    float4 R[M][NO][NT];
#pragma unroll
    for (int b = 0; b < M; ++b)
#pragma unroll
        for (int no = 0; no < NO; ++no)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) R[b][no][nt] = make_float4(0.f, 0.f, 0.f, 0.f);

    if constexpr (CPG1) {
        load_scales(0);
        __builtin_amdgcn_sched_barrier(0);
    }
    Stage<K64, NT, NO> st[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {   // in the order the loop expects them back
        load_stage(st[d]);
        __builtin_amdgcn_sched_barrier(0);
    }

    // compute cursor (uniform)
    int j_cp = 0, k_left = cps, kg_cp = 0, gam_cp = 0, in_chunk = 0;
    v4i acc[NO][NT];
    float4 Mc[NO][NT];
    double Mt[NO][NT][4];
#pragma unroll
    for (int no = 0; no < NO; ++no)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            acc[no][nt] = v4i{0, 0, 0, 0};
            Mc[no][nt] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int r = 0; r < 4; ++r) Mt[no][nt][r] = 0.0;
        }
    float atc[M];
#pragma unroll
    for (int b = 0; b < M; ++b) atc[b] = a.xf.AT[b * n];   // column of tap j = 0

    const v4i magic = {kMagic, kMagic, kMagic, kMagic};
    // (no exit test and no run-time condition on a request inside a round: with either of them the
    // compiler cannot count the loads in flight and waits for all of them at the top of every round)
    int slot = 0;
    auto round = [&](auto last) {
        const char *sc = mine + slot * SLOT;
        if constexpr (CPG1) {
            if constexpr (!last.value) load_scales(slot ^ 1);
            slot ^= 1;
            // everything but the operands in flight (and the scales just asked for) has landed: this round's scales
            wait_loads<D * (NT + NO) + (last.value ? 0 : 2)>();
        }
#pragma unroll
        for (int step = 0; step < n; ++step) {
            Stage<K64, NT, NO> &s = st[step % D];
            v4f sw4[NO];
            float sx1[NT];
            if constexpr (CPG1) {
#pragma unroll
                for (int no = 0; no < NO; ++no)
                    sw4[no] = *reinterpret_cast<const v4f *>(sc + (step * NO + no) * 64 + q * 16);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    sx1[nt] = *reinterpret_cast<const float *>(sc + 1024 + (step * NT + nt) * 64 + l16 * 4);
            }
            const bool group_end = CPG1 || ((++kg_cp & cpg_mask) == 0);
#pragma unroll
            for (int no = 0; no < NO; ++no)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const v4i c0 = MAGIC ? magic : acc[no][nt];
                    if constexpr (K64) {
                        acc[no][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(s.a[no], s.b[nt], c0, 0, 0, 0);
                    } else {
                        const long av = __builtin_bit_cast(long, v2i{s.a[no].x, s.a[no].y});
                        const long bv = __builtin_bit_cast(long, v2i{s.b[nt].x, s.b[nt].y});
                        acc[no][nt] = __builtin_amdgcn_mfma_i32_16x16x32_i8(av, bv, c0, 0, 0, 0);
                    }
                }
            // the scales of longer groups leave the stage, whose registers are then refilled while the MFMAs run
            if constexpr (!CPG1) {
                spread_rows<NT>(s.sx, sx1);
#pragma unroll
                for (int no = 0; no < NO; ++no)
                    sw4[no] = v4f{quad_bcast<0>(s.sw[no]), quad_bcast<1>(s.sw[no]), quad_bcast<2>(s.sw[no]), quad_bcast<3>(s.sw[no])};
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!last.value) load_stage(s);   // D steps ahead
            else if (step + D < n) load_stage(s);
            __builtin_amdgcn_sched_barrier(0);
            if (group_end) {
#pragma unroll
                for (int no = 0; no < NO; ++no)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        Mc[no][nt].x = __builtin_fmaf(group_sum<MAGIC>(acc[no][nt][0]), sw4[no].x * sx1[nt], Mc[no][nt].x);
                        Mc[no][nt].y = __builtin_fmaf(group_sum<MAGIC>(acc[no][nt][1]), sw4[no].y * sx1[nt], Mc[no][nt].y);
                        Mc[no][nt].z = __builtin_fmaf(group_sum<MAGIC>(acc[no][nt][2]), sw4[no].z * sx1[nt], Mc[no][nt].z);
                        Mc[no][nt].w = __builtin_fmaf(group_sum<MAGIC>(acc[no][nt][3]), sw4[no].w * sx1[nt], Mc[no][nt].w);
                        if constexpr (DUMP) {   // the debug entry point's instance of this kernel
                            constexpr int off = MAGIC ? kMagic : 0;
                            const int v[4] = {acc[no][nt][0] - off, acc[no][nt][1] - off, acc[no][nt][2] - off,
                                              acc[no][nt][3] - off};
                            wq_dump_store(a.dump, i * n + j_cp, tau0 + nt * 16 + l16,
                                          ks * gps + gam_cp, groups, o0 + no * 16 + 4 * q, a.Cout,
                                          a.T, v);
                        }
                        if constexpr (!CPG1) acc[no][nt] = v4i{0, 0, 0, 0};
                    }
                ++gam_cp;
                if (WIDE && ++in_chunk == 4) {   // fp64 totals of 4-group fp32 chunks (long reductions)
                    in_chunk = 0;
#pragma unroll
                    for (int no = 0; no < NO; ++no)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            Mt[no][nt][0] += (double)Mc[no][nt].x;
                            Mt[no][nt][1] += (double)Mc[no][nt].y;
                            Mt[no][nt][2] += (double)Mc[no][nt].z;
                            Mt[no][nt][3] += (double)Mc[no][nt].w;
                            Mc[no][nt] = make_float4(0.f, 0.f, 0.f, 0.f);
                        }
                }
            }
            if (--k_left == 0) {   // end of tap j_cp: fold into (this slice's share of) row i of Y A
                k_left = cps;
                gam_cp = 0;
                in_chunk = 0;
                // branch-free on purpose: entries of A^T that are zero simply add nothing
#pragma unroll
                for (int no = 0; no < NO; ++no)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        float4 Mv = Mc[no][nt];
                        if constexpr (WIDE) {
                            Mv = make_float4((float)(Mt[no][nt][0] + (double)Mv.x),
                                             (float)(Mt[no][nt][1] + (double)Mv.y),
                                             (float)(Mt[no][nt][2] + (double)Mv.z),
                                             (float)(Mt[no][nt][3] + (double)Mv.w));
#pragma unroll
                            for (int r = 0; r < 4; ++r) Mt[no][nt][r] = 0.0;
                        }
                        Mc[no][nt] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int b = 0; b < M; ++b) {
                            float4 &Rb = R[b][no][nt];
                            Rb.x = __builtin_fmaf(atc[b], Mv.x, Rb.x);
                            Rb.y = __builtin_fmaf(atc[b], Mv.y, Rb.y);
                            Rb.z = __builtin_fmaf(atc[b], Mv.z, Rb.z);
                            Rb.w = __builtin_fmaf(atc[b], Mv.w, Rb.w);
                        }
                    }
                ++j_cp;
                const int jn = j_cp < n ? j_cp : 0;
#pragma unroll
                for (int b = 0; b < M; ++b) atc[b] = a.xf.AT[b * n + jn];
            }
        }
    };
    for (int it = cps - 1; it > 0; --it) round(std::false_type{});
    round(std::true_type{});

    // ---- output transform across tap rows, 16 tiles and BP columns at a time ----
    // A thread forms V neighbouring channels of one column of a tile.  Four with two channel blocks (a store
    // instruction covers 8 lines of 128 bytes: 2x128x128 320->320 44.6 us, with one channel per thread 48.7; 32x56x56
    // 64->64 F(6,3) 15.0, 15.9), one with a single block (4 half lines, against 16 half lines).
    auto finish = [&](auto vec, auto plain, int nt, int p) {
        constexpr int V = decltype(vec)::value, Q = 16 * NO / V, PC = 16 * Q;   // PC threads form a column
        constexpr int TH = 64 * NW, COLS = TH >= PC ? TH / PC : 1;              // columns at a time
        if (TH >= PC && tid >= COLS * PC) return;
        for (int pos = TH >= PC ? tid % PC : tid; pos < PC; pos += TH >= PC ? PC : TH) {
            const int ch = (pos % Q) * V, tl = pos / Q;
            const int tau = tau0 + nt * 16 + tl, o = o0 + ch;
            if (tau >= a.T || o >= a.Cout) continue;
            const int tw = tau % a.TW, th = (tau / a.TW) % a.TH, bb = tau / (a.TW * a.TH);
            const int hv = min(M, a.H - th * M), wv = min(M, a.W - tw * M);
            float bias[V];
#pragma unroll
            for (int v = 0; v < V; ++v) bias[v] = a.bias[o + v];   // (padded to Cout_pad)
            float *const base = a.y + ((size_t)(bb * a.H + th * M) * a.W + tw * M) * a.Cout + o;
            for (int bp = TH >= PC ? tid / PC : 0; bp < BP; bp += COLS) {
                const int b = p * BP + bp;
                if (b >= wv) break;
                float rv[V][n], Yv[V][M];
#pragma unroll
                for (int ii = 0; ii < n; ++ii) {
                    const float *src = Rs + (ii * BP + bp) * RSW + tl * RS + ch;
#pragma unroll
                    for (int v = 0; v < V; ++v) rv[v][ii] = src[v];
#pragma unroll
                    for (int k2 = 1; k2 < KS; ++k2)
#pragma unroll
                        for (int v = 0; v < V; ++v) rv[v][ii] += src[k2 * n * BP * RSW + v];
                }
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (M == 4 && a.dense_rows) wq_apply_at<M, false>(a.xf, rv[v], Yv[v]);
                    else wq_apply_at<M, ATSP>(a.xf, rv[v], Yv[v]);
                }
                float *const dst = base + b * a.Cout;
#pragma unroll
                for (int aa = 0; aa < M; ++aa) {
                    if (aa >= hv) break;
                    float *d = dst + (size_t)aa * a.W * a.Cout;
                    typedef float vec_t __attribute__((ext_vector_type(V)));
                    vec_t out;
#pragma unroll
                    for (int v = 0; v < V; ++v) out[v] = Yv[v][aa] + bias[v];
                    if constexpr (decltype(plain)::value) *reinterpret_cast<vec_t *>(d) = out;
                    else store_y(out, reinterpret_cast<vec_t *>(d));
                }
            }
        }
    };
    // four channels per thread where every pixel's channels start at a multiple of 16 bytes, otherwise one:
    // scalar stores of a lane's four channels would be scattered
    const bool vec4 = (a.Cout & 3) == 0;
    constexpr int P = M / BP;
    // One copy of this stage's code for all passes.  With a copy each the kernels had 29 to 35 KB in place of 13 to 21,
    // which a program of several layers fetches into the instruction cache (64 KB for two CUs) on every call: a
    // step of the ResNet-18 layers, F(6,3), batch 32, 111.2 -> 106.8 us, the kernel of its 56x56 layer 19.7 -> 15.2 there
    // and 15.1 either way when that layer repeats.
#pragma unroll 1
    for (int pass = 0; pass < NT * P; ++pass) {
        __syncthreads();   // the scales, or the tiles before, have been read
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (pass == nt * P + p) {
#pragma unroll
                    for (int bp = 0; bp < BP; ++bp)
#pragma unroll
                        for (int no = 0; no < NO; ++no)
                            *reinterpret_cast<float4 *>(&Rs[(w * BP + bp) * RSW + l16 * RS + 16 * no + 4 * q]) = R[p * BP + bp][no][nt];
                }
        __syncthreads();
        constexpr std::integral_constant<int, 1> one;
        if constexpr (NO == 2) {
            constexpr std::integral_constant<int, 4> many;
            if (!vec4) finish(one, std::false_type{}, pass / P, pass % P);
            else if (kPlainY<M, NT, NO> && a.plain_y) finish(many, std::true_type{}, pass / P, pass % P);   // (a branch at the store would be merged)
            else finish(many, std::false_type{}, pass / P, pass % P);
        } else {
            finish(one, std::false_type{}, pass / P, pass % P);
        }
    }
}

template <int M, bool K64, bool CPG1, bool WIDE, bool ATSP, int NT, int NO, int KS, int D, bool ONE>
hipError_t launch_one(const Args &a, hipStream_t s) {
    // the debug entry point runs the same template with the stores of the int32 sums compiled in
    Args b = a;
    b.blocks = wq_fused_launch_blocks(a.T_pad, a.Cout_pad, a.Cin, M + 2, NT, NO);
    const unsigned grid = wq_fused_grid(b.blocks);
    if (a.dump.P)
        hipLaunchKernelGGL((k_contract_output<M, K64, CPG1, WIDE, ATSP, true, NT, NO, KS, D, ONE>), dim3(grid),
                           dim3(64 * (M + 2) * KS), 0, s, b);
    else
        hipLaunchKernelGGL((k_contract_output<M, K64, CPG1, WIDE, ATSP, false, NT, NO, KS, D, ONE>), dim3(grid),
                           dim3(64 * (M + 2) * KS), 0, s, b);
    return hipGetLastError();
}

template <int M, bool K64, bool CPG1, bool WIDE, bool ATSP, int NT, int NO, int KS, int D>
hipError_t launch_cfg(const Args &a, hipStream_t s) {
    // The exchange of all columns at once is a pass less, of half of them half the LDS, which lets more
    // workgroups of F(6,3) onto a CU (F(4,3)'s fit as they are): where there are any more than two.
    if constexpr (M == 6 && NT * NO == 1 && KS == 1 && CPG1) {
        if ((long)(a.T_pad / 16) * (a.Cout_pad / 16) <= 512 || (a.Cin >> a.log2g) <= 2) return launch_one<M, K64, CPG1, WIDE, ATSP, NT, NO, KS, D, true>(a, s);
    }
    constexpr bool one = NO == 1 && M != 6;
    return launch_one<M, K64, CPG1, WIDE, ATSP, NT, NO, KS, D, one>(a, s);
}

// fp64 chunk totals only where a wave reduces more than the plan's fp32_groups per tap
template <int M, bool K64, bool CPG1, bool ATSP>
hipError_t launch_base(const Args &a, hipStream_t s, bool wide) {
    return wide ? launch_cfg<M, K64, CPG1, true, ATSP, 1, 1, 1, kDepth<M, 1, 1>>(a, s)
                : launch_cfg<M, K64, CPG1, false, ATSP, 1, 1, 1, kDepth<M, 1, 1>>(a, s);
}

// the register-tile variants: one K-step per group, paired form of A^T
template <int M, bool K64>
hipError_t launch_fast(const Args &a, hipStream_t s, int variant, bool wide) {
    if (variant == WQ_K2_FUSED_KSPLIT)
        return wide ? launch_cfg<M, K64, true, true, true, 1, 1, 2, kDepth<M, 1, 1>>(a, s)
                    : launch_cfg<M, K64, true, false, true, 1, 1, 2, kDepth<M, 1, 1>>(a, s);
    if (variant == WQ_K2_FUSED_32x16)
        return wide ? launch_cfg<M, K64, true, true, true, 2, 1, 1, kDepth<M, 2, 1, K64>>(a, s)
                    : launch_cfg<M, K64, true, false, true, 2, 1, 1, kDepth<M, 2, 1, K64>>(a, s);
    return wide ? launch_cfg<M, K64, true, true, true, 2, 2, 1, kDepth<M, 2, 2>>(a, s)
                : launch_cfg<M, K64, true, false, true, 2, 2, 1, kDepth<M, 2, 2>>(a, s);
}

template <int M>
hipError_t launch_m(const wq_plan *p, hipStream_t s, const int8_t *Xq, const float *sX,
                    const int8_t *Wq, const float *sW, const float *bias, float *y,
                    const wq_dump &dump) {
    Args a;
    a.xf = p->xf;
    a.Xq = Xq; a.sX = sX; a.Wq = Wq; a.sW = sW; a.bias = bias; a.y = y; a.dump = dump;
    a.H = p->H; a.W = p->W; a.Cin = p->Cin; a.Cout = p->Cout; a.TH = p->TH; a.TW = p->TW;
    a.T = p->T; a.T_pad = p->T_pad; a.Cout_pad = p->Cout_pad;
    a.log2g = 0;
    while ((1 << a.log2g) < p->g) ++a.log2g;
    a.blocks = {};
    {   // see finish
        const long long bytes = (long long)p->N * p->H * p->W * p->Cout * 4;
        a.plain_y = M == 4 && p->k2_variant == WQ_K2_FUSED_32x32 && bytes >= (32LL << 20) && bytes <= (56LL << 20);
    }
    const bool k64 = p->kstep == 64, cpg1 = p->g == p->kstep;
    const int variant = p->k2_variant;   // a fused one, checked for this plan when it was chosen
    const bool wide = p->groups / (variant == WQ_K2_FUSED_KSPLIT ? 2 : 1) > p->fp32_groups;
    a.dense_rows = p->dense_rows;
    if constexpr (M != 2) {
        if (variant != WQ_K2_FUSED_16x16)
            return k64 ? launch_fast<M, true>(a, s, variant, wide) : launch_fast<M, false>(a, s, variant, wide);
    }
    if (!k64)
        return p->sparse_at ? launch_base<M, false, true, true>(a, s, wide)
                            : launch_base<M, false, true, false>(a, s, wide);
    if (cpg1)
        return p->sparse_at ? launch_base<M, true, true, true>(a, s, wide)
                            : launch_base<M, true, true, false>(a, s, wide);
    return p->sparse_at ? launch_base<M, true, false, true>(a, s, wide)
                        : launch_base<M, true, false, false>(a, s, wide);
}

}  // namespace
