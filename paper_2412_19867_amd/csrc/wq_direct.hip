// Group-wise int8 quantized STANDARD 3x3 convolution (stride 1, zero pad 1): the layer the
// paper's runtime section compares the quantized Winograd convolution against.  Same
// quantizer, same groups along the input channels, no transforms:
//   activations  one dynamic scale per (pixel, group)            k_quantize_pixels
//   weights      one scale per (filter tap, out-channel, group)  the offline weight kernel run
//                                                                 as F(1,3) with G = I
//   y[p][o] = bias[o] + sum over the 9 taps and the groups of
//             float(int32 dot product) * sx[shifted pixel][group] * sw[tap][group][o]
//                                                                 k_direct_conv
// k_direct_conv is an implicit GEMM without LDS staging: both operands lie in memory in the order
// the MFMA reads them, a wave loads them straight into its registers (see the kernel).
#include <float.h>

#include <cstdlib>
#include <cstring>
#include <new>

#include "wq_device.h"
#include "wq_direct_walk.h"
#include "wq_internal.h"

struct wq_direct_plan {
    wq_plan w;   // the offline weight stage as F(1,3): m = 1, n = 3, G = identity
    int N, H, W, Cin, Cout, g, groups, P, Cout_pad, kstep;
    int taps;     // 9 = 3x3 convolution, 1 = linear layer (every row is its own "image")
    int wbits;    // width of the weight codes: 8, or 4 (W4A8: two codes per byte)
    wq_direct_tile tile;   // the kernel instance and its launch shape
    int splits;   // the number of slices wq_direct_plan_tune asked for, 0 = the plan's own choice
    wq_direct_layout_t lay;
    std::atomic<int> prepared;
};

namespace {

// ------------------------------------------------------------ activations
// xq is stored as [Cin/kstep][4][P][kstep/4]: planes of one K-quarter of one MFMA K-step, pixels
// in order inside a plane.  The wave that multiplies 16 consecutive pixels then reads four runs of
// 16 pieces, and a filter tap shifts all of them by the same number of bytes.  (From a pixel-major
// tensor the same load takes 64 cycles of the address unit instead of 16: neighbouring lanes hold
// different pixels.)  Scales are [groups][P], so that neighbouring pixels' scales are neighbours too.
// 8 lanes per (pixel, group); a lane owns CPL = g/8 consecutive channels.  A workgroup holds 16
// pixels x 2 groups: its code stores fill whole 128-byte lines.
template <int CPL>
__global__ __launch_bounds__(256) void k_quantize_pixels(const float *__restrict__ x,
                                                         int8_t *__restrict__ xq,
                                                         float *__restrict__ sx, int P, int Cin,
                                                         int groups, int gpairs) {
    const int tid = threadIdx.x, l8 = tid & 7, unit = tid >> 3;
    const int pb = blockIdx.x / gpairs, gi = (blockIdx.x % gpairs) * 2 + (unit >> 4);
    const int row = unit & 15, p = pb * 16 + row;
    if (p >= P || gi >= groups) return;   // the 8 lanes of a unit leave together
    const int c0 = gi * (CPL * 8) + l8 * CPL;
    const float *src = x + (size_t)p * Cin + c0;
    float v[CPL];
#pragma unroll
    for (int k = 0; k < CPL / 4; ++k) {
        const float4 t = *reinterpret_cast<const float4 *>(src + 4 * k);
        v[4 * k] = t.x; v[4 * k + 1] = t.y; v[4 * k + 2] = t.z; v[4 * k + 3] = t.w;
    }
    uint32_t a = 0;
#pragma unroll
    for (int k = 0; k < CPL; ++k) a = max(a, __float_as_uint(v[k]) & 0x7fffffffu);
    a = dpp_max<0xB1>(a);    // quad_perm [1,0,3,2]
    a = dpp_max<0x4E>(a);    // quad_perm [2,3,0,1]
    a = dpp_max<0x141>(a);   // row_half_mirror: the 8 lanes of the unit
    const float af = __uint_as_float(a);
    float s = 0.0f, r = 0.0f;
    if (af >= 127.0f * FLT_MIN) {
        s = af / 127.0f;   // correctly rounded
        r = 127.0f / af;
    }
    uint32_t words[CPL / 4];
#pragma unroll
    for (int k = 0; k < CPL / 4; ++k)
        words[k] = quant_code(v[4 * k], r) | (quant_code(v[4 * k + 1], r) << 8) |
                   (quant_code(v[4 * k + 2], r) << 16) | (quant_code(v[4 * k + 3], r) << 24);
    if constexpr (CPL == 4) {   // K-step 32: the lane's 4 codes are half of a K-quarter of 8
        *reinterpret_cast<uint32_t *>(xq + ((size_t)(gi * 4 + (l8 >> 1)) * P + p) * 8 + (l8 & 1) * 4) = words[0];
    } else if constexpr (CPL == 8) {   // K-step 64: half of a K-quarter of 16
        *reinterpret_cast<uint2 *>(xq + ((size_t)(gi * 4 + (l8 >> 1)) * P + p) * 16 + (l8 & 1) * 8) =
            make_uint2(words[0], words[1]);
    } else {
#pragma unroll
        for (int k = 0; k < CPL / 16; ++k)
            *reinterpret_cast<uint4 *>(xq + ((size_t)((c0 >> 4) + k) * P + p) * 16) =
                make_uint4(words[4 * k], words[4 * k + 1], words[4 * k + 2], words[4 * k + 3]);
    }
    if (l8 == 0) sx[(size_t)gi * P + p] = s;
}

// ------------------------------------------------------------ convolution
struct DArgs {
    const int8_t *xq;
    const float *sx;
    const int8_t *Wq;
    const float *sW;
    const float *bias;
    float *y;
    int H, W, Cin, Cout, Cout_pad, P, log2g;
    // how a workgroup's waves share its work: `slices` waves split the reduction of one wave tile,
    // wo x wt wave tiles lie side by side along channels x pixels (slices * wo * wt waves)
    int slices, wo, wt;
    int nOt, total, per_xcd;   // workgroup tiles along channels, workgroups, share of each XCD
};

// Pixel rows of a wave tile that go through LDS at a time: two blocks where eight (16) waves' rows fit 64 KB,
// so that more of the waves that share a reduction take part in the sums behind it.
template <int NO, int NB>
constexpr int kRowsPerPass = (NB > 1 && NO <= 2) ? 32 : 16;

// A wave owns a (16 NO channels) x (16 NB pixels) tile and one slice of its reduction (whole
// groups of the flat sequence tap-major, then channels).  Operands go from memory straight into
// the registers the MFMA reads (both tensors are in its operand order) and are requested D
// K-steps ahead; there is no LDS and no barrier before the slices are added up at the end, so a
// wave waits for nothing but its own loads.
//   bound: 12 vector-ALU instructions and one MFMA per 16x16 block and group (46 cycles of a
//   SIMD, the two do not overlap), against 64 bytes per cycle and CU into registers: with NO x NB
//   = 2 x 4 blocks a block costs 768 bytes = 12 cycles of the CU's load path for 11.5 of its
//   four SIMDs.
//   scales: one word per lane and load (the 64 pixels' scales in one load, spread over the lanes by
//   row swaps; the channel scales of a quarter by DPP quad broadcasts): 256 bytes per load where a
//   16-byte load per lane would move 1 KiB for the same 16 values, on the busier of the two paths.
//   With one K-step per group the MFMA starts from kMagic instead of 0, which makes its int32
//   result the bit pattern of 1.5 * 2^23 + sum: a subtraction (2.4 cycles) then replaces the
//   conversion (4.3).  Exact while |sum| < 2^22: 64 * 127 * 127 and, for 4-bit weights, 64 * 16 * 7 * 127.
// W4: the weight codes are 4 bits wide, two per byte (see the weight kernels for the packing of a
// 16-byte piece into 8).  A lane loads the packed half of its piece and unpacks it as 16 * code
// (a nibble moved to the top of its byte), so the MFMA loop is the 8-bit one; 16 * |sum| stays below
// 2^24 for every group size, and the factor leaves before the running sum, so that outputs reach as far as
// the 8-bit path's: with one K-step per group by the subtraction that makes the sum a float, otherwise with
// the channel scales (one product per 16 channels and group, where on the sums it is four per block:
// 14x33x33 640->584 g 128 131 us, 137 on the sums; exact for scales of 2^-122 and more).
template <bool K64, bool CPG1, bool W4, bool T9, int NO, int NB, int D, int NWMAX>
__global__ __launch_bounds__(64 * NWMAX, 2) void k_direct_conv(const DArgs a) {
    constexpr int KSTEP = K64 ? 64 : 32, KB = KSTEP / 4;
    using Walk = wq_direct_walk<KSTEP, W4, T9>;
    constexpr int RS = 16 * NO + 4;                        // floats per pixel row of the LDS staging
    extern __shared__ __attribute__((aligned(16))) float part_s[];   // [waves][kRowsPerPass][RS]
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = w % a.slices, wtile = w / a.slices, wo = wtile % a.wo, wt = wtile / a.wo;
    // workgroup ids go round-robin over the XCDs: each takes a contiguous share of the tile order
    // (channel tiles fastest), whose pixels its L2 then holds
    const int logical = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (logical >= a.total) return;   // the whole workgroup leaves, before any barrier
    const int ob0 = ((logical % a.nOt) * a.wo + wo) * NO, p0 = ((logical / a.nOt) * a.wt + wt) * 16 * NB;
    const int Cin = a.Cin, P = a.P, groups = Cin >> a.log2g, back = Walk::back(a.W);

    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t *>(a.Wq), 0, (int)Walk::bytes_w(a.Cout_pad, Cin), kBufFlags);
    const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t *>(a.xq) - back * KB, 0, (int)Walk::bytes_x(P, a.W, Cin), kBufFlags);
    const __amdgpu_buffer_rsrc_t rSW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.sW), 0, (int)Walk::bytes_sw(a.Cout_pad, groups), kBufFlags);
    const __amdgpu_buffer_rsrc_t rSX = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.sx) - back, 0, (int)Walk::bytes_sx(P, a.W, groups), kBufFlags);

    // The lane's pixel of each row block, and the one whose scale it loads: a position that lies outside
    // the image, or past the last pixel, loads neither codes nor scale (its neighbour in memory is a
    // pixel of another row or image, whose scale may be infinite: 0 * Inf would reach this pixel's sum)
    // (one pixel's divisions per lane, its mask spread over the row blocks)
    const int ps = p0 + (lane & (16 * NB - 1));
    const unsigned vSX = ps < P ? Walk::lane_sx(ps) : kPastEnd, outS = Walk::outside((unsigned)ps, (unsigned)a.H, (unsigned)a.W);
    unsigned vX[NB];
    // (two row blocks' masks in one register: with one each the 32 x 64 tile of 4-bit weights takes 170
    // registers and a wave less fits a SIMD: 8x19x19 896->832 g 128 79 us, 69 so)
    unsigned out[(NB + 1) / 2] = {};
    if constexpr (T9) {
        float o[NB];
        spread_rows<NB>(__uint_as_float(outS), o);
#pragma unroll
        for (int f = 0; f < NB; ++f) out[f / 2] |= __float_as_uint(o[f]) << (f % 2 * 16);
    }
#pragma unroll
    for (int f = 0; f < NB; ++f) {
        const int p = p0 + 16 * f + l16;
        vX[f] = p < P ? Walk::lane_x(q, p, P) : kPastEnd;
    }

    // ---- the loader: its cursor walks (tap, K-step) of the wave's slice and stops at the end ----
    Walk at(P, a.W, Cin, a.Cout_pad, a.log2g, ks, a.slices);
    const int NI = at.steps, cpg = at.cpg;
    const unsigned vW = Walk::lane_w(lane), vSW = Walk::lane_sw(lane);
    unsigned oe[NO];
#pragma unroll
    for (int e = 0; e < NO; ++e) oe[e] = wq_direct_block(ob0, e, a.Cout_pad);
    v4i av[D][NO], bv[D][NB];
    float swv[D][NO], sxv[D];
    auto fetch = [&](int slot) {   // (slot is a constant after unrolling)
#pragma unroll
        for (int e = 0; e < NO; ++e) {
            const unsigned so = at.weights(oe[e]);
            if constexpr (K64 && !W4) {
                av[slot][e] = __builtin_amdgcn_raw_buffer_load_b128(rW, vW, so, 0);
            } else if constexpr (K64 || !W4) {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rW, vW, so, 0);
                av[slot][e] = v4i{t.x, t.y, 0, 0};
            } else {
                av[slot][e] = v4i{(int)__builtin_amdgcn_raw_buffer_load_b32(rW, vW, so, 0), 0, 0, 0};
            }
        }
#pragma unroll
        for (int f = 0; f < NB; ++f) {
            const unsigned vo = at.masked(vX[f], out[f / 2], f % 2);
            if constexpr (K64) {
                bv[slot][f] = __builtin_amdgcn_raw_buffer_load_b128(rX, vo, at.oX, 0);
            } else {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rX, vo, at.oX, 0);
                bv[slot][f] = v4i{t.x, t.y, 0, 0};
            }
        }
#pragma unroll
        for (int e = 0; e < NO; ++e)
            swv[slot][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rSW, vSW, at.weight_scales(oe[e]), 0));
        sxv[slot] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rSX, at.masked(vSX, outS), at.oSX, 0));
        at.advance();
    };
    auto unpack = [](const v4i &pk) {
        if constexpr (!W4) return pk;
        const unsigned a0 = (unsigned)pk.x, a1 = (unsigned)pk.y;
        if constexpr (K64)
            return v4i{(int)((a0 << 4) & 0xf0f0f0f0u), (int)(a0 & 0xf0f0f0f0u), (int)((a1 << 4) & 0xf0f0f0f0u),
                       (int)(a1 & 0xf0f0f0f0u)};
        return v4i{(int)((a0 << 4) & 0xf0f0f0f0u), (int)(a0 & 0xf0f0f0f0u), 0, 0};
    };

    // 16 x 16 tiles add the sums of every twelve groups up in a second set of registers: their slices may be
    // a quarter of the reduction, a longer chain of fp32 additions than the sum's precision allows
    constexpr bool TOTALS = NB == 1;
    static_assert(!TOTALS || D == 6, "twelve groups are two rounds of K-steps each");
    float4 Mc[NO][NB], Mt[NO][NB];
    v4i acc[NO][NB];
#pragma unroll
    for (int e = 0; e < NO; ++e)
#pragma unroll
        for (int f = 0; f < NB; ++f) {
            Mc[e][f] = Mt[e][f] = make_float4(0.f, 0.f, 0.f, 0.f);
            acc[e][f] = v4i{0, 0, 0, 0};
        }
#pragma unroll
    for (int d = 0; d < D; ++d) {   // in the order the loop expects them back
        fetch(d);
        __builtin_amdgcn_sched_barrier(0);
    }
    constexpr int start = W4 ? kMagic16 : kMagic;
    const v4i magic = {start, start, start, start};
    int k_c = 0;
    auto compute = [&](int u) {   // the K-step in slot u (a constant after unrolling)
        const bool done = CPG1 || ++k_c == cpg;   // the step completes a group: dequantize
        k_c = done ? 0 : k_c;
        float sx[NB];
        if (done) spread_rows<NB>(sxv[u], sx);
#pragma unroll
        for (int e = 0; e < NO; ++e) {
            const v4i aw = unpack(av[u][e]);
            v4i P4[NB];
#pragma unroll
            for (int f = 0; f < NB; ++f) {
                const v4i c0 = CPG1 ? magic : acc[e][f];
                if constexpr (K64) {
                    P4[f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aw, bv[u][f], c0, 0, 0, 0);
                } else {
                    const long x = __builtin_bit_cast(long, v2i{aw.x, aw.y});
                    const long y = __builtin_bit_cast(long, v2i{bv[u][f].x, bv[u][f].y});
                    P4[f] = __builtin_amdgcn_mfma_i32_16x16x32_i8(x, y, c0, 0, 0, 0);
                }
            }
            if (done) {
                const float sw = W4 && !CPG1 ? swv[u][e] * 0.0625f : swv[u][e];
                const float s0 = quad_bcast<0>(sw), s1 = quad_bcast<1>(sw), s2 = quad_bcast<2>(sw), s3 = quad_bcast<3>(sw);
#pragma unroll
                for (int f = 0; f < NB; ++f) {
                    Mc[e][f].x = __builtin_fmaf(group_sum<CPG1, W4>(P4[f][0]), s0 * sx[f], Mc[e][f].x);
                    Mc[e][f].y = __builtin_fmaf(group_sum<CPG1, W4>(P4[f][1]), s1 * sx[f], Mc[e][f].y);
                    Mc[e][f].z = __builtin_fmaf(group_sum<CPG1, W4>(P4[f][2]), s2 * sx[f], Mc[e][f].z);
                    Mc[e][f].w = __builtin_fmaf(group_sum<CPG1, W4>(P4[f][3]), s3 * sx[f], Mc[e][f].w);
                    P4[f] = v4i{0, 0, 0, 0};
                }
            }
            if constexpr (!CPG1) {
#pragma unroll
                for (int f = 0; f < NB; ++f) acc[e][f] = P4[f];
            }
        }
    };
    auto add_totals = [&]() {
#pragma unroll
        for (int e = 0; e < NO; ++e)
#pragma unroll
            for (int f = 0; f < NB; ++f) {
                Mt[e][f].x += Mc[e][f].x; Mt[e][f].y += Mc[e][f].y; Mt[e][f].z += Mc[e][f].z; Mt[e][f].w += Mc[e][f].w;
                Mc[e][f] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
    };
    // (whole rounds of the ring, then the rest: with the exit test inside the unrolled round the
    // compiler waits for ALL outstanding loads at the top of every round)
    int fold = 2 * cpg;
    for (int r = NI / D; r > 0; --r) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            compute(u);
            // (nothing moves across: with the steps' instructions mixed the registers do not suffice)
            __builtin_amdgcn_sched_barrier(0);
            fetch(u);   // D steps ahead (past the end: the last one again, never used)
            __builtin_amdgcn_sched_barrier(0);
        }
        if (TOTALS && --fold == 0) {
            fold = 2 * cpg;
            add_totals();
        }
    }
    const int rest = NI % D;
#pragma unroll
    for (int u = 0; u < D - 1; ++u)
        if (u < rest) compute(u);
    if constexpr (TOTALS) add_totals();

    // ---- sum of the slices through LDS, FB row blocks of pixels at a time, + bias; whole rows of 16 NO
    // channels stored ----
    // More than two slices are added in fp64, which costs a conversion per term: fp32 additions of sums
    // as large as the result would add as much error as the chain of groups they replace (with G groups
    // in c chains the squared error goes with G / (2 c) + c / 2).  The four slices of the 64-wide tiles
    // add in fp32: they come in place of as many, or of longer chains.  Relative error before and after:
    // 2x32x32 1280->320 g 32 1.76e-7, 1.26e-7 (28.4, 27.9 us on 2x32x32 640->640); 64x5120->2048 g 32
    // 1.25e-7, 8.4e-8 (12.1, 12.5 us).
    const bool wide = a.slices > 2 && (NO <= 2 || (!T9 && groups < 10));
    constexpr int FB = kRowsPerPass<NO, NB> / 16, ROWS = 16 * FB;
    float *mine = part_s + w * (ROWS * RS);
    constexpr int CQ = 4 * NO, RPP = 64 / CQ;   // 4 channels per lane, RPP pixel rows per wave and pass
    const float *tile = part_s + wtile * a.slices * (ROWS * RS) + (lane / CQ) * RS + (lane % CQ) * 4;
    const int o = ob0 * 16 + (lane % CQ) * 4;
    float bv4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) bv4[r] = o + r < a.Cout ? a.bias[o + r] : 0.f;
#pragma unroll
    for (int f = 0; f < NB; f += FB) {
        if (f) __syncthreads();   // the rows of the blocks before have been read
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int e = 0; e < NO; ++e)
                *reinterpret_cast<float4 *>(&mine[(16 * fb + l16) * RS + 16 * e + 4 * q]) = TOTALS ? Mt[e][f + fb] : Mc[e][f + fb];
        __syncthreads();
        for (int r0 = ks * RPP; r0 < ROWS; r0 += a.slices * RPP) {   // the slices' waves share the rows
            const int p = p0 + 16 * f + r0 + lane / CQ;
            if (p >= P || o >= a.Cout) continue;
            const float4 t0 = *reinterpret_cast<const float4 *>(&tile[r0 * RS]);
            float sum[4];
            if (wide) {
                double s[4] = {(double)t0.x + bv4[0], (double)t0.y + bv4[1], (double)t0.z + bv4[2], (double)t0.w + bv4[3]};
                for (int z = 1; z < a.slices; ++z) {
                    const float4 t = *reinterpret_cast<const float4 *>(&tile[(z * ROWS + r0) * RS]);
                    s[0] += (double)t.x; s[1] += (double)t.y; s[2] += (double)t.z; s[3] += (double)t.w;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) sum[r] = (float)s[r];
            } else {   // (the bias with the first slice, where the sums are smallest)
                float4 s = make_float4(t0.x + bv4[0], t0.y + bv4[1], t0.z + bv4[2], t0.w + bv4[3]);
                for (int z = 1; z < a.slices; ++z) {
                    const float4 t = *reinterpret_cast<const float4 *>(&tile[(z * ROWS + r0) * RS]);
                    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
                }
                sum[0] = s.x; sum[1] = s.y; sum[2] = s.z; sum[3] = s.w;
            }
            float *dst = a.y + (size_t)p * a.Cout + o;
            if ((a.Cout & 3) == 0) {   // o is a multiple of 4, so o + 3 < Cout and the address is 16-byte aligned
                __builtin_nontemporal_store(v4f{sum[0], sum[1], sum[2], sum[3]}, reinterpret_cast<v4f *>(dst));
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (o + r < a.Cout) dst[r] = sum[r];
            }
        }
    }
}

int ilog2(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

uint64_t align256(uint64_t v) { return (v + 255) / 256 * 256; }

void choose_tile(wq_direct_plan *p) {
    p->tile = wq_direct_choose_tile(p->P, p->Cout_pad, p->taps, p->groups, p->g, p->kstep, p->splits);
    p->lay.splits = p->splits ? p->splits : 1;
    p->lay.launch = (16 * p->tile.no) << 16 | (16 * p->tile.nb) << 8 | p->tile.slices;
}

template <bool K64, bool CPG1, bool W4, bool T9, int NO, int NB, int D, int NWMAX>
void launch_conv(const DArgs &a0, hipStream_t s) {
    DArgs a = a0;
    const long ob = a.Cout_pad / 16, pb = (a.P + 15) / 16;
    a.nOt = (int)((ob + NO * a.wo - 1) / (NO * a.wo));
    const long nPt = (pb + NB * a.wt - 1) / (NB * a.wt);
    a.total = (int)(a.nOt * nPt);
    a.per_xcd = (a.total + 7) / 8;
    const int waves = a.slices * a.wo * a.wt;
    hipLaunchKernelGGL((k_direct_conv<K64, CPG1, W4, T9, NO, NB, D, NWMAX>), dim3((unsigned)a.per_xcd * 8u),
                       dim3(64 * waves), (size_t)waves * (kRowsPerPass<NO, NB>) * (16 * NO + 4) * 4, s, a);
}

template <bool K64, bool CPG1, bool W4, bool T9>
void launch_conv_tile(const wq_direct_plan *p, const DArgs &a, hipStream_t s) {
    if (p->tile.no == 4) launch_conv<K64, CPG1, W4, T9, 4, 4, 2, 8>(a, s);
    else if (p->tile.no == 2) launch_conv<K64, CPG1, W4, T9, 2, 4, 3, 8>(a, s);
    else if (p->tile.nb == 4) launch_conv<K64, CPG1, W4, T9, 1, 4, 3, 16>(a, s);
    else launch_conv<K64, CPG1, W4, T9, 1, 1, 6, 16>(a, s);
}

template <bool K64, bool CPG1, bool W4>
void launch_conv_taps(const wq_direct_plan *p, const DArgs &a, hipStream_t s) {
    if (p->taps == 9) launch_conv_tile<K64, CPG1, W4, true>(p, a, s);
    else launch_conv_tile<K64, CPG1, W4, false>(p, a, s);
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

static wq_status_t make_plan(wq_direct_plan_t **out, int N, int H, int W, int Cin, int Cout,
                             int group_size, int taps, int weight_bits) {
    if (!out) return WQ_ERR_INVALID_ARG;
    *out = nullptr;
    if (weight_bits != 8 && weight_bits != 4) return WQ_ERR_UNSUPPORTED;
    if (N <= 0 || H <= 0 || W <= 0 || Cin <= 0 || Cout <= 0 || group_size <= 0) return WQ_ERR_INVALID_ARG;
    if (group_size != 32 && group_size != 64 && group_size != 128 && group_size != 256 && group_size != 512)
        return WQ_ERR_UNSUPPORTED;
    if (Cin % group_size != 0) return WQ_ERR_INVALID_ARG;
    const long long P = (long long)N * H * W, Cp = (Cout + 31) / 32 * 32, lim = (1LL << 31) - 1;
    if (P * Cin * 4 > lim || P * Cout * 4 > lim || taps * Cp * Cin > lim ||
        taps * Cp * (Cin / group_size) * 4 > lim)
        return WQ_ERR_UNSUPPORTED;
    if ((P + 63) / 64 > 65535) return WQ_ERR_UNSUPPORTED;   // the largest layer tested: offsets and launch would allow more
    wq_direct_plan *p = new (std::nothrow) wq_direct_plan();
    if (!p) return WQ_ERR_INVALID_ARG;
    p->N = N; p->H = H; p->W = W; p->Cin = Cin; p->Cout = Cout; p->g = group_size;
    p->groups = Cin / group_size; p->P = (int)P; p->Cout_pad = (int)Cp;
    p->kstep = group_size == 32 ? 32 : 64;
    p->taps = taps;
    p->wbits = weight_bits;
    // the weight stage: the offline Winograd weight kernel as F(1,3) with G = I leaves the nine
    // filter taps untransformed and quantizes them per (tap, out-channel, group)
    wq_plan &w = p->w;
    w.N = N; w.H = H; w.W = W; w.Cin = Cin; w.Cout = Cout; w.m = 1; w.n = 3; w.g = group_size;
    w.groups = p->groups; w.TH = H; w.TW = W; w.T = (int)P; w.T_pad = (int)((P + 31) / 32 * 32);
    w.Cout_pad = p->Cout_pad; w.kstep = p->kstep; w.wbits = weight_bits;
    w.k1_rows = 1; w.k2_variant = WQ_K2_FUSED_16x16;
    std::memset(&w.xf, 0, sizeof(w.xf));
    w.xf.G[0] = w.xf.G[4] = w.xf.G[8] = 1.0f;
    w.sparse_bt = w.sparse_g = w.sparse_at = false;
    w.prepared.store(0);
    wq_direct_layout_t &L = p->lay;
    L.N = N; L.H = H; L.W = W; L.Cin = Cin; L.Cout = Cout; L.group_size = group_size;
    L.groups = p->groups; L.P = p->P; L.Cout_pad = p->Cout_pad; L.kstep = p->kstep;
    L.taps = taps;
    L.weight_bits = weight_bits;
    L.blob_Wq_off = 0;
    L.blob_sW_off = align256(((uint64_t)taps * p->Cout_pad * Cin * weight_bits) / 8);
    L.blob_bias_off = L.blob_sW_off + align256((uint64_t)taps * p->groups * p->Cout_pad * 4);
    L.blob_bytes = L.blob_bias_off + align256((uint64_t)p->Cout_pad * 4);
    L.ws_xq_off = 0;
    L.ws_sx_off = align256((uint64_t)P * Cin);
    p->splits = 0;
    choose_tile(p);
    L.ws_part_off = L.ws_sx_off + align256((uint64_t)P * p->groups * 4);
    L.ws_bytes = L.ws_part_off;
    p->prepared.store(0);
    *out = p;
    return WQ_OK;
}

wq_status_t wq_direct_plan_create(wq_direct_plan_t **out, int N, int H, int W, int Cin, int Cout,
                                  int group_size) {
    return make_plan(out, N, H, W, Cin, Cout, group_size, 9, 8);
}

wq_status_t wq_direct_plan_create_bits(wq_direct_plan_t **out, int N, int H, int W, int Cin, int Cout,
                                       int group_size, int weight_bits) {
    return make_plan(out, N, H, W, Cin, Cout, group_size, 9, weight_bits);
}

wq_status_t wq_linear_plan_create(wq_direct_plan_t **out, int R, int Cin, int Cout, int group_size) {
    return make_plan(out, R, 1, 1, Cin, Cout, group_size, 1, 8);
}

wq_status_t wq_linear_plan_create_bits(wq_direct_plan_t **out, int R, int Cin, int Cout, int group_size,
                                       int weight_bits) {
    return make_plan(out, R, 1, 1, Cin, Cout, group_size, 1, weight_bits);
}

wq_status_t wq_direct_plan_tune(wq_direct_plan_t *plan, int splits) {
    if (!plan || splits < 0) return WQ_ERR_INVALID_ARG;
    if (splits == 0) return WQ_OK;
    const bool ok = plan->taps == 9 ? (splits == 1 || splits == 3 || splits == 9)
                                    : (splits <= 16 && (splits & (splits - 1)) == 0 &&
                                       plan->groups % splits == 0);
    if (!ok) return WQ_ERR_UNSUPPORTED;
    plan->splits = splits;
    choose_tile(plan);
    return WQ_OK;
}

wq_status_t wq_direct_plan_destroy(wq_direct_plan_t *plan) {
    if (!plan) return WQ_ERR_INVALID_ARG;
    delete plan;
    return WQ_OK;
}

wq_status_t wq_direct_plan_layout(const wq_direct_plan_t *plan, wq_direct_layout_t *out) {
    if (!plan || !out) return WQ_ERR_INVALID_ARG;
    *out = plan->lay;
    return WQ_OK;
}

wq_status_t wq_direct_weight_prepare(wq_direct_plan_t *plan, void *stream, const float *w_dev,
                                     const float *bias_dev, void *weight_blob_dev, size_t blob_bytes) {
    if (!plan || !w_dev || !weight_blob_dev) return WQ_ERR_INVALID_ARG;
    if (blob_bytes < plan->lay.blob_bytes) return WQ_ERR_WORKSPACE;
    char *b = (char *)weight_blob_dev;
    hipError_t e = (plan->taps == 1 ? wq_launch_weight_rows : wq_launch_weight)(
        &plan->w, (hipStream_t)stream, w_dev, bias_dev, (int8_t *)(b + plan->lay.blob_Wq_off),
        (float *)(b + plan->lay.blob_sW_off), (float *)(b + plan->lay.blob_bias_off));
    if (e != hipSuccess) return WQ_ERR_DEVICE;
    plan->prepared.store(1);
    return WQ_OK;
}

wq_status_t wq_direct_quantize(const wq_direct_plan_t *plan, void *stream, const float *x_dev,
                               void *workspace_dev, size_t workspace_bytes) {
    if (!plan || !x_dev || !workspace_dev) return WQ_ERR_INVALID_ARG;
    if (workspace_bytes < plan->lay.ws_bytes) return WQ_ERR_WORKSPACE;
    char *ws = (char *)workspace_dev;
    int8_t *xq = (int8_t *)(ws + plan->lay.ws_xq_off);
    float *sx = (float *)(ws + plan->lay.ws_sx_off);
    const int gpairs = (plan->groups + 1) / 2;
    const dim3 grid((unsigned)((plan->P + 15) / 16) * (unsigned)gpairs), block(256);
    hipStream_t s = (hipStream_t)stream;
    switch (plan->g) {
        case 32: hipLaunchKernelGGL((k_quantize_pixels<4>), grid, block, 0, s, x_dev, xq, sx, plan->P, plan->Cin, plan->groups, gpairs); break;
        case 64: hipLaunchKernelGGL((k_quantize_pixels<8>), grid, block, 0, s, x_dev, xq, sx, plan->P, plan->Cin, plan->groups, gpairs); break;
        case 128: hipLaunchKernelGGL((k_quantize_pixels<16>), grid, block, 0, s, x_dev, xq, sx, plan->P, plan->Cin, plan->groups, gpairs); break;
        case 256: hipLaunchKernelGGL((k_quantize_pixels<32>), grid, block, 0, s, x_dev, xq, sx, plan->P, plan->Cin, plan->groups, gpairs); break;
        default: hipLaunchKernelGGL((k_quantize_pixels<64>), grid, block, 0, s, x_dev, xq, sx, plan->P, plan->Cin, plan->groups, gpairs); break;
    }
    return hipGetLastError() == hipSuccess ? WQ_OK : WQ_ERR_DEVICE;
}

wq_status_t wq_direct_conv(const wq_direct_plan_t *plan, void *stream, void *workspace_dev,
                           size_t workspace_bytes, const void *weight_blob_dev, size_t blob_bytes,
                           float *y_dev) {
    if (!plan || !workspace_dev || !weight_blob_dev || !y_dev) return WQ_ERR_INVALID_ARG;
    if (workspace_bytes < plan->lay.ws_bytes || blob_bytes < plan->lay.blob_bytes) return WQ_ERR_WORKSPACE;
    if (!plan->prepared.load()) return WQ_ERR_NOT_PREPARED;
    const char *ws = (const char *)workspace_dev, *b = (const char *)weight_blob_dev;
    DArgs a;
    a.xq = (const int8_t *)(ws + plan->lay.ws_xq_off);
    a.sx = (const float *)(ws + plan->lay.ws_sx_off);
    a.Wq = (const int8_t *)(b + plan->lay.blob_Wq_off);
    a.sW = (const float *)(b + plan->lay.blob_sW_off);
    a.bias = (const float *)(b + plan->lay.blob_bias_off);
    a.y = y_dev;
    a.H = plan->H; a.W = plan->W; a.Cin = plan->Cin; a.Cout = plan->Cout;
    a.Cout_pad = plan->Cout_pad; a.P = plan->P; a.log2g = ilog2(plan->g);
    a.slices = plan->tile.slices; a.wo = plan->tile.wo; a.wt = plan->tile.wt;
    hipStream_t s = (hipStream_t)stream;
    const bool k32 = plan->kstep == 32, one = plan->g == 64;
    if (plan->wbits == 4) {
        if (k32) launch_conv_taps<false, true, true>(plan, a, s);
        else if (one) launch_conv_taps<true, true, true>(plan, a, s);
        else launch_conv_taps<true, false, true>(plan, a, s);
    } else {
        if (k32) launch_conv_taps<false, true, false>(plan, a, s);
        else if (one) launch_conv_taps<true, true, false>(plan, a, s);
        else launch_conv_taps<true, false, false>(plan, a, s);
    }
    return hipGetLastError() == hipSuccess ? WQ_OK : WQ_ERR_DEVICE;
}

wq_status_t wq_direct_forward(const wq_direct_plan_t *plan, void *stream, const float *x_dev,
                              const void *weight_blob_dev, size_t blob_bytes, void *workspace_dev,
                              size_t workspace_bytes, float *y_dev) {
    if (!plan || !x_dev || !y_dev || !weight_blob_dev || !workspace_dev) return WQ_ERR_INVALID_ARG;
    if (workspace_bytes < plan->lay.ws_bytes || blob_bytes < plan->lay.blob_bytes) return WQ_ERR_WORKSPACE;
    if (!plan->prepared.load()) return WQ_ERR_NOT_PREPARED;
    wq_status_t st = wq_direct_quantize(plan, stream, x_dev, workspace_dev, workspace_bytes);
    if (st != WQ_OK) return st;
    return wq_direct_conv(plan, stream, workspace_dev, workspace_bytes, weight_blob_dev, blob_bytes, y_dev);
}

}  // extern "C"
