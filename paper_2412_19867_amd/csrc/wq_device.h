// Device-side helpers shared by the kernels: vector types, buffer-resource constants, the
// cross-lane maximum and the quantizer's code (Section "Quantization": symmetric int8,
// round-half-to-even, one reciprocal per group).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kBufFlags = 0x00020000;   // raw buffer, 32-bit elements (gfx9 family)
// cache policy sc0 sc1 of a store: the data is written through to memory while the kernel runs
// instead of being flushed from the XCD's L2 when it ends
constexpr int kWriteThrough = 17;
// a buffer offset past the end of any buffer (all are below 2 GiB): such a load returns 0
constexpr unsigned kPastEnd = 1u << 31;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
    // bound_ctrl with a zero fill lets the compiler fold the move into v_max_u32_dpp
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true));
}

// rint(v*r) as the low byte of a two's-complement code; |v*r| <= 127 + ulp.
__device__ __forceinline__ uint32_t quant_code(float v, float r) {
    const float p = v * r;                   // one rounded product (contraction is off)
    const float z = p + 12582912.0f;         // 1.5*2^23: the add rounds p to nearest-even integer
    return __float_as_uint(z) & 0xffu;
}

// The integer transforms' code clamp(rint(v), -127, 127); a NaN becomes -127.  Clamping first gives
// the same code, and adding 1.5 * 2^52 rounds half to even and leaves the integer in the low word:
// one fp64 addition in place of a rounding and a conversion.
__device__ __forceinline__ int quant_code_f64(double v) {
    return (int)__double_as_longlong(__builtin_fmin(127.0, __builtin_fmax(-127.0, v)) + 6755399441055744.0);
}

// m * v + c for a wave-uniform matrix entry m, |m|, |v| < 2^23 and a result below 2^31: one
// instruction at the full rate, where a 32-bit product runs at a quarter of it and needs an addition.
// (Written out: of __mul24 the compiler turned a third back into 32-bit products.)  With it and the
// code above 2x64x64 640->640 F(4,3) with integer transforms went from 65.3 to 62.3 us.
__device__ __forceinline__ int mad24(int m, int v, int c) {
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "s"(m), "v"(v), "v"(c));
    return r;
}

// Store of an output value: streaming (non-temporal), the layer does not read y again.  (Plain
// stores make the next layer's input kernel faster when it follows at once, and this layer's
// output stage slower: a gain only where y is large and still fits the caches, where the fused kernel's
// four-block form takes them.)
template <typename T>
__device__ __forceinline__ void store_y(T v, T *p) {
    __builtin_nontemporal_store(v, p);
}

// An MFMA whose accumulator starts at kMagic = the bits of 1.5 * 2^23 leaves the bits of
// 1.5 * 2^23 + sum while |sum| < 2^22 (any group of up to 256 int8 products): the float of the sum
// is then one exact subtraction (2.4 cycles of a SIMD with two waves) instead of a conversion (4.3).
constexpr int kMagic = 0x4B400000;
// The same for sums that are multiples of 16 (4-bit weight codes, unpacked as 16 * code): from the bits
// of 1.5 * 2^19, whose last place is 2^-4, the result is 1.5 * 2^19 + sum / 16.
constexpr int kMagic16 = 0x49400000;

// the float of a group's int32 sum (with MAGIC and SIXTEENTH: of a sixteenth of it)
template <bool MAGIC, bool SIXTEENTH = false>
__device__ __forceinline__ float group_sum(int v) {
    if constexpr (MAGIC) return __int_as_float(v) - (SIXTEENTH ? 786432.0f : 12582912.0f);
    return (float)v;
}

// Broadcast of 16-lane rows: lane l of `v` holds the value of pixel l of the wave's 64 (16) pixels;
// r[f] gets pixel 16 f + l % 16 in every lane.
template <int NB>
__device__ __forceinline__ void spread_rows(float v, float (&r)[NB]) {
    static_assert(NB == 1 || NB == 2 || NB == 4, "row blocks per wave");
    if constexpr (NB == 1) {
        r[0] = v;
    } else {
        const unsigned u = __float_as_uint(v);
        const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // rows 0 0 2 2 | 1 1 3 3
        if constexpr (NB == 2) {   // (the lane rows carry 0 1 0 1)
            r[0] = __uint_as_float(s[0]);
            r[1] = __uint_as_float(s[1]);
            return;
        }
        const auto e = __builtin_amdgcn_permlane32_swap(s[0], s[0], false, false);
        const auto o = __builtin_amdgcn_permlane32_swap(s[1], s[1], false, false);
        r[0] = __uint_as_float(e[0]);
        r[1] = __uint_as_float(o[0]);
        r[2] = __uint_as_float(e[1]);
        r[3] = __uint_as_float(o[1]);
    }
}

template <int R>
__device__ __forceinline__ float quad_bcast(float v) {   // lane 4k + R of every quad to its four lanes
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), R * 0x55, 0xf, 0xf, true));
}

#define WQ_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// Buffer loads whose destination is LDS: lane l's 16 bytes land at lds + 16 l; `lds` and
// `soff` are wave-uniform.  Completion is counted by the wave's vector-memory counter.  (Plain
// device functions on purpose: called from a lambda inside the kernel template, the builtin makes
// the host pass drop the kernel's launch stub without a diagnostic.)
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, char *lds, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, WQ_LDS_PTR(lds), 16, voff, soff, 0, 0);
}

// s_waitcnt until at most VM of the wave's vector-memory operations are outstanding (they complete in
// order); the "memory" clobber keeps LDS accesses behind it.  (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// the other counters left alone.)
template <int VM>
__device__ __forceinline__ void wait_loads() {
    static_assert(VM >= 0 && VM < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt %0" ::"n"(0x0f70 | (VM & 0xf) | ((VM >> 4) << 14)) : "memory");
}
