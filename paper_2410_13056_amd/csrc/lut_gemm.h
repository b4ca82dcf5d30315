// The product of several tokens with deployed layers (lut_gemm.hip), as lut_matvec.hip calls it.
#pragma once
#include "common.h"
#include <type_traits>

// Whether a layer's product with m tokens runs here (otherwise token by token in lut_matvec.hip).
// Depends on nothing but these sizes, so that a layer gives the same bits in any group.
bool lut_gemm_takes(int64_t d_in, int64_t d_out, int64_t m);

// Scratch for a layer's product with m tokens on the matrix cores: what is enough for any layer of
// these sizes, and what this layer's plan takes.
size_t lut_gemm_ws_bytes(int64_t d_in, int64_t d_out, int64_t m);
size_t lut_gemm_need(const cmpq_deployed_layer &layer, int64_t m);

// Enqueues the products of `layers` (checked by the caller, d_out > 0, m > 0).  `ws` holds the
// sum of lut_gemm_need over the layers.
int launch_lut_gemm(const cmpq_deployed_layer *const *layers, int n_layers, int64_t m, void *ws, hipStream_t s);

// How that cuts a layer up: see cmpq_lut_matvec_shape.
void lut_gemm_shape(const cmpq_deployed_layer &layer, int64_t m, int64_t *shape, int64_t *parts, int64_t room);

// Where share `i` of `n` things in `parts` even shares begins: floor(n * i / parts).  The product passes 32 bits from
// 741 441 rows of width 4 on, and a division in 64 bits is 100 instructions, in fp64 a tenth of that.  Exact: n and
// parts stay below 2^22 (limit of 65535 slabs of 128 rows), so the product does below 2^44, and a quotient below
// 2^22 that is no whole number lies further than 2^-22 from the next, its rounding less than 2^-30.
__host__ __device__ __forceinline__ int share_of(int n, int i, int parts) {
    return (int)((double)n * (double)i / (double)parts);
}

// What both kinds of product use of LDS tables.

// base + byte q of t in one instruction (written out: the compiler takes the byte out first).
template <int Q>
__device__ __forceinline__ uint32_t add_byte(uint32_t base, uint32_t t) {
    uint32_t r;
    if constexpr (Q == 0) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(base), "v"(t));
    else if constexpr (Q == 1) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(base), "v"(t));
    else if constexpr (Q == 2) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(base), "v"(t));
    else asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(base), "v"(t));
    return r;
}

__device__ __forceinline__ uint32_t add_byte(uint32_t base, uint32_t t, int q) {  // q known at compile time
    return q == 0 ? add_byte<0>(base, t) : (q == 1 ? add_byte<1>(base, t) : (q == 2 ? add_byte<2>(base, t) : add_byte<3>(base, t)));
}

template <typename T>
__device__ __forceinline__ T lds_read(uint32_t at) {
    typedef const T __attribute__((address_space(3))) *P;
    return *(P)(uintptr_t)at;
}

// Outputs o .. o + 7 of a row of O_act, from any even address.  In the last tile of a row the last eight are read
// instead where not all are there, and shifted into place; what is not there is not written.  One load, no branch
// between lanes: with a branch for every output the last tile (or, where rows are not 16 bytes apart, every one of
// the product with one token) waited for its loads one after the other.  Kernel times, us: 7872 -> 476, 24 tokens
// 19.1, now 13.4; 2048 -> 2006, 5 tokens 14.1 and 9.5; 832 -> 5118, one token 15.8 and 8.4.
// MODE, the same in all lanes: all lanes have all of their outputs; some do not; rows of fewer than eight.
enum { kActFull, kActShifted, kActFew };
template <int MODE>
__device__ __forceinline__ uint4 act_outputs8(const __half *row, int o, int d_out) {
    const char *p = reinterpret_cast<const char *>(row);
    if constexpr (MODE == kActFew) {
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = reinterpret_cast<const uint16_t *>(p)[min(e, d_out - 1)];
        return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    }
    typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(2)));
    const Words4 v = *reinterpret_cast<const Words4 *>(p + (uint32_t)(MODE == kActFull ? o : min(o, d_out - 8)) * 2u);
    if constexpr (MODE == kActFull) return make_uint4(v[0], v[1], v[2], v[3]);
    const int s = max(o + 8 - d_out, 0);  // that many of the eight are not there (8 and more: none is)
    const uint32_t a0 = s & 4 ? v[2] : v[0], a1 = s & 4 ? v[3] : v[1];
    const uint32_t b0 = s & 2 ? a1 : a0, b1 = s & 2 ? v[2] : a1, b2 = s & 2 ? v[3] : v[2];
    const uint32_t bits = (s & 1) * 16;
    return make_uint4(__builtin_amdgcn_alignbit(b1, b0, bits), __builtin_amdgcn_alignbit(b2, b1, bits),
                      __builtin_amdgcn_alignbit(v[3], b2, bits), v[3] >> bits);
}
template <typename F>
__device__ __forceinline__ void with_act_mode(int d_out, bool full, F &&f) {
    if (full) f(std::integral_constant<int, kActFull>());
    else if (d_out >= 8) f(std::integral_constant<int, kActShifted>());
    else f(std::integral_constant<int, kActFew>());
}

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
