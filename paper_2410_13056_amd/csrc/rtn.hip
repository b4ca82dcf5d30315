// cmpq_rtn_quantize: CMPQ with the uniform quantizer of Sec. 3 of arXiv 2410.13056 in place of
// K-means (App. A.2, Tab. 10): round-to-nearest on the grid min + k * Delta,
// Delta = (max - min) / (2^N - 1), per group of consecutive outputs of an input channel, with
// the channel's width N from Algorithm 1.
//
// One workgroup per channel; a lane takes 8 consecutive weights per step (FP16: one 16-byte load a step ahead; one
// 8-byte store), so a group of g weights is g / 8 neighbouring lanes and its range is found with exchanges
// between them - min and max do not depend on the order.  The code is the whole number nearest to the correctly
// rounded fp32 quotient (w - min) / Delta; the squared error is summed in fp64 per lane and reduced in a fixed
// order.
//
// Bound by instruction issue and HBM alike: 3 B a weight (FP16; 5120 x 13824 in 56 us = 3.8 TB/s, a plain copy
// here 4.8) and 25 vector instructions, 46 us of it.  It took 77 us with 36: a division in 64 bits for the
// group's number, the group's range exchanged through LDS float by float, the quotient carried to its last bit
// for every weight.
#include "common.h"

namespace {

constexpr int kT = 256;
constexpr int kPer = 8;  // weights per lane and step

// Eight consecutive weights of one channel at any alignment and end.
// Returns the mask of entries that exist (o0 + j < d_out).
template <typename TW>
__device__ __forceinline__ uint32_t load8w(const TW *__restrict__ wrow, int64_t o0, int64_t d_out, float (&w)[kPer]) {
    uint32_t valid = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        w[j] = 0.f;
        if (o0 + j < d_out) {
            valid |= 1u << j;
            w[j] = load_as_f32<TW>(wrow, o0 + j);
        }
    }
    return valid;
}

// The 8 weights of a lane as they lie in memory (16-byte aligned), and as floats.  FP32 takes two loads from a
// line, and a streamed first one lets the line go: groups of 8, 300 x 32768 29 us streamed, 19 plain; 100000 x 128 126
// and 102.
template <typename TW>
struct Piece {
    uint4 v[sizeof(TW) / 2];
    __device__ __forceinline__ void fetch(const TW *p, bool there) {
#pragma unroll
        for (int q = 0; q < (int)(sizeof(TW) / 2); ++q) {
            const TW *at = p + q * (16 / sizeof(TW));
            v[q] = make_uint4(0, 0, 0, 0);
            if (there) v[q] = sizeof(TW) == 2 ? load16_stream(at) : *reinterpret_cast<const uint4 *>(at);
        }
    }
    __device__ __forceinline__ void floats(float (&w)[kPer]) const {
        if constexpr (sizeof(TW) == 2) {
            const __half2 *h = reinterpret_cast<const __half2 *>(&v[0]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 t = __half22float2(h[j]);
                w[2 * j] = t.x;
                w[2 * j + 1] = t.y;
            }
        } else {
            __builtin_memcpy(w, v, sizeof(w));
        }
    }
};

// Packed FP16 minimum (the compiler's own form first quiets both operands).
__device__ __forceinline__ uint32_t pk_min_f16(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <int CTRL>
__device__ __forceinline__ uint32_t min_step(uint32_t x) {
    return pk_min_f16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true));
}
// FP16: range of the group from a lane's 8 weights, and whether one of these is not finite.  Smallest and
// negated largest travel as one pair: 2 instructions an exchange where single floats take 8.
__device__ __forceinline__ void range_of_halves(const uint4 &v, bool there, int lanes, float &lo, float &hi, bool &bad) {
    typedef unsigned short Bits2 __attribute__((ext_vector_type(2)));
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    Bits2 m = __builtin_bit_cast(Bits2, d[0] & 0x7fff7fffu);
#pragma unroll
    for (int q = 1; q < 4; ++q) m = __builtin_elementwise_max(m, __builtin_bit_cast(Bits2, d[q] & 0x7fff7fffu));
    bad |= (m.x > m.y ? m.x : m.y) >= 0x7c00;
    const uint32_t mn = pk_min_f16(pk_min_f16(d[0], d[1]), pk_min_f16(d[2], d[3]));
    const uint32_t s = 0x80008000u;
    const uint32_t mx = pk_min_f16(pk_min_f16(d[0] ^ s, d[1] ^ s), pk_min_f16(d[2] ^ s, d[3] ^ s));
    uint32_t x = pk_min_f16(__builtin_amdgcn_perm(mx, mn, 0x05040100u), __builtin_amdgcn_perm(mx, mn, 0x07060302u));
    if (!there) x = 0x7c007c00u;  // a lane past the end (its weights read as 0) brings nothing into its group
    if (lanes >= 2) x = min_step<0xB1>(x);    // quad_perm [1,0,3,2]
    if (lanes >= 4) x = min_step<0x4E>(x);    // quad_perm [2,3,0,1]
    if (lanes >= 8) x = min_step<0x141>(x);   // row_half_mirror
    if (lanes >= 16) x = min_step<0x140>(x);  // row_mirror
    if (lanes >= 32) {
        const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = pk_min_f16(a[0], a[1]);
    }
    if (lanes >= 64) {
        const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        x = pk_min_f16(a[0], a[1]);
    }
    lo = __half2float(__ushort_as_half((unsigned short)x));
    hi = -__half2float(__ushort_as_half((unsigned short)(x >> 16)));
}

// Smallest lo and largest hi over aligned groups of `lanes` lanes (a power of two, the same for all), in every
// lane of a group.  On the DPP path inside a row of 16 lanes, by row swaps across rows: as exchanges through
// LDS these were 8 trips of some 130 cycles one after the other for a group of 128 weights.
template <int CTRL>
__device__ __forceinline__ void range_step(float &lo, float &hi) {
    lo = fminf(lo, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(lo), CTRL, 0xF, 0xF, true)));
    hi = fmaxf(hi, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(hi), CTRL, 0xF, 0xF, true)));
}
__device__ __forceinline__ void range_of_group(float &lo, float &hi, int lanes) {
    if (lanes >= 2) range_step<0xB1>(lo, hi);    // quad_perm [1,0,3,2]
    if (lanes >= 4) range_step<0x4E>(lo, hi);    // quad_perm [2,3,0,1]
    if (lanes >= 8) range_step<0x141>(lo, hi);   // row_half_mirror
    if (lanes >= 16) range_step<0x140>(lo, hi);  // row_mirror
    if (lanes >= 32) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(lo), false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(hi), __float_as_uint(hi), false, false);
        lo = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        hi = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    }
    if (lanes >= 64) {
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(lo), false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(hi), __float_as_uint(hi), false, false);
        lo = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        hi = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    }
}

// lanes_per_group: a power of two in 1..64 (group / 8).  VEC: rows are read and written in
// whole 8-weight pieces (aligned, d_out a multiple of 8), so a lane's piece exists entirely
// or not at all and no entry needs a test of its own.
template <typename TW, bool WITH_ERR, bool VEC>
__global__ __launch_bounds__(kT) void rtn_kernel(const TW *__restrict__ W, int64_t d_out, int64_t ldw,
                                                  const uint8_t *__restrict__ bits, int lanes_per_group,
                                                  int64_t n_groups, uint8_t *__restrict__ codes,
                                                  float *__restrict__ scale, float *__restrict__ zero,
                                                  double *__restrict__ err_ch, int32_t *__restrict__ status) {
    __shared__ double red[kT / CMPQ_WAVE];
    const int64_t i = blockIdx.x;
    const int tid = threadIdx.x;
    const int N = bits[i];
    const bool kept = N < 1 || N > 4;  // a channel of O_act: stays FP16, no codes
    const float top = (float)((1 << (kept ? 1 : N)) - 1);
    const TW *wrow = W + i * ldw;
    uint8_t *crow = codes + i * d_out;
    const int group_shift = __ffs(lanes_per_group * kPer) - 1;  // (a division in 64 bits is 130 instructions)
    double s = 0.0;
    bool bad = false;
    Piece<TW> next;
    constexpr bool kAhead = sizeof(TW) == 2;  // (FP32 a step ahead: nothing gained, 8 registers more)
    if constexpr (VEC && kAhead) next.fetch(wrow + (int64_t)tid * kPer, (int64_t)tid * kPer < d_out);
    for (int64_t base = 0; base < d_out; base += (int64_t)kT * kPer) {
        const int64_t o0 = base + (int64_t)tid * kPer;
        float w[kPer];
        uint32_t valid;
        float lo = INFINITY, hi = -INFINITY;
        if constexpr (VEC) {  // FP16: the next step's weights are on their way while these are worked on
            if constexpr (!kAhead) next.fetch(wrow + o0, o0 < d_out);
            const Piece<TW> piece = next;
            valid = o0 < d_out ? 0xffu : 0u;
            if constexpr (kAhead) next.fetch(wrow + o0 + (int64_t)kT * kPer, o0 + (int64_t)kT * kPer < d_out);
            piece.floats(w);
            if constexpr (sizeof(TW) == 2) {
                bool odd = false;
                range_of_halves(piece.v[0], valid != 0, lanes_per_group, lo, hi, odd);
                bad |= odd;
            } else if (valid) {
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    lo = fminf(lo, w[j]);
                    hi = fmaxf(hi, w[j]);
                    bad |= !isfinite(w[j]);
                }
            }
        } else {
            valid = load8w<TW>(wrow, o0, d_out, w);
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if ((valid >> j) & 1u) {
                    lo = fminf(lo, w[j]);
                    hi = fmaxf(hi, w[j]);
                    bad |= !isfinite(w[j]);
                }
        }
        auto has = [&](int j) -> bool { return VEC ? valid != 0u : ((valid >> j) & 1u) != 0u; };
        // range of the group: every lane of the wavefront takes part, also those past the end
        if constexpr (!(VEC && sizeof(TW) == 2)) range_of_group(lo, hi, lanes_per_group);
        if (!valid) continue;
        float r[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) r[j] = 0.f;
        if (kept) {
            if (WITH_ERR) {
#pragma unroll
                for (int j = 0; j < kPer; ++j)
                    if (has(j)) {
                        const double d = (double)w[j] - (double)__half2float(__float2half_rn(w[j]));
                        s = fma(d, d, s);
                    }
            }
            lo = 0.f;
            hi = 0.f;
        }
        const float delta = (hi - lo) / top;
        if ((tid & (lanes_per_group - 1)) == 0) {
            const int64_t g = o0 >> group_shift;
            scale[i * n_groups + g] = delta;
            zero[i * n_groups + g] = lo;
        }
        if (!kept && delta != 0.f) {
            // The code is the whole number nearest to the correctly rounded quotient (w - lo) / delta.  A product
            // with the reciprocal is within 2^-17 of that quotient (16 * 2^-21): where none of the 8 comes
            // closer than 2^-16 to half way between two codes, it rounds to the same number.  Otherwise (one
            // wavefront step in 60), and for tiny or huge delta, the quotient itself.
            float farthest = 1.f;
            if (delta >= 0x1p-60f && delta <= 0x1p60f) {
                const float y0 = __builtin_amdgcn_rcpf(delta);
                const float y = fmaf(fmaf(-delta, y0, 1.f), y0, y0);
                farthest = 0.f;
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    const float q = (w[j] - lo) * y;
                    r[j] = rintf(q);
                    farthest = fmaxf(farthest, fabsf(q - r[j]));
                }
            }
            if (farthest > 0.5f - 0x1p-16f) {
#pragma unroll
                for (int j = 0; j < kPer; ++j) r[j] = fminf(fmaxf(rintf((w[j] - lo) / delta), 0.f), top);
            }
        }
        if (WITH_ERR && !kept) {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (has(j)) {
                    const double d = (double)w[j] - fma((double)r[j], (double)delta, (double)lo);
                    s = fma(d, d, s);
                }
        }
        // r holds whole numbers in 0..15: the conversion packs them as bytes
        uint2 out = make_uint2(0u, 0u);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            out.x = __builtin_amdgcn_cvt_pk_u8_f32(r[j], j, out.x);
            out.y = __builtin_amdgcn_cvt_pk_u8_f32(r[4 + j], j, out.y);
        }
        if (VEC) {
            *reinterpret_cast<uint2 *>(crow + o0) = out;
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if ((valid >> j) & 1u) crow[o0 + j] = (uint8_t)(((j < 4 ? out.x : out.y) >> (8 * (j & 3))) & 0xffu);
        }
    }
    if (status && __syncthreads_or(bad) && tid == 0) atomicOr(status, CMPQ_STATUS_NONFINITE);
    if (WITH_ERR) {
        s = wave_sum_f64(s);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int wv = 0; wv < kT / CMPQ_WAVE; ++wv) t += red[wv];
            err_ch[i] = t;
        }
    }
}

}  // namespace

extern "C" int cmpq_rtn_quantize(const void *W, int dtype, int64_t d_in, int64_t d_out, int64_t ldw,
                                 const uint8_t *bits, int64_t group, uint8_t *codes, float *scale,
                                 float *zero, double *err_ch, int32_t *status, void *stream) {
    if (d_in < 0 || d_out < 0 || (dtype != CMPQ_F16 && dtype != CMPQ_F32)) return CMPQ_EINVAL;
    if (group < 8 || group > 512 || (group & (group - 1)) != 0) return CMPQ_EINVAL;
    if (d_in == 0 || d_out == 0) return CMPQ_OK;
    if (!W || !bits || !codes || !scale || !zero) return CMPQ_EINVAL;
    if (ldw < d_out) return CMPQ_ESHAPE;
    if (d_in > 0x7fffffff) return CMPQ_ESHAPE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int esz = dtype == CMPQ_F16 ? 2 : 4;
    const int vec_ok = reinterpret_cast<uintptr_t>(W) % 16 == 0 && (ldw * esz) % 16 == 0 &&
                       reinterpret_cast<uintptr_t>(codes) % 8 == 0 && d_out % 8 == 0;
    const int lpg = (int)(group / kPer);
    const int64_t n_groups = cdiv(d_out, group);
    const unsigned grid = (unsigned)d_in;
#define CMPQ_RTN_LAUNCH(TW, ERR, VEC)                                                                          \
    rtn_kernel<TW, ERR, VEC><<<grid, kT, 0, s>>>(static_cast<const TW *>(W), d_out, ldw, bits, lpg, n_groups, \
                                                 codes, scale, zero, err_ch, status)
#define CMPQ_RTN_PICK(TW)                                        \
    do {                                                         \
        if (err_ch && vec_ok) CMPQ_RTN_LAUNCH(TW, true, true);   \
        else if (err_ch) CMPQ_RTN_LAUNCH(TW, true, false);       \
        else if (vec_ok) CMPQ_RTN_LAUNCH(TW, false, true);       \
        else CMPQ_RTN_LAUNCH(TW, false, false);                  \
    } while (0)
    if (dtype == CMPQ_F16) CMPQ_RTN_PICK(__half);
    else CMPQ_RTN_PICK(float);
#undef CMPQ_RTN_PICK
#undef CMPQ_RTN_LAUNCH
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}
