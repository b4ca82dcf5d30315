// Small entry points of libcmpq: error names, counts, workspace sizes, and the
// orientation helper that turns a framework's [d_out, d_in] weight into the
// d_in x d_out matrix of Sec. 3.2.1 (arXiv 2410.13056), one row per input channel.
#include "common.h"

size_t cmpq_ws_act_stats(int64_t d_in, int64_t n);
size_t cmpq_ws_allocate_bits(int64_t d_in);
size_t cmpq_ws_outlier_channels(int64_t d_in);
size_t cmpq_ws_outlier_weights(int64_t d_in, int64_t d_out, int64_t k);
size_t cmpq_ws_kmeans(int64_t d_in, int64_t d_out);
size_t cmpq_ws_pack(int64_t d_in);
size_t cmpq_ws_dequant_error(int64_t d_in);
size_t cmpq_ws_outliers_by_column(int64_t d_out, int64_t n_out);
size_t cmpq_ws_lut_matvec(int64_t d_in, int64_t d_out, int64_t m);
size_t cmpq_ws_pack_with_error(int64_t d_in);
size_t cmpq_ws_lut4();
size_t cmpq_ws_kmeans_arrangement(int64_t d_in, int64_t d_out);

extern "C" size_t cmpq_workspace_bytes(int op, int64_t d_in, int64_t d_out, int64_t n) {
    if (d_in < 0 || d_out < 0 || n < 0) return 0;
    switch (op) {
        case CMPQ_OP_ACT_STATS: return cmpq_ws_act_stats(d_in, n);
        case CMPQ_OP_ALLOCATE_BITS: return cmpq_ws_allocate_bits(d_in);
        case CMPQ_OP_OUTLIER_CHANNELS: return cmpq_ws_outlier_channels(d_in);
        case CMPQ_OP_OUTLIER_WEIGHTS: return cmpq_ws_outlier_weights(d_in, d_out, n);
        case CMPQ_OP_KMEANS: return cmpq_ws_kmeans(d_in, d_out);
        case CMPQ_OP_PACK: return cmpq_ws_pack(d_in);
        case CMPQ_OP_DEQUANT_ERROR: return cmpq_ws_dequant_error(d_in);
        case CMPQ_OP_OUTLIERS_BY_COLUMN: return cmpq_ws_outliers_by_column(d_out, n);
        case CMPQ_OP_LUT_MATVEC: return cmpq_ws_lut_matvec(d_in, d_out, n);
        case CMPQ_OP_PACK_WITH_ERROR: return cmpq_ws_pack_with_error(d_in);
        case CMPQ_OP_LUT4: return cmpq_ws_lut4();
        case CMPQ_OP_KMEANS_ARRANGEMENT: return cmpq_ws_kmeans_arrangement(d_in, d_out);
        default: return 0;
    }
}

extern "C" const char *cmpq_strerror(int code) {
    switch (code) {
        case CMPQ_OK: return "ok";
        case CMPQ_EINVAL: return "invalid argument (null pointer, negative size or unknown enum)";
        case CMPQ_ESHAPE: return "shape not supported (leading dimension or size limit)";
        case CMPQ_EBUDGET: return "bit set must be consecutive within 1..4 and hold avg_bits";
        case CMPQ_ECOUNT: return "more outliers requested than candidates";
        case CMPQ_EWORKSPACE: return "workspace missing, misaligned or too small";
        case CMPQ_EHIP: return "HIP launch failed";
        default: return "unknown cmpq error";
    }
}

extern "C" int64_t cmpq_count_ppm(int64_t ppm, int64_t n) {
    return (int64_t)(((unsigned __int128)ppm * (unsigned __int128)n + 500000u) / 1000000u);
}

namespace {

struct ArmedTimer {
    int kernel = -1;
    hipEvent_t begin = nullptr, end = nullptr;
};
thread_local ArmedTimer g_timer;

}  // namespace

extern "C" int cmpq_time_kernel(int kernel, void *event_begin, void *event_end) {
    if (kernel < 0 || kernel >= CMPQ_KERNEL_COUNT) return CMPQ_EINVAL;
    if (!event_begin || !event_end) {
        g_timer = ArmedTimer();
        return CMPQ_OK;
    }
    g_timer.kernel = kernel;
    g_timer.begin = static_cast<hipEvent_t>(event_begin);
    g_timer.end = static_cast<hipEvent_t>(event_end);
    return CMPQ_OK;
}

namespace {

// Four independent chains of dependent fused multiply-adds per lane between two readings of
// the shader-clock counter and of the constant-rate wall counter.
__global__ __launch_bounds__(256) void shader_clock_kernel(int iters, unsigned long long *ticks) {
    float a0 = (float)threadIdx.x * 1e-3f, a1 = a0 + 1.f, a2 = a0 + 2.f, a3 = a0 + 3.f;
    const float m = 0.999f, c = 1e-3f;
    const unsigned long long t0 = clock64(), w0 = wall_clock64();
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            a0 = fmaf(a0, m, c);
            a1 = fmaf(a1, m, c);
            a2 = fmaf(a2, m, c);
            a3 = fmaf(a3, m, c);
        }
    }
    const unsigned long long t1 = clock64(), w1 = wall_clock64();
    if (threadIdx.x == 0) {
        ticks[2 * blockIdx.x] = t1 - t0;
        ticks[2 * blockIdx.x + 1] = w1 - w0;
    }
    if (a0 + a1 + a2 + a3 == 12345.678f) ticks[0] = 0;  // keeps the chains alive
}

}  // namespace

extern "C" int cmpq_shader_clock_probe(int iters, int n_workgroups, uint64_t *ticks, int *wall_khz, void *stream) {
    if (!ticks || !wall_khz || iters < 1 || n_workgroups < 1 || n_workgroups > 65536) return CMPQ_EINVAL;
    int dev = 0, khz = 0;
    if (hipGetDevice(&dev) != hipSuccess) return CMPQ_EHIP;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) return CMPQ_EHIP;
    *wall_khz = khz;
    shader_clock_kernel<<<dim3((unsigned)n_workgroups), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(
        iters, reinterpret_cast<unsigned long long *>(ticks));
    return hipGetLastError() == hipSuccess ? CMPQ_OK : CMPQ_EHIP;
}

void cmpq_timing_before(int kernel, hipStream_t s) {
    if (g_timer.kernel == kernel) (void)hipEventRecord(g_timer.begin, s);
}

void cmpq_timing_after(int kernel, hipStream_t s) {
    if (g_timer.kernel == kernel) {
        (void)hipEventRecord(g_timer.end, s);
        g_timer = ArmedTimer();
    }
}

namespace {

constexpr int kTile = 64;

// dst[c, r] = src[r, c]; a 64x64 tile goes through LDS so that both the read
// and the write touch whole rows.  256 threads, each moves 16 elements.
__global__ __launch_bounds__(256) void transpose32_kernel(const uint32_t *__restrict__ src, int64_t rows,
                                                          int64_t cols, int64_t ld_src,
                                                          uint32_t *__restrict__ dst, int64_t ld_dst) {
    __shared__ uint32_t tile[kTile][kTile + 1];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.y * kTile, c0 = (int64_t)blockIdx.x * kTile;
#pragma unroll
    for (int k = 0; k < kTile; k += 4) {
        const int64_t r = r0 + ty + k, c = c0 + tx;
        if (r < rows && c < cols) tile[ty + k][tx] = src[r * ld_src + c];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTile; k += 4) {
        const int64_t c = c0 + ty + k, r = r0 + tx;
        if (c < cols && r < rows) dst[c * ld_dst + r] = tile[tx][ty + k];
    }
}

// 2-byte elements: a lane moves 4 elements (8 bytes) per access on both sides of an LDS tile of T x T.  RAGGED: any
// dimensions and alignment, 8 bytes from any even address, the last 1 to 3 elements of a row one by one.  The rows
// of a tile begin and end inside lines of memory there, so its tiles are of 128 where they fill the chip and its loads
// leave the lines they share in the cache (4099 x 3001: 13.2 us; tiles of 64 15.9, streamed loads 18.5, element by
// element 18.5).
// Else every dimension and leading dimension is a multiple of 4 and the bases are 8-byte aligned.
template <int T, bool RAGGED>
__global__ __launch_bounds__(256) void transpose16_vec_kernel(const uint16_t *__restrict__ src,
                                                              int64_t rows, int64_t cols,
                                                              int64_t ld_src,
                                                              uint16_t *__restrict__ dst,
                                                              int64_t ld_dst) {
    __shared__ uint16_t tile[T][T + 2];  // row stride T / 2 + 1 words: column reads spread over banks
    constexpr int kQuads = T / 4, kStep = 256 / kQuads, kPieces = T / kStep;
    const int t = threadIdx.x, q = t % kQuads, p = t / kQuads;  // q: group of 4 along the fast axis
    const int64_t r0 = (int64_t)blockIdx.y * T, c0 = (int64_t)blockIdx.x * T;
    uint2 v[kPieces];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int64_t r = r0 + p + kStep * k, c = c0 + 4 * q;
        v[k] = make_uint2(0, 0);
        if (r < rows && (RAGGED ? c + 4 <= cols : c < cols)) {  // the source is read once
            typedef uint32_t U2 __attribute__((ext_vector_type(2)));
            typedef uint32_t U2Any __attribute__((ext_vector_type(2), aligned(2)));
            const uint16_t *p4 = src + r * ld_src + c;
            const U2 nt = RAGGED ? (U2) * reinterpret_cast<const U2Any *>(p4)
                                 : __builtin_nontemporal_load(reinterpret_cast<const U2 *>(p4));
            v[k] = make_uint2(nt.x, nt.y);
        } else if (RAGGED && r < rows && c < cols) {
            const uint16_t *p4 = src + r * ld_src + c;
            v[k].x = p4[0];
            if (c + 1 < cols) v[k].x |= (uint32_t)p4[1] << 16;
            if (c + 2 < cols) v[k].y = p4[2];
        }
    }
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        uint32_t *w = reinterpret_cast<uint32_t *>(&tile[p + kStep * k][4 * q]);
        w[0] = v[k].x;
        w[1] = v[k].y;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int c = p + kStep * k;  // row of dst inside the tile
        const int64_t orow = c0 + c, ocol = r0 + 4 * q;
        if (orow < cols && ocol < rows) {
            uint16_t *out = dst + orow * ld_dst + ocol;
            const uint32_t a0 = tile[4 * q][c], a1 = tile[4 * q + 1][c];
            const uint32_t a2 = tile[4 * q + 2][c], a3 = tile[4 * q + 3][c];
            const uint2 four = make_uint2(a0 | (a1 << 16), a2 | (a3 << 16));
            if (!RAGGED) {
                *reinterpret_cast<uint2 *>(out) = four;
            } else if (ocol + 4 <= rows) {
                __builtin_memcpy(out, &four, 8);
            } else {
                out[0] = (uint16_t)a0;
                if (ocol + 1 < rows) out[1] = (uint16_t)a1;
                if (ocol + 2 < rows) out[2] = (uint16_t)a2;
            }
        }
    }
}

}  // namespace

extern "C" int cmpq_transpose(const void *src, int dtype, int64_t rows, int64_t cols,
                              int64_t ld_src, void *dst, int64_t ld_dst, void *stream) {
    if (rows < 0 || cols < 0 || (dtype != CMPQ_F16 && dtype != CMPQ_F32)) return CMPQ_EINVAL;
    if (rows == 0 || cols == 0) return CMPQ_OK;
    if (!src || !dst) return CMPQ_EINVAL;
    if (ld_src < cols || ld_dst < rows) return CMPQ_ESHAPE;
    const int64_t gx = cdiv(cols, kTile), gy = cdiv(rows, kTile);
    if (gy > 65535) return CMPQ_ESHAPE;
    dim3 grid((unsigned)gx, (unsigned)gy);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = dtype == CMPQ_F16 && rows % 4 == 0 && cols % 4 == 0 && ld_src % 4 == 0 &&
                     ld_dst % 4 == 0 && reinterpret_cast<uintptr_t>(src) % 8 == 0 &&
                     reinterpret_cast<uintptr_t>(dst) % 8 == 0;
    if (dtype == CMPQ_F16) {
        const uint16_t *from = static_cast<const uint16_t *>(src);
        uint16_t *to = static_cast<uint16_t *>(dst);
        if (vec) {
            cmpq_timing_before(CMPQ_KERNEL_TRANSPOSE, st);
            transpose16_vec_kernel<kTile, false><<<grid, 256, 0, st>>>(from, rows, cols, ld_src, to, ld_dst);
            cmpq_timing_after(CMPQ_KERNEL_TRANSPOSE, st);
        } else {
            // Tiles of 128 where they make 704 workgroups; with fewer, below three a compute unit, their longer way shows.
            // Us, tiles of 128 and of 64: 33 x 70000 (547 of 128) 6.2 and 5.4, 1024 x 8190 (512) 10.9 and 6.7, 2500 x
            // 2501 (400) 9.7 and 6.1, 3201 x 3200 (650) 11.7 and 10.0, 3333 x 3333 (729) 12.2 and 13.3, 4099 x 3001
            // (792) 12.4 and 15.0.
            const dim3 wide((unsigned)cdiv(cols, 2 * kTile), (unsigned)cdiv(rows, 2 * kTile));
            if ((int64_t)wide.x * wide.y >= 704)
                transpose16_vec_kernel<2 * kTile, true><<<wide, 256, 0, st>>>(from, rows, cols, ld_src, to, ld_dst);
            else
                transpose16_vec_kernel<kTile, true><<<grid, 256, 0, st>>>(from, rows, cols, ld_src, to, ld_dst);
        }
    } else {
        transpose32_kernel<<<grid, 256, 0, st>>>(static_cast<const uint32_t *>(src), rows, cols, ld_src,
                                                 static_cast<uint32_t *>(dst), ld_dst);
    }
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}
