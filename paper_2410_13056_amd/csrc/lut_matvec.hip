// The product with the deployed weight (Sec. 6 / Fig. 4 of arXiv 2410.13056): per width a
// table-driven product of the input with the packed codes of cmpq_pack, plus the rows of
// O_act and the entries of O_q.
//
//   Y[t,o] = sum_i X[t,i] * W_hat[i,o]
//
// This file multiplies one token at a time; several tokens go to the matrix cores
// (lut_gemm.hip) wherever that is faster.
//
// The packed rows are input channels, so a row contributes X[t,i] * lut_i[code] to every
// output: tables of levels are formed once per row (or pair of rows) and the rest is table
// look-ups and additions.  b/8 bytes per weight are read once per token.
//
//   * lut_matvec_kernel: a wavefront adds up a part, up to 48 rows of one width (or 8 of O_act), for a tile
//     of 2048 outputs (a lane 32 consecutive outputs: exactly B words of a row); a workgroup is
//     four parts, whose sums are added in pairs, and leaves one partial row per token.  Up to 3 bits two
//     rows are looked up at once (lut_part).  A launch serves up to 8 products (cmpq_lut_matvec_group).
//   * lut_matvec_finish_kernel: per output, the partial rows in order, then the column's O_q entries -
//     every sum in a fixed order, so the result is reproducible bit for bit.
//     One token through the seven products of a 70B-shaped block, four groups: 193 -> 158 us (main
//     kernels 158 -> 120 under the profiler: 3.9 TB/s on the largest; the finish kernels 43 -> 38).
//   * lut_matvec_half_kernel: the variant with FP16 sums, in slabs of four times 8, 16 or 32 rows.
//   * cmpq_outliers_by_column / cmpq_gather_channels prepare O_q and O_act for this once,
//     at quantization time.
#include "common.h"
#include "lut_gemm.h"
#include <limits.h>

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / CMPQ_WAVE;
constexpr int kOutPerLane = 32;                        // 32 codes = B whole words
constexpr int kTileOut = CMPQ_WAVE * kOutPerLane;      // outputs per workgroup
constexpr int kMaxRowsPerWave = 32;                    // FP16 sums: a workgroup's slab is 4 wavefronts x 8, 16 or 32 rows
constexpr int kGroup = 4;                              // FP16 sums: rows whose tables are in LDS at once
constexpr int kMaxWidths = 4;

struct LmWidth {
    const uint32_t *packed;
    const int32_t *chan_idx;
    const uint16_t *lut;
    int64_t rows, words_per_row;
    int slab0;  // index of this width's first slab among all slabs
    int bits;
};

// One product of a launch, as the kernel with FP16 sums sees it.
struct LmArgs {
    LmWidth w[kMaxWidths];
    const __half *X;
    int64_t ldx, d_out;
    float *partial;                // [tokens][n_rows_total][d_out]
    const int32_t *act_idx;
    const __half *W_act;
    int64_t k_act, ld_act;
    int n_widths, rows_per_wave;
    int n_lut_slabs, n_act_slabs;  // a layer's blockIdx.y range: O_act slabs first, then the packed slabs
    int n_rows_total;              // partial rows per token: packed slabs, then O_act slabs
    int tiles;                     // tiles of 2048 outputs
    int y0;                        // first blockIdx.y of this layer
};

constexpr int kMaxLayers = CMPQ_MAX_GROUP;

struct LmGroup {
    LmArgs l[kMaxLayers];
    int n_layers;
};

constexpr int kRedStride = CMPQ_WAVE + 1;  // sums of output k of all lanes: 64 floats, padded by one
constexpr int kRedHalf = kOutPerLane / 2;  // the sums meet in LDS in two halves of 16 outputs per lane
constexpr int kRedFloats = kRedHalf * kRedStride;

// The four wavefronts' sums of a 2048-output tile (from output o_tile on), added in pairs, into a
// partial row.  Called once by every lane of the workgroup.  Lanes write with stride 1 and read with
// stride 65: no bank is hit twice by a half-wavefront either way.  Two halves, so that the
// LDS of a workgroup stays small enough for five workgroups per compute unit.
__device__ __forceinline__ void store_partial(const float (&acc)[kOutPerLane], float (*red)[kRedFloats],
                                              float *__restrict__ prow, int64_t o_tile, int64_t d_out) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();  // the sums reuse the LDS of the tables (and of the first half)
#pragma unroll
        for (int k = 0; k < kRedHalf; ++k) red[wave][k * kRedStride + lane] = acc[h * kRedHalf + k];
        __syncthreads();
        // lane l holds outputs 32 l .. 32 l + 31 of the tile; this half covers k = 16 h .. 16 h + 15
        for (int c = threadIdx.x; c < kTileOut / 2; c += kThreads) {
            const int l = c / kRedHalf, k = c % kRedHalf;
            const int64_t o = o_tile + l * kOutPerLane + h * kRedHalf + k;
            if (o < d_out) {
                const int at = k * kRedStride + l;
                static_assert(kWaves == 4, "");
                prow[o] = (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]);
            }
        }
    }
}

// (code << 2) + base in one instruction.  Written out because the compiler otherwise turns
// the extract-then-shift into shift-mask-add, one instruction more per weight.
__device__ __forceinline__ uint32_t entry_offset(uint32_t code, uint32_t base) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(r) : "v"(code), "v"(base));
    return r;
}

// Field p of `bits` bits of a lane's words (two instructions where it straddles two words).
template <int B, int PB>
__device__ __forceinline__ uint32_t field_at(const uint32_t (&w)[B], int p) {
    const int bit = p * PB, idx = bit >> 5, sh = bit & 31;
    if (sh + PB <= 32) return __builtin_amdgcn_ubfe(w[idx], sh, PB);
    return __builtin_amdgcn_alignbit(w[idx + 1 < B ? idx + 1 : idx], w[idx], sh) & ((1u << PB) - 1u);
}

// ---- fp32 sums: a wavefront's part

// A layer's rows of one width (or of O_act, bits = 16), in parts of about even cost: a wavefront adds up
// one part for a tile of 2048 outputs, a workgroup four parts.
struct MvWidth {
    const uint32_t *packed;
    const int32_t *chan;
    const uint16_t *lut;
    int rows, words_per_row, bits, part0, parts;
};
constexpr int kActBits = 16;
struct MvLayer {
    MvWidth w[kMaxWidths + 1];
    const __half *X, *W_act;
    int64_t ldx, ld_act;
    float *partial;                // [tokens][slabs][d_out]
    int d_out, n_w, slabs;
};
struct MvGroup {
    int wg0[kMaxLayers];  // first workgroup of each layer (past the last layer: INT_MAX)
    MvLayer l[kMaxLayers];
};
static_assert(sizeof(MvGroup) <= 4096, "travels in the kernel arguments");

// Widths 1 to 3: the rows of a pair are looked up at once.  Their codes of one output make an index into
// a table of 4^B sums x0 * level0 + x1 * level1 (products exact, sum rounded once), so an output costs
// one extract, one address, one LDS read and one addition for two weights.
template <int B>
struct PairWords {
    static constexpr uint32_t mask(int q) {  // word q: the fields of even outputs
        uint32_t m = 0;
        for (int p = 0; p < 32; ++p) m |= (uint32_t)((32 * q + p) % (2 * B) < B) << p;
        return m;
    }
    uint32_t even[B], odd[B];  // pairs of codes of the even / odd outputs: pair i at bit 2 B i
    __device__ __forceinline__ PairWords(const uint32_t (&a)[B], const uint32_t (&b)[B]) {
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const uint32_t up = q ? __builtin_amdgcn_alignbit(b[q], b[q - 1], 32 - B) : b[0] << B;
            const uint32_t down = q + 1 < B ? __builtin_amdgcn_alignbit(a[q + 1], a[q], B) : a[q] >> B;
            even[q] = (a[q] & mask(q)) | (up & ~mask(q));
            odd[q] = (down & mask(q)) | (b[q] & ~mask(q));
        }
    }
};

// base + 4 * (nibble I of n), t the even or odd nibbles of n times 4, a byte each.
__device__ __forceinline__ uint32_t nibbles4(uint32_t n, bool odd) { return (odd ? n >> 2 : n << 2) & 0x3c3c3c3cu; }

// Rows whose tables are in LDS at once, LDS of a wavefront: two such groups.
template <int B>
constexpr int kPartGroup = B <= 2 ? 8 : 4;
constexpr int kPartTable = 512;  // bytes of a group's tables: 16 entries for each of 4 rows or pairs, 64 for each of 2 pairs
constexpr int kMaxPartRows = CMPQ_WAVE;  // a lane keeps the input of one row

// What bounds it: vector instructions - 1.9 a weight at 3 bits, 2.6 at 4, 1.5 at 2 - and LDS reads (half
// a read a weight up to 3 bits, with two-way conflicts at 3).  With one table a row at 3 bits, extracts
// of single codes at 4 and pairs of outputs at 2 it were 3.1, 3.1 and 2.1.
template <int B>
__device__ __forceinline__ void lut_part(const MvLayer &a, const MvWidth &wd, const __half *__restrict__ x, int r0, int n,
                                         int tile, unsigned char *tables, float (&acc)[kOutPerLane]) {
    constexpr int K = 1 << B, G = kPartGroup<B>;
    constexpr bool kPairs = B <= 3;
    constexpr int KP = kPairs ? K * K : K, kTables = kPairs ? G / 2 : G;  // entries of a table, tables of a group
    constexpr int kPasses = kTables * KP > CMPQ_WAVE ? kTables * KP / CMPQ_WAVE : 1, kPerPass = kTables / kPasses;
    static_assert(kTables * KP * 4 <= kPartTable && kPerPass * KP <= CMPQ_WAVE, "");
    const int lane = threadIdx.x & (CMPQ_WAVE - 1);
    const float x_mine = lane < n ? __half2float(x[wd.chan[r0 + lane]]) : 0.f;
    // entry `fe` of table `ft` of a pass
    const int ft = lane / KP, fe = lane % KP;
    const uint16_t *lut = wd.lut + (int64_t)r0 * K;
    // levels of a group's tables (past the end those of the last row again, dropped when they are written)
    struct Levels {
        uint16_t lo[kPasses], hi[kPasses];
    };
    auto fetch_levels = [&](int r, Levels &v) {
#pragma unroll
        for (int f = 0; f < kPasses; ++f) {
            if constexpr (kPairs) {
                const int row = r + 2 * (f * kPerPass + ft);
                v.lo[f] = lut[min(row, n - 1) * K + (fe & (K - 1))];
                v.hi[f] = lut[min(row + 1, n - 1) * K + ((fe >> B) & (K - 1))];
            } else {
                v.lo[f] = lut[min(r + ft, n - 1) * K + fe];
            }
        }
    };
    auto write_tables = [&](int r, const Levels &v, unsigned char *buf) {
#pragma unroll
        for (int f = 0; f < kPasses; ++f) {
            const int row = r + (kPairs ? 2 : 1) * (f * kPerPass + ft);
            float e = row < n ? __half2float(__ushort_as_half(v.lo[f])) : 0.f;
            if constexpr (kPairs) {
                const float x0 = __shfl(x_mine, row & (CMPQ_WAVE - 1), CMPQ_WAVE), x1 = __shfl(x_mine, (row + 1) & (CMPQ_WAVE - 1), CMPQ_WAVE);
                e = fmaf(x0, e, x1 * (row + 1 < n ? __half2float(__ushort_as_half(v.hi[f])) : 0.f));
            }
            if (kPerPass * KP == CMPQ_WAVE || lane < kPerPass * KP) reinterpret_cast<float *>(buf)[f * CMPQ_WAVE + lane] = e;
        }
    };
    // A lane's B words of a row: one vector load where the tile is whole, else word by word, past the end of
    // the row its last one again (outputs that are not there are not written).  Past the last row that one
    // again: its tables are zero.
    const int64_t wpr = wd.words_per_row;
    const bool whole = (tile + 1) * (kTileOut / 32) * B <= wd.words_per_row;
    const uint32_t *packed = wd.packed + (int64_t)r0 * wpr + (whole ? tile * (kTileOut / 32) * B : 0);
    const uint32_t word0 = (uint32_t)((whole ? 0 : tile * (kTileOut / 32) * B) + lane * B);
    auto load_words = [&](int r, uint32_t (&w)[G][B]) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t *p = packed + (int64_t)min(r + g, n - 1) * wpr;  // uniform
            if (whole) {
                typedef uint32_t WordsB __attribute__((ext_vector_type(B), aligned(4)));
                // (a uniform base and a 32-bit offset; a token reads the codes once)
                const WordsB v = __builtin_nontemporal_load(reinterpret_cast<const WordsB *>(reinterpret_cast<const char *>(p) + word0 * 4u));
#pragma unroll
                for (int j = 0; j < B; ++j) w[g][j] = v[j];
            } else {
#pragma unroll
                for (int j = 0; j < B; ++j)
                    w[g][j] = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(p) + min(word0 + j, (uint32_t)wpr - 1u) * 4u);
            }
        }
    };
    auto add_up = [&](int r, const uint32_t (&w)[G][B], uint32_t at) {
#pragma unroll
        for (int t = 0; t < kTables; ++t) {
            if constexpr (B == 4) {
                // (the input multiplies here, not in the table: no lane needs another row's)
                const float xi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x_mine), (r + t) & (CMPQ_WAVE - 1)));
#pragma unroll
                for (int q = 0; q < B; ++q)
#pragma unroll
                    for (int odd = 0; odd < 2; ++odd) {
                        const uint32_t n4 = nibbles4(w[t][q], odd);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float &y = acc[8 * q + 2 * i + odd];
                            y = fmaf(xi, lds_read<float>(add_byte(at, n4, i) + t * KP * 4), y);
                        }
                    }
            } else {
                const PairWords<B> pw(w[2 * t], w[2 * t + 1]);
                if constexpr (B == 2) {
#pragma unroll
                    for (int q = 0; q < B; ++q)
#pragma unroll
                        for (int odd = 0; odd < 2; ++odd) {
                            const uint32_t ne = nibbles4(pw.even[q], odd), no = nibbles4(pw.odd[q], odd);
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int o = 16 * q + 2 * (2 * i + odd);
                                acc[o] += lds_read<float>(add_byte(at, ne, i) + t * KP * 4);
                                acc[o + 1] += lds_read<float>(add_byte(at, no, i) + t * KP * 4);
                            }
                        }
                } else {
#pragma unroll
                    for (int i = 0; i < kOutPerLane / 2; ++i) {
                        acc[2 * i] += lds_read<float>(entry_offset(field_at<B, 2 * B>(pw.even, i), at) + t * KP * 4);
                        acc[2 * i + 1] += lds_read<float>(entry_offset(field_at<B, 2 * B>(pw.odd, i), at) + t * KP * 4);
                    }
                }
            }
        }
    };
    // Words are fetched one group ahead, levels two; a group's tables are written while the group
    // before is worked on, into the buffer its predecessor has left.
    uint32_t w0[G][B], w1[G][B];
    Levels v;
    const uint32_t at = (uint32_t)reinterpret_cast<uintptr_t>(tables);
    fetch_levels(0, v);
    load_words(0, w0);
    write_tables(0, v, tables);
    fetch_levels(G, v);
    wave_fence();
#pragma unroll 1
    for (int r = 0; r < n; r += 2 * G) {
        write_tables(r + G, v, tables + kPartTable);
        load_words(r + G, w1);
        fetch_levels(r + 2 * G, v);
        add_up(r, w0, at);
        wave_fence();
        if (r + G >= n) break;
        write_tables(r + 2 * G, v, tables);
        load_words(r + 2 * G, w0);
        fetch_levels(r + 3 * G, v);
        add_up(r + G, w1, at + kPartTable);
        wave_fence();
    }
}

// The variant that adds up in FP16 (the paper's product keeps FP16 throughout, Sec. 6): the
// products x * level are rounded to FP16, and a wavefront adds those of its run of at most 32
// rows of a slab in FP16, two outputs per packed addition; the run's sums are then widened
// to fp32 and take the same way as the fp32 parts' (added over wavefronts, slabs, O_act and O_q in
// fp32, in a fixed order).  Every width looks two neighbouring codes up at once: per row a
// table of 2^(2B) pairs (product of the even output's code, product of the odd one's), 4
// bytes an entry, built from the row's 2^B products with two LDS reads per entry (for width
// 4: four entries per lane and row from one 8-byte read, one 2-byte read and one 16-byte
// store).  A weight then costs half an extract, half a shift-and-add, half an LDS read and
// half a packed addition.  Tables of 64 and 256 entries wrap around the LDS banks, so their
// reads collide; with 4-byte entries that costs less than the instructions saved (with the
// 8-byte entries of fp32 pairs it did not).  Words and levels are
// fetched a group ahead, tables are double-buffered.
constexpr int kHalfPairBytes = kGroup * 256 * 4;               // pair tables of a group of rows at width 4
constexpr int kHalfBufBytes = kHalfPairBytes + kGroup * 16 * 2;  // + the rows' own products
constexpr int kHalfLdsBytes = kWaves * 2 * kHalfBufBytes;

template <int B>
__device__ __forceinline__ void lut_slab_half(const LmArgs &a, const LmWidth &wd, int slab, unsigned char *smem,
                                              float (*red)[kRedFloats]) {
    constexpr int K = 1 << B, PB = 2 * B, KP = 1 << PB;
    const __half *__restrict__ X = a.X;
    const int64_t d_out = a.d_out;
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const int64_t token = blockIdx.z;
    const __half *x = X + token * a.ldx;
    const int64_t word0 = (int64_t)blockIdx.x * (kTileOut / 32) * B + (int64_t)lane * B;
    const int64_t r0 = ((int64_t)slab * kWaves + wave) * a.rows_per_wave;
    const int64_t r1 = min(wd.rows, r0 + a.rows_per_wave);
    __half2 acc2[kOutPerLane / 2];
#pragma unroll
    for (int p = 0; p < kOutPerLane / 2; ++p) acc2[p] = __half2{__ushort_as_half(0), __ushort_as_half(0)};

    // product (row g, level c) of a group is formed by lane g * K + c
    const int fill_g = lane / K, fill_c = lane % K;
    auto product = [&](int64_t r) -> uint32_t {
        if (fill_g >= kGroup || r + fill_g >= r1) return 0u;  // rows past the end: tables of zeros
        const int64_t row = r + fill_g;
        const float xi = __half2float(x[wd.chan_idx[row]]);
        return __half_as_ushort(__float2half_rn(xi * __half2float(__ushort_as_half(wd.lut[row * K + fill_c]))));
    };
    const bool full = word0 + B <= wd.words_per_row;
    auto load_words = [&](int64_t r, uint32_t (&w)[kGroup][B]) {
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            const uint32_t *p = wd.packed + (r + g) * wd.words_per_row + word0;
            if (r + g < r1 && full) {
                typedef uint32_t WordsB __attribute__((ext_vector_type(B), aligned(4)));
                const WordsB v = __builtin_nontemporal_load(reinterpret_cast<const WordsB *>(p));
#pragma unroll
                for (int j = 0; j < B; ++j) w[g][j] = v[j];
            } else {
#pragma unroll
                for (int j = 0; j < B; ++j) w[g][j] = (r + g < r1 && word0 + j < wd.words_per_row) ? p[j] : 0u;
            }
        }
    };

    if (r0 < r1) {
        uint32_t w[kGroup][B], wn[kGroup][B];
        uint32_t e = product(r0), en = 0u;
        load_words(r0, w);
        int buf = 0;
        for (int64_t r = r0; r < r1; r += kGroup) {
            unsigned char *mine = smem + (wave * 2 + buf) * kHalfBufBytes;
            uint32_t *pair = reinterpret_cast<uint32_t *>(mine);
            uint16_t *own = reinterpret_cast<uint16_t *>(mine + kHalfPairBytes);  // [row of the group][level]
            if (kGroup * K >= CMPQ_WAVE || lane < kGroup * K) own[lane % (kGroup * K)] = (uint16_t)e;
            if (r + kGroup < r1) {
                en = product(r + kGroup);
                load_words(r + kGroup, wn);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if constexpr (B == 4) {
                // lane: odd output's code c1 = lane / 4, even output's codes 4 (lane % 4) .. + 3
                const int c1 = lane >> 2, c0 = (lane & 3) * 4;
#pragma unroll
                for (int g = 0; g < kGroup; ++g) {
                    const uint32_t hi = (uint32_t)own[g * K + c1] << 16;
                    const uint2 q = *reinterpret_cast<const uint2 *>(own + g * K + c0);
                    uint4 v;
                    v.x = (q.x & 0xffffu) | hi;
                    v.y = (q.x >> 16) | hi;
                    v.z = (q.y & 0xffffu) | hi;
                    v.w = (q.y >> 16) | hi;
                    *reinterpret_cast<uint4 *>(pair + g * KP + c1 * K + c0) = v;
                }
            } else {
#pragma unroll
                for (int t0 = 0; t0 < kGroup * KP; t0 += CMPQ_WAVE) {
                    const int t = t0 + lane;
                    if (kGroup * KP % CMPQ_WAVE == 0 || t < kGroup * KP) {
                        const int g = t / KP, ent = t % KP;
                        pair[t] = (uint32_t)own[g * K + (ent & (K - 1))] | ((uint32_t)own[g * K + (ent >> B)] << 16);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const char *base = reinterpret_cast<const char *>(smem);
            const uint32_t wb = (uint32_t)((wave * 2 + buf) * kHalfBufBytes);
#pragma unroll
            for (int g = 0; g < kGroup; ++g) {
#pragma unroll
                for (int p = 0; p < kOutPerLane / 2; ++p) {
                    const uint32_t v = *reinterpret_cast<const uint32_t *>(base + g * (KP * 4) + entry_offset(field_at<B, PB>(w[g], p), wb));
                    acc2[p] = __hadd2(acc2[p], __half2{__ushort_as_half((unsigned short)(v & 0xffffu)), __ushort_as_half((unsigned short)(v >> 16))});
                }
            }
            __builtin_amdgcn_wave_barrier();
            buf ^= 1;
            e = en;
#pragma unroll
            for (int g = 0; g < kGroup; ++g)
#pragma unroll
                for (int j = 0; j < B; ++j) w[g][j] = wn[g][j];
        }
    }
    float acc[kOutPerLane];
#pragma unroll
    for (int p = 0; p < kOutPerLane / 2; ++p) {
        acc[2 * p] = __low2float(acc2[p]);
        acc[2 * p + 1] = __high2float(acc2[p]);
    }
    store_partial(acc, red, a.partial + (token * a.n_rows_total + wd.slab0 + slab) * d_out, (int64_t)blockIdx.x * kTileOut, d_out);
}

// Rows of O_act: up to 8 rows of FP16 weights per wavefront times their inputs (few rows, so
// short parts: the loop over rows is bound by latency).  A lane reads its 32 outputs of a
// row as four 16-byte pieces, two rows in flight; the rows' inputs are fetched up front,
// one per lane.
constexpr int kActRowsPerWave = 8;

template <typename Args>
__device__ __forceinline__ void act_rows(const Args &a, const int32_t *__restrict__ act_idx, const __half *__restrict__ x,
                                         int64_t r0, int n, int64_t o0, float (&acc)[kOutPerLane]) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1);
    const float x_mine = lane < n ? __half2float(x[act_idx[r0 + lane]]) : 0.f;
    // every row's input in a scalar register (rows past the count: 0), read before lanes part ways
    float xs[kActRowsPerWave];
#pragma unroll
    for (int j = 0; j < kActRowsPerWave; ++j)
        xs[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x_mine), j));
    const int d_out = (int)a.d_out;
    with_act_mode(d_out, o0 - lane * kOutPerLane + kTileOut <= d_out, [&](auto mode) {
#pragma unroll
        for (int j = 0; j < kActRowsPerWave; j += 2) {
            if (j >= n) break;
            uint4 raw[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // (a second row that is not there is read again from the first, and left out)
                const __half *row = a.W_act + (r0 + (j + u < n ? j + u : j)) * a.ld_act;
#pragma unroll
                for (int q = 0; q < 4; ++q) raw[u][q] = act_outputs8<decltype(mode)::value>(row, (int)o0 + 8 * q, d_out);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (j + u >= n) break;
                const __half2 *h = reinterpret_cast<const __half2 *>(raw[u]);
#pragma unroll
                for (int k = 0; k < kOutPerLane / 2; ++k) {
                    const float2 wv = __half22float2(h[k]);
                    acc[2 * k] = fmaf(xs[j + u], wv.x, acc[2 * k]);
                    acc[2 * k + 1] = fmaf(xs[j + u], wv.y, acc[2 * k + 1]);
                }
            }
        }
    });
}

__device__ __forceinline__ void act_slab(const LmArgs &a, int slab, float (*red)[kRedFloats]) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const int64_t token = blockIdx.z, o_tile = (int64_t)blockIdx.x * kTileOut;
    const int64_t r0 = ((int64_t)slab * kWaves + wave) * kActRowsPerWave;
    float acc[kOutPerLane];
#pragma unroll
    for (int k = 0; k < kOutPerLane; ++k) acc[k] = 0.f;
    act_rows(a, a.act_idx, a.X + token * a.ldx, r0, (int)max((int64_t)0, min(a.k_act - r0, (int64_t)kActRowsPerWave)),
             o_tile + (int64_t)lane * kOutPerLane, acc);
    store_partial(acc, red, a.partial + (token * a.n_rows_total + a.n_lut_slabs + slab) * a.d_out, o_tile, a.d_out);
}

// The rows of part `p` of a width: even shares of its row groups (of O_act: kActRowsPerWave rows).  Past the last part: none.
__host__ __device__ __forceinline__ void rows_of_part(const MvWidth &wd, int p, int &r0, int &n) {
    if (wd.bits == kActBits) {
        r0 = p * kActRowsPerWave;
        n = wd.rows - r0 < kActRowsPerWave ? wd.rows - r0 : kActRowsPerWave;
        return;
    }
    const int shift = wd.bits <= 2 ? 3 : 2, groups = (wd.rows + (1 << shift) - 1) >> shift;
    const int at = p < wd.parts ? p : wd.parts, next = at < wd.parts ? at + 1 : at;
    r0 = share_of(groups, at, wd.parts) << shift;
    const int r1 = share_of(groups, next, wd.parts) << shift;
    n = (r1 < wd.rows ? r1 : wd.rows) - r0;
}

// Workgroups of a layer: per tile of 2048 outputs its slabs of four parts, side by side, so that every
// compute unit gets parts of all widths; blockIdx.y: token.
__global__ __launch_bounds__(kThreads) void lut_matvec_kernel(MvGroup g) {
    // the tables of the look-ups and, after them, the wavefronts' sums share one piece of LDS
    __shared__ __align__(16) float smem[kWaves * kRedFloats];
    static_assert(kWaves * 2 * kPartTable <= kWaves * kRedFloats * (int)sizeof(float), "the tables fit the shared piece");
    float(*red)[kRedFloats] = reinterpret_cast<float(*)[kRedFloats]>(smem);
    int l = 0;
#pragma unroll
    for (int i = 1; i < kMaxLayers; ++i) l += (int)blockIdx.x >= g.wg0[i];
    const MvLayer &a = g.l[l];
    const int wg = (int)blockIdx.x - g.wg0[l], slab = wg % a.slabs, tile = wg / a.slabs;
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const int64_t token = blockIdx.y, o_tile = (int64_t)tile * kTileOut;
    const int part = slab * kWaves + wave;
    int j = 0;
#pragma unroll
    for (int i = 1; i <= kMaxWidths; ++i) j += i < a.n_w && part >= a.w[i].part0;
    const MvWidth &wd = a.w[j];
    const __half *x = a.X + token * a.ldx;
    const int p = part - wd.part0;  // parts past the last one of the last slab are empty
    int r0, n;
    rows_of_part(wd, p, r0, n);
    float acc[kOutPerLane];
#pragma unroll
    for (int k = 0; k < kOutPerLane; ++k) acc[k] = 0.f;
    if (n > 0) {
        unsigned char *tables = reinterpret_cast<unsigned char *>(smem) + wave * 2 * kPartTable;
        switch (wd.bits) {
            case 1: lut_part<1>(a, wd, x, r0, n, tile, tables, acc); break;
            case 2: lut_part<2>(a, wd, x, r0, n, tile, tables, acc); break;
            case 3: lut_part<3>(a, wd, x, r0, n, tile, tables, acc); break;
            case 4: lut_part<4>(a, wd, x, r0, n, tile, tables, acc); break;
            default: act_rows(a, wd.chan, x, r0, n, o_tile + (int64_t)lane * kOutPerLane, acc); break;
        }
    }
    store_partial(acc, red, a.partial + (token * a.slabs + slab) * a.d_out, o_tile, a.d_out);
}

// The packed rows added up in FP16 (lut_slab_half); grid: (tiles of 2048 outputs of the widest layer; per
// layer its O_act slabs, then its packed slabs of all widths one after the other; tokens).
__global__ __launch_bounds__(kThreads) void lut_matvec_half_kernel(LmGroup g) {
    __shared__ __align__(16) unsigned char smem[kHalfLdsBytes];
    static_assert(kHalfLdsBytes >= kWaves * kRedFloats * (int)sizeof(float), "the wavefronts' sums fit the shared piece");
    float(*red)[kRedFloats] = reinterpret_cast<float(*)[kRedFloats]>(smem);
    int l = 0;
    while (l + 1 < g.n_layers && (int)blockIdx.y >= g.l[l + 1].y0) ++l;
    const LmArgs &a = g.l[l];
    if ((int)blockIdx.x >= a.tiles) return;
    int y = (int)blockIdx.y - a.y0;
    if (y < a.n_act_slabs) {
        act_slab(a, y, red);
        return;
    }
    y -= a.n_act_slabs;
    int j = 0;
    while (j + 1 < a.n_widths && y >= a.w[j + 1].slab0) ++j;
    const LmWidth &wd = a.w[j];
    const int slab = y - wd.slab0;
    switch (wd.bits) {
        case 1: lut_slab_half<1>(a, wd, slab, smem, red); break;
        case 2: lut_slab_half<2>(a, wd, slab, smem, red); break;
        case 3: lut_slab_half<3>(a, wd, slab, smem, red); break;
        default: lut_slab_half<4>(a, wd, slab, smem, red); break;
    }
}

constexpr int kFinCols = 16;  // outputs per workgroup
constexpr int kFinRuns = kThreads / kFinCols;

// 16 consecutive outputs per workgroup of 256 lanes.
//   * partial rows: cut into 16 runs of consecutive rows; lane (run, output) adds its run up in eights,
//     each in pairs; the loads of the first eight are on their way before anything else.
//   * O_q: 16 lanes per column; lane l takes the column's entries l, l+16, ... (8 in flight)
//     and adds them in that order.
// Per output, the 16 run sums are added in pairs, then the 16 O_q sums in lane order.
struct FinArgs {
    const __half *X;
    int64_t ldx, d_out;
    const float *partial;
    const int32_t *colptr, *row_idx;
    const float *delta;
    float *Y;
    int64_t ldy;
    int n_rows_total;
    int x0;  // first blockIdx.x of this layer
};

struct FinGroup {
    FinArgs l[kMaxLayers];
    int n_layers;
};

__global__ __launch_bounds__(kThreads, 8) void lut_matvec_finish_kernel(FinGroup g) {
    int l = 0;
    while (l + 1 < g.n_layers && (int)blockIdx.x >= g.l[l + 1].x0) ++l;
    const FinArgs &a = g.l[l];
    constexpr int U = 8, kInFlight = 8;
    __shared__ float part[kFinRuns][kFinCols + 1];
    __shared__ float sp[kFinCols][kFinRuns + 1];
    const int hi = threadIdx.x / kFinCols, lo = threadIdx.x % kFinCols;
    const int64_t d_out = a.d_out, token = blockIdx.y, o0 = (int64_t)((int)blockIdx.x - a.x0) * kFinCols;
    const int n_rows = a.n_rows_total;
    // partial rows of output o0 + lo, run hi
    const int per = (n_rows + kFinRuns - 1) / kFinRuns, r0 = hi * per, r1 = o0 + lo < d_out ? min(n_rows, r0 + per) : 0;
    const float *p = a.partial + token * n_rows * d_out + o0 + lo;
    float v[kInFlight];
    auto fetch = [&](int r) {
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) v[q] = r + q < r1 ? p[(int64_t)(r + q) * d_out] : 0.f;
    };
    auto pairwise = [&] { return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])); };
    static_assert(kInFlight == 8, "");
    fetch(r0);
    // O_q of column o0 + hi, entries lo, lo + 16, ...
    const int32_t *__restrict__ colptr = a.colptr;
    float t = 0.f;
    if (colptr && o0 + hi < d_out) {
        const int32_t *__restrict__ row_idx = a.row_idx;
        const float *__restrict__ delta = a.delta;
        const __half *x = a.X + token * a.ldx;
        const int e1 = colptr[o0 + hi + 1];
        for (int e = colptr[o0 + hi] + lo; e < e1; e += 16 * U) {
            int32_t r[U];
            float d[U], xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ee = e + 16 * u;
                const bool ok = ee < e1;
                r[u] = ok ? row_idx[ee] : -1;
                d[u] = ok ? delta[ee] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = r[u] >= 0 ? __half2float(x[r[u]]) : 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) t = fmaf(xv[u], d[u], t);
        }
    }
    sp[hi][lo] = t;
    float y = pairwise();
    for (int r = r0 + kInFlight; r < r1; r += kInFlight) {
        fetch(r);
        y += pairwise();
    }
    part[hi][lo] = y;
    __syncthreads();
    if (threadIdx.x < kFinCols && o0 + threadIdx.x < d_out) {
        float dense[kFinRuns], sparse = 0.f;
#pragma unroll
        for (int q = 0; q < kFinRuns; ++q) dense[q] = part[q][threadIdx.x];
#pragma unroll
        for (int n = kFinRuns / 2; n > 0; n /= 2)
#pragma unroll
            for (int q = 0; q < n; ++q) dense[q] = dense[2 * q] + dense[2 * q + 1];
#pragma unroll
        for (int q = 0; q < 16; ++q) sparse += sp[threadIdx.x][q];
        a.Y[token * a.ldy + o0 + threadIdx.x] = dense[0] + sparse;
    }
}

template <typename TW>
__global__ __launch_bounds__(kThreads) void gather_channels_kernel(const TW *__restrict__ W, int64_t d_out,
                                                                    int64_t ldw,
                                                                    const int32_t *__restrict__ act_idx,
                                                                    uint16_t *__restrict__ W_act,
                                                                    int64_t ld_act) {
    const int64_t j = blockIdx.y;
    const int64_t i = act_idx[j];
    for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < d_out; o += (int64_t)gridDim.x * kThreads)
        W_act[j * ld_act + o] = __half_as_ushort(__float2half_rn(load_as_f32<TW>(W, i * ldw + o)));
}

// ---- O_q by output column

__global__ void obc_zero_kernel(int32_t *cnt, int64_t n) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        cnt[t] = 0;
}

__global__ void obc_count_kernel(const int32_t *__restrict__ out_idx, int64_t n_out, int64_t d_out,
                                 int32_t *__restrict__ cnt) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_out; e += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[out_idx[e] % d_out], 1);
}

// One workgroup: exclusive prefix of the column counts -> colptr and the scatter cursors.
__global__ __launch_bounds__(1024) void obc_scan_kernel(const int32_t *__restrict__ cnt, int64_t d_out,
                                                        int32_t *__restrict__ colptr,
                                                        int32_t *__restrict__ cursor) {
    __shared__ uint32_t scan[17];
    uint32_t run = 0;
    for (int64_t base = 0; base < d_out; base += 1024) {
        const int64_t o = base + threadIdx.x;
        const uint32_t c = o < d_out ? (uint32_t)cnt[o] : 0u;
        uint32_t total;
        const uint32_t before = run + block_scan_excl_u32(c, scan, &total);
        if (o < d_out) {
            colptr[o] = (int32_t)before;
            cursor[o] = (int32_t)before;
        }
        run += total;
    }
    if (threadIdx.x == 0) colptr[d_out] = (int32_t)run;
}

__global__ void obc_scatter_kernel(const int32_t *__restrict__ out_idx, const uint16_t *__restrict__ out_val,
                                   int64_t n_out, int64_t d_out, const float *__restrict__ centroids,
                                   const uint8_t *__restrict__ codes, int32_t *__restrict__ cursor,
                                   int32_t *__restrict__ row_idx, float *__restrict__ delta) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_out; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t lin = out_idx[e];
        const int32_t i = lin / (int32_t)d_out, o = lin % (int32_t)d_out;
        const float level = __half2float(__float2half_rn(centroids[(int64_t)i * CMPQ_KMAX + (codes[lin] & 15)]));
        const int32_t pos = atomicAdd(&cursor[o], 1);
        row_idx[pos] = i;
        delta[pos] = __half2float(__ushort_as_half(out_val[e])) - level;
    }
}

// The scatter leaves a column's entries in any order.  Channels are distinct inside a
// column, so ordering by channel gives one well-defined result.  A wavefront per column:
// an entry's final place is the number of entries of the column with a smaller channel
// (every lane walks the whole column; columns hold a few hundred entries).  A column longer
// than kRankLimit is ordered by one lane with a shell sort instead.
constexpr int kRankLimit = 2048;

__global__ __launch_bounds__(kThreads) void obc_order_kernel(const int32_t *__restrict__ colptr, int64_t d_out,
                                                              const int32_t *__restrict__ tmp_row,
                                                              const float *__restrict__ tmp_delta,
                                                              int32_t *__restrict__ row_idx,
                                                              float *__restrict__ delta) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const int64_t o = (int64_t)blockIdx.x * kWaves + wave;
    if (o >= d_out) return;
    const int b = colptr[o], n = colptr[o + 1] - b;
    if (n <= kRankLimit) {
        for (int e = lane; e < n; e += CMPQ_WAVE) {
            const int32_t mine = tmp_row[b + e];
            int rank = 0;
            for (int f = 0; f < n; ++f) rank += tmp_row[b + f] < mine;
            row_idx[b + rank] = mine;
            delta[b + rank] = tmp_delta[b + e];
        }
        return;
    }
    for (int e = lane; e < n; e += CMPQ_WAVE) {
        row_idx[b + e] = tmp_row[b + e];
        delta[b + e] = tmp_delta[b + e];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane != 0) return;
    int32_t *r = row_idx + b;
    float *d = delta + b;
    int gap = 1;
    while (gap < n / 3) gap = 3 * gap + 1;
    for (; gap >= 1; gap /= 3) {
        for (int i = gap; i < n; ++i) {
            const int32_t kr = r[i];
            const float kd = d[i];
            int j = i;
            while (j >= gap && r[j - gap] > kr) {
                r[j] = r[j - gap];
                d[j] = d[j - gap];
                j -= gap;
            }
            r[j] = kr;
            d[j] = kd;
        }
    }
}

int64_t total_slabs(const int64_t *counts, int n_set, int rows_per_wave) {
    int64_t s = 0;
    for (int j = 0; j < n_set; ++j) s += cdiv(counts[j] > 0 ? counts[j] : 0, (int64_t)kWaves * rows_per_wave);
    return s;
}

}  // namespace

// counts | cursors | channel and delta of every entry in scatter order
size_t cmpq_ws_outliers_by_column(int64_t d_out, int64_t n_out) {
    return align_up((size_t)(d_out + 1) * sizeof(int32_t), 256) * 2 + align_up((size_t)n_out * 4, 256) * 2;
}

// Token by token.  Upper bound without the per-width counts: every width and O_act may end with a
// partly filled slab.
static size_t ws_token_by_token(int64_t d_in, int64_t d_out, int64_t m) {
    const int64_t slabs = cdiv(d_in, (int64_t)kWaves * 8) + kMaxWidths + 2;  // the smallest slabs
    return align_up((size_t)m * (size_t)slabs * (size_t)d_out * sizeof(float), 256);
}

// Where several tokens go to the matrix cores: what they need there, and room for the product with
// FP16 sums, which works through its tokens in as many parts as that makes: one token at least, up to
// 32 MB of tokens with the smallest slabs (which it cuts where there is little work) and up to 128 MB
// with the largest (8192x28672, 16 tokens: 418 us in one part, 436 in two, 472 in six).
size_t cmpq_ws_lut_matvec(int64_t d_in, int64_t d_out, int64_t m) {
    if (m < 2 || d_in <= 0 || d_out <= 0 || !lut_gemm_takes(d_in, d_out, m)) return ws_token_by_token(d_in, d_out, m);
    auto tokens = [&](int64_t room, int64_t token) { return room / token < 1 ? 1 : (room / token < m ? room / token : m); };
    const int64_t slabs = cdiv(d_in, (int64_t)kWaves * kMaxRowsPerWave) + kMaxWidths + 2;
    const int64_t token = slabs * d_out * (int64_t)sizeof(float);
    size_t b = ws_token_by_token(d_in, d_out, tokens((int64_t)32 << 20, (int64_t)ws_token_by_token(d_in, d_out, 1)));
    const size_t large = align_up((size_t)token * (size_t)tokens((int64_t)128 << 20, token), 256);
    const size_t together = lut_gemm_ws_bytes(d_in, d_out, m);
    if (large > b) b = large;
    return together > b ? together : b;
}

extern "C" int cmpq_gather_channels(const void *W, int dtype, int64_t d_in, int64_t d_out, int64_t ldw,
                                    const int32_t *act_idx, int64_t k_act, uint16_t *W_act,
                                    int64_t ld_act, void *stream) {
    if (d_in < 0 || d_out < 0 || k_act < 0 || k_act > d_in) return CMPQ_EINVAL;
    if (dtype != CMPQ_F16 && dtype != CMPQ_F32) return CMPQ_EINVAL;
    if (k_act == 0 || d_out == 0) return CMPQ_OK;
    if (!W || !act_idx || !W_act) return CMPQ_EINVAL;
    if (ldw < d_out || ld_act < d_out || k_act > 65535) return CMPQ_ESHAPE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int64_t gx = cdiv(d_out, kThreads);
    if (gx > 64) gx = 64;
    const dim3 grid((unsigned)gx, (unsigned)k_act);
    if (dtype == CMPQ_F16)
        gather_channels_kernel<__half><<<grid, kThreads, 0, s>>>(static_cast<const __half *>(W), d_out, ldw, act_idx, W_act, ld_act);
    else
        gather_channels_kernel<float><<<grid, kThreads, 0, s>>>(static_cast<const float *>(W), d_out, ldw, act_idx, W_act, ld_act);
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

extern "C" int cmpq_outliers_by_column(const int32_t *out_idx, const uint16_t *out_val, int64_t n_out,
                                       int64_t d_in, int64_t d_out, const float *centroids,
                                       const uint8_t *codes, int32_t *colptr, int32_t *row_idx,
                                       float *delta, void *ws, size_t ws_bytes, void *stream) {
    if (n_out < 0 || d_in < 0 || d_out < 0 || !colptr) return CMPQ_EINVAL;
    if (n_out > 0 && (!out_idx || !out_val || !centroids || !codes || !row_idx || !delta)) return CMPQ_EINVAL;
    if (d_out >= (1 << 20)) return CMPQ_ESHAPE;
    if (d_in > 0 && d_out > ((int64_t)1 << 31) / d_in) return CMPQ_ESHAPE;
    if (n_out > d_in * d_out) return CMPQ_ECOUNT;
    if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 != 0 || ws_bytes < cmpq_ws_outliers_by_column(d_out, n_out))
        return CMPQ_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int32_t *cnt = static_cast<int32_t *>(ws);
    const size_t col_bytes = align_up((size_t)(d_out + 1) * sizeof(int32_t), 256);
    int32_t *cursor = reinterpret_cast<int32_t *>(static_cast<char *>(ws) + col_bytes);
    int32_t *tmp_row = reinterpret_cast<int32_t *>(static_cast<char *>(ws) + 2 * col_bytes);
    float *tmp_delta = reinterpret_cast<float *>(static_cast<char *>(ws) + 2 * col_bytes + align_up((size_t)n_out * 4, 256));
    obc_zero_kernel<<<64, 256, 0, s>>>(cnt, d_out + 1);
    if (n_out > 0) {
        int64_t g = cdiv(n_out, 256);
        if (g > 2048) g = 2048;
        obc_count_kernel<<<(unsigned)g, 256, 0, s>>>(out_idx, n_out, d_out, cnt);
    }
    obc_scan_kernel<<<1, 1024, 0, s>>>(cnt, d_out, colptr, cursor);
    if (n_out > 0 && d_out > 0) {
        int64_t g = cdiv(n_out, 256);
        if (g > 2048) g = 2048;
        obc_scatter_kernel<<<(unsigned)g, 256, 0, s>>>(out_idx, out_val, n_out, d_out, centroids, codes, cursor, tmp_row, tmp_delta);
        obc_order_kernel<<<(unsigned)cdiv(d_out, kWaves), kThreads, 0, s>>>(colptr, d_out, tmp_row, tmp_delta, row_idx, delta);
    }
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

namespace {

// Host-side checks of one layer of a product (the rules of cmpq_lut_matvec).
int check_layer(const cmpq_deployed_layer &L, int64_t m) {
    if (L.d_in < 0 || L.d_out < 0 || L.k_act < 0 || L.n_set < 0 || L.n_set > kMaxWidths) return CMPQ_EINVAL;
    if (L.n_set > 0 && (!L.bit_set || !L.counts_host || !L.packed || !L.chan_idx || !L.lut)) return CMPQ_EINVAL;
    int64_t rows_total = L.k_act;
    for (int j = 0; j < L.n_set; ++j) {
        if (L.bit_set[j] < 1 || L.bit_set[j] > 4 || L.counts_host[j] < 0) return CMPQ_EINVAL;
        if (L.counts_host[j] > 0 && (!L.packed[j] || !L.chan_idx[j] || !L.lut[j])) return CMPQ_EINVAL;
        rows_total += L.counts_host[j];
    }
    if (rows_total > L.d_in) return CMPQ_EINVAL;
    if (m == 0 || L.d_out == 0) return CMPQ_OK;
    if (!L.Y || (L.d_in > 0 && !L.X)) return CMPQ_EINVAL;
    if (L.k_act > 0 && (!L.act_idx || !L.W_act)) return CMPQ_EINVAL;
    if (L.colptr && (!L.row_idx || !L.delta)) return CMPQ_EINVAL;
    if (L.ldx < L.d_in || L.ldy < L.d_out || (L.k_act > 0 && L.ld_act < L.d_out)) return CMPQ_ESHAPE;
    if (L.d_out >= (1 << 20)) return CMPQ_ESHAPE;
    return CMPQ_OK;
}

// The token-by-token launch of the layers order[0..n), `tokens` of the call's m at a time: arguments
// of its two kernels, grid and scratch.
struct Plan {
    LmGroup g;    // FP16 sums
    MvGroup mv;   // fp32 sums
    FinGroup f;
    size_t ws_used;
    int64_t y_total, x_total, max_tiles, wgs;
};

// Parts of a layer for fp32 sums: up to 512 workgroups in all, two per compute unit, of 8 rows a
// wavefront or more; larger layers in more, of 32 rows at width 4 (40 at 3, 48 at 2; with fewer the partial rows would need
// more scratch than calls had to bring before).  A width's rows
// count by what one costs (vector instructions a weight, see lut_part).  Kernel times of an earlier build,
// us: query, key and value of 8192 channels in 978 workgroups 20.6, in 1370 24.9; 8192 outputs of 28672
// channels in 496 39.8, in 740 34.6, in 976 32.5; twice 28672 of 8192 in 1008 56.1, in 1484 62.3, in 1960 57.5.
// (Bounds checks taken out of the loops, now: 17.5 in 978, 33.3 in 820, 53.1 in 1652.)
constexpr int64_t kMostCost = 160;
int part_rows(int bits, int64_t cost) {
    static const int kCost[5] = {0, 3, 3, 4, 5};
    const int group = bits <= 2 ? kPartGroup<1> : kPartGroup<4>;
    int64_t n = cost / kCost[bits] / group * group;
    return (int)(n < 8 ? 8 : (n > kMaxPartRows ? kMaxPartRows : n));
}
void choose_parts(MvLayer &a, int64_t tiles, int64_t tokens) {
    int64_t want = 512 / (tiles * tokens) * kWaves, act = 0, cost = 0;
    for (int j = 0; j < a.n_w; ++j) {
        if (a.w[j].bits == kActBits) act = cdiv(a.w[j].rows, (int64_t)kActRowsPerWave);
        else cost += (int64_t)a.w[j].rows * (a.w[j].bits + 1);  // no more than what the parts will cost
    }
    want = want > act + kWaves ? want - act : kWaves;
    cost /= want;
    cost = cost < 16 ? 16 : (cost > kMostCost ? kMostCost : cost);
    for (;; cost += 4) {
        int64_t parts = 0;
        for (int j = 0; j < a.n_w; ++j)
            if (a.w[j].bits != kActBits) parts += cdiv(a.w[j].rows, (int64_t)part_rows(a.w[j].bits, cost));
        if (parts <= want || cost >= kMostCost) break;
    }
    int part = 0;
    for (int j = 0; j < a.n_w; ++j) {
        MvWidth &w = a.w[j];
        w.part0 = part;
        w.parts = (int)cdiv(w.rows, (int64_t)(w.bits == kActBits ? kActRowsPerWave : part_rows(w.bits, cost)));
        part += w.parts;
    }
    a.slabs = (int)cdiv((int64_t)part, (int64_t)kWaves);
}

void plan_token_by_token(const cmpq_deployed_layer *layers, const int *order, int n, int64_t m, int64_t tokens, void *ws,
                         Plan &p, bool half_sums) {
    LmGroup &g = p.g;
    FinGroup &f = p.f;
    g.n_layers = f.n_layers = n;
    p.ws_used = 0;
    p.y_total = p.x_total = p.max_tiles = p.wgs = 0;
    for (int s = 0; s < kMaxLayers; ++s) p.mv.wg0[s] = INT_MAX;
    for (int s = 0; s < n; ++s) {
        const cmpq_deployed_layer &L = layers[order[s]];
        LmArgs &a = g.l[s];
        // rows per wavefront: the largest of 32, 16, 8 that still gives two workgroups per compute unit
        const int64_t tiles = cdiv(L.d_out, kTileOut);
        int rpw = kMaxRowsPerWave;
        while (rpw > 8 && tiles * total_slabs(L.counts_host, L.n_set, rpw) * m < 512) rpw /= 2;
        const int64_t n_lut = total_slabs(L.counts_host, L.n_set, rpw);
        const int64_t n_act = cdiv(L.k_act, (int64_t)kWaves * kActRowsPerWave);
        const int64_t n_rows = n_lut + n_act;
        a.n_widths = 0;
        a.rows_per_wave = rpw;
        a.n_lut_slabs = (int)n_lut;
        a.n_act_slabs = (int)n_act;
        a.n_rows_total = (int)n_rows;
        a.tiles = (int)tiles;
        a.y0 = (int)p.y_total;
        a.X = static_cast<const __half *>(L.X);
        a.ldx = L.ldx;
        a.d_out = L.d_out;
        a.partial = reinterpret_cast<float *>(static_cast<char *>(ws) + p.ws_used);
        a.act_idx = L.act_idx;
        a.W_act = reinterpret_cast<const __half *>(L.W_act);
        a.k_act = L.k_act;
        a.ld_act = L.ld_act;
        int slab0 = 0;
        for (int j = 0; j < L.n_set; ++j) {
            if (L.counts_host[j] == 0) continue;
            LmWidth &wd = a.w[a.n_widths++];
            wd.packed = L.packed[j];
            wd.chan_idx = L.chan_idx[j];
            wd.lut = L.lut[j];
            wd.rows = L.counts_host[j];
            wd.words_per_row = cdiv(L.d_out * L.bit_set[j], 32);
            wd.slab0 = slab0;
            wd.bits = L.bit_set[j];
            slab0 += (int)cdiv(wd.rows, (int64_t)kWaves * rpw);
        }
        for (int j = a.n_widths; j < kMaxWidths; ++j) a.w[j] = LmWidth{nullptr, nullptr, nullptr, 0, 0, 0, 0};
        FinArgs &fa = f.l[s];
        fa.X = a.X;
        fa.ldx = L.ldx;
        fa.d_out = L.d_out;
        fa.partial = a.partial;
        fa.colptr = L.colptr;
        fa.row_idx = L.row_idx;
        fa.delta = L.delta;
        fa.Y = L.Y;
        fa.ldy = L.ldy;
        fa.n_rows_total = (int)n_rows;
        if (!half_sums) {
            // (fewer parts than what the scratch is reserved for, which a caller may count on)
            MvLayer &v = p.mv.l[s];
            v.n_w = 0;
            for (int j = 0; j < a.n_widths; ++j)
                v.w[v.n_w++] = MvWidth{a.w[j].packed, a.w[j].chan_idx, a.w[j].lut, (int)a.w[j].rows, (int)a.w[j].words_per_row, a.w[j].bits, 0, 0};
            if (L.k_act > 0) v.w[v.n_w++] = MvWidth{nullptr, L.act_idx, nullptr, (int)L.k_act, 0, kActBits, 0, 0};
            for (int j = v.n_w; j <= kMaxWidths; ++j) v.w[j] = MvWidth{};
            v.X = a.X;
            v.W_act = a.W_act;
            v.ldx = L.ldx;
            v.ld_act = L.ld_act;
            v.partial = a.partial;
            v.d_out = (int)L.d_out;
            choose_parts(v, tiles, m);
            fa.n_rows_total = v.slabs;
            p.mv.wg0[s] = (int)p.wgs;
            p.wgs += tiles * v.slabs;
        }
        fa.x0 = (int)p.x_total;
        p.ws_used += align_up((size_t)tokens * (size_t)n_rows * (size_t)L.d_out * sizeof(float), 256);
        p.y_total += n_rows;
        p.x_total += cdiv(L.d_out, kFinCols);
        if (tiles > p.max_tiles) p.max_tiles = tiles;
    }
    for (int s = n; s < kMaxLayers; ++s) {
        g.l[s] = g.l[0];
        f.l[s] = f.l[0];
        p.mv.l[s] = p.mv.l[0];
    }
}

int launch_token_by_token(const Plan &p, int64_t tokens, bool half_sums, hipStream_t st) {
    if (half_sums && p.y_total > 0)
        lut_matvec_half_kernel<<<dim3((unsigned)p.max_tiles, (unsigned)p.y_total, (unsigned)tokens), kThreads, 0, st>>>(p.g);
    if (!half_sums && p.wgs > 0) lut_matvec_kernel<<<dim3((unsigned)p.wgs, (unsigned)tokens), kThreads, 0, st>>>(p.mv);
    const dim3 fgrid((unsigned)p.x_total, (unsigned)tokens);
    lut_matvec_finish_kernel<<<fgrid, kThreads, 0, st>>>(p.f);
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

int launch_group(const cmpq_deployed_layer *layers, int n_layers, int64_t m, void *ws, size_t ws_bytes,
                 void *stream, bool half_sums = false) {
    if (n_layers < 0 || n_layers > kMaxLayers || m < 0 || (n_layers > 0 && !layers)) return CMPQ_EINVAL;
    for (int i = 0; i < n_layers; ++i) {
        const int rc = check_layer(layers[i], m);
        if (rc != CMPQ_OK) return rc;
    }
    if (m > 65535) return CMPQ_ESHAPE;
    if (m == 0) return CMPQ_OK;
    // the longest products first: their workgroups are dispatched first
    int order[kMaxLayers], n_live = 0;
    for (int i = 0; i < n_layers; ++i)
        if (layers[i].d_out > 0) order[n_live++] = i;
    for (int i = 1; i < n_live; ++i)
        for (int j = i; j > 0; --j) {
            const cmpq_deployed_layer &p = layers[order[j - 1]], &q = layers[order[j]];
            if (p.d_in * p.d_out >= q.d_in * q.d_out) break;
            const int t = order[j];
            order[j] = order[j - 1];
            order[j - 1] = t;
        }
    if (n_live == 0) return CMPQ_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t have = ws && reinterpret_cast<uintptr_t>(ws) % 256 == 0 ? ws_bytes : 0;
    Plan p;
    plan_token_by_token(layers, order, n_live, m, m, ws, p, half_sums);
    if (p.y_total > 65535 || p.x_total > 0x7fffffff) return CMPQ_ESHAPE;
    if (half_sums) {
        // as many tokens at a time as the workspace holds, the same numbers however many
        int64_t tokens = m;
        if (p.ws_used > have) {
            plan_token_by_token(layers, order, n_live, m, 1, ws, p, true);
            if (p.ws_used > have) return CMPQ_EWORKSPACE;
            // (a token's rows fill whole 256 bytes at most once over; parts of even size)
            tokens = cdiv(m, cdiv(m, (int64_t)(have / p.ws_used)));
            plan_token_by_token(layers, order, n_live, m, tokens, ws, p, true);
        }
        for (int64_t t = 0; t < m; t += tokens) {
            const int rc = launch_token_by_token(p, m - t < tokens ? m - t : tokens, true, st);
            if (rc != CMPQ_OK) return rc;
            for (int i = 0; i < n_live; ++i) {
                p.g.l[i].X += tokens * p.g.l[i].ldx;
                p.f.l[i].X += tokens * p.f.l[i].ldx;
                p.f.l[i].Y += tokens * p.f.l[i].ldy;
            }
        }
        return CMPQ_OK;
    }
    // Layers that the matrix cores take (several tokens) go first, the others token by token.  A
    // workspace is enough if it holds either launch, or the token-by-token launch of all layers (which
    // is what calls had to bring before there were others): a layer whose plan does not fit into the
    // workspace goes token by token then, whatever else is in the group.
    size_t need[kMaxLayers], sum = 0;
    bool fits[kMaxLayers];
    int rest[kMaxLayers], n_rest = 0;
    for (int i = 0; i < n_live; ++i) {
        const cmpq_deployed_layer &L = layers[order[i]];
        fits[i] = m > 1 && lut_gemm_takes(L.d_in, L.d_out, m);
        need[i] = fits[i] ? lut_gemm_need(L, m) : 0;
        sum += need[i];
        if (!fits[i]) rest[n_rest++] = order[i];
    }
    if (n_rest == n_live) return p.ws_used > have ? CMPQ_EWORKSPACE : launch_token_by_token(p, m, false, st);
    if (p.ws_used > have) {
        if (sum > have) return CMPQ_EWORKSPACE;
        if (n_rest > 0) plan_token_by_token(layers, rest, n_rest, m, m, ws, p, false);
        if (n_rest > 0 && p.ws_used > have) return CMPQ_EWORKSPACE;
    }
    const cmpq_deployed_layer *batch[kMaxLayers];
    int n_batch = 0;
    n_rest = 0;
    char *at = static_cast<char *>(ws);
    size_t used = 0;
    for (int i = 0; i <= n_live; ++i) {
        if (i < n_live && !(fits[i] && need[i] <= have)) {
            rest[n_rest++] = order[i];
            continue;
        }
        if (n_batch > 0 && (i == n_live || used + need[i] > have)) {  // (launches on one stream run in order)
            const int rc = launch_lut_gemm(batch, n_batch, m, at, st);
            if (rc != CMPQ_OK) return rc;
            n_batch = 0;
            used = 0;
        }
        if (i < n_live) {
            batch[n_batch++] = &layers[order[i]];
            used += need[i];
        }
    }
    if (n_rest == 0) return CMPQ_OK;
    plan_token_by_token(layers, rest, n_rest, m, m, ws, p, false);
    return launch_token_by_token(p, m, false, st);
}

}  // namespace

extern "C" int cmpq_lut_matvec_group(const cmpq_deployed_layer *layers, int n_layers, int64_t m, void *ws,
                                     size_t ws_bytes, void *stream) {
    return launch_group(layers, n_layers, m, ws, ws_bytes, stream);
}

extern "C" int cmpq_lut_matvec_group_fp16acc(const cmpq_deployed_layer *layers, int n_layers, int64_t m, void *ws,
                                             size_t ws_bytes, void *stream) {
    return launch_group(layers, n_layers, m, ws, ws_bytes, stream, true);
}

extern "C" int cmpq_lut_matvec(const void *X, int64_t m, int64_t d_in, int64_t ldx, int64_t d_out,
                               const int32_t *bit_set, int n_set, const int64_t *counts_host,
                               const uint32_t *const *packed, const int32_t *const *chan_idx,
                               const uint16_t *const *lut, const int32_t *act_idx,
                               const uint16_t *W_act, int64_t k_act, int64_t ld_act,
                               const int32_t *colptr, const int32_t *row_idx, const float *delta,
                               float *Y, int64_t ldy, void *ws, size_t ws_bytes, void *stream) {
    cmpq_deployed_layer L;
    L.X = X;
    L.d_in = d_in;
    L.ldx = ldx;
    L.d_out = d_out;
    L.bit_set = bit_set;
    L.n_set = n_set;
    L.counts_host = counts_host;
    L.packed = packed;
    L.chan_idx = chan_idx;
    L.lut = lut;
    L.act_idx = act_idx;
    L.W_act = W_act;
    L.k_act = k_act;
    L.ld_act = ld_act;
    L.colptr = colptr;
    L.row_idx = row_idx;
    L.delta = delta;
    L.Y = Y;
    L.ldy = ldy;
    if (m < 0) return CMPQ_EINVAL;
    return launch_group(&L, 1, m, ws, ws_bytes, stream);
}

extern "C" int cmpq_lut_matvec_shape(const cmpq_deployed_layer *layer, int64_t m, int64_t *shape, int64_t *parts,
                                     int64_t room) {
    if (!layer || !shape || room < 0 || (room > 0 && !parts)) return CMPQ_EINVAL;
    // sizes alone: what check_layer asks of the pointers is not looked at
    static const uint32_t *const packed[kMaxWidths] = {};
    static const int32_t *const chan_idx[kMaxWidths] = {};
    static const uint16_t *const lut[kMaxWidths] = {};
    cmpq_deployed_layer L = {};
    L.d_in = L.ldx = layer->d_in;
    L.d_out = L.ldy = L.ld_act = layer->d_out;
    L.bit_set = layer->bit_set, L.n_set = layer->n_set, L.counts_host = layer->counts_host, L.k_act = layer->k_act;
    L.packed = packed, L.chan_idx = chan_idx, L.lut = lut;
    if (m < 1 || L.d_in < 1 || L.d_out < 1 || L.k_act < 0 || L.n_set < 0 || L.n_set > kMaxWidths) return CMPQ_EINVAL;
    if (L.n_set > 0 && (!L.bit_set || !L.counts_host)) return CMPQ_EINVAL;
    int64_t rows = L.k_act;
    for (int j = 0; j < L.n_set; ++j) {
        if (L.bit_set[j] < 1 || L.bit_set[j] > 4 || L.counts_host[j] < 0) return CMPQ_EINVAL;
        rows += L.counts_host[j];
    }
    if (rows > L.d_in) return CMPQ_EINVAL;
    const int order = 0;
    Plan p;
    plan_token_by_token(&L, &order, 1, m, m, nullptr, p, false);
    if (m > 65535 || L.d_out >= (1 << 20) || p.y_total > 65535) return CMPQ_ESHAPE;
    for (int i = 0; i < 6; ++i) shape[i] = 0;
    if (m > 1 && lut_gemm_takes(L.d_in, L.d_out, m)) {
        lut_gemm_shape(L, m, shape, parts, room);
        return CMPQ_OK;
    }
    const MvLayer &v = p.mv.l[0];
    shape[1] = m, shape[2] = v.slabs;
    for (int j = 0; j < v.n_w; ++j)
        for (int i = 0; i < v.w[j].parts; ++i) {
            int r0, n;
            rows_of_part(v.w[j], i, r0, n);
            const int64_t at = shape[3]++;
            if (at < room) parts[3 * at] = v.w[j].bits, parts[3 * at + 1] = r0, parts[3 * at + 2] = n;
        }
    return CMPQ_OK;
}
