// The product with the deployed weight for several tokens (Sec. 6 / Fig. 4 of arXiv 2410.13056):
// Y[t,o] = sum_i X[t,i] * W_hat[i,o] as a matrix product on the matrix cores, from the stored
// format.  FP16 levels and inputs multiply exactly, sums are fp32, as in the single-token kernel.
//
// Work is cut into steps of 32 rows of one width (or of O_act): the 32 rows are the depth of one
// v_mfma_f32_16x16x32_f16, and because the order of the rows is free, a lane may hold any 8 of
// them.  A wavefront takes 256 outputs: lane (i, kg) = (lane % 16, lane / 16) reads the codes of
// its 16 outputs 16 i .. 16 i + 15 in each of the rows 8 kg .. 8 kg + 7, and turns them into 16
// operands, one per output, of 8 rows each: operand e of the wavefront covers the outputs
// 16 i + e.  No code passes between lanes.
//
//   * order_tokens      X in operand order (rows as the steps take them), and channel by channel
//                       for the entries of O_q;
//   * few tokens: lut_tokens_kernel multiplies while it decodes - a weight is decoded once per
//     16 or 32 tokens and never stored - and leaves one partial result per slab of rows;
//     tokens_finish_kernel adds the slabs and the entries of O_q in a fixed order;
//   * many tokens: lut_decode_kernel writes W_hat once in operand order, override_kernel puts the
//     entries of O_q in, and weight_gemm_kernel multiplies.
// Every sum has a fixed order: results are reproducible bit for bit, and a layer's result does
// not depend on the other layers of a call (a workspace too small for a layer's plan aside, which
// sends that layer token by token).
//
// Measured against one token after the other (us per call): two 13824x5120 layers, 16 tokens 281 ->
// 41, 96 tokens -> 160; a 4096-wide attention and MLP group, 512 tokens 9183 -> 303, of which, under
// the profiler, the product 233 (618 TFLOP/s of the 1144 that a large library product reaches here),
// decoding with the inputs put in order beside it 75 (in launches of their own 65 + 26).  The error against 64 bits is
// 0.8e-7 to 1.4e-7, no larger than token by token.  What bounds the few-token kernel is its decoding: an LDS look-up a weight at 3
// and 4 bits (2.6 clocks of a compute unit each, measured; 4 of the 5 thousand clocks that a step of
// 32 rows takes 12 wavefronts) and 2.3 vector instructions; at 2 bits half of either.  Of its 26 us at
// 16 tokens (37 with a fourth instruction a weight, the parts split without regard to their cost
// and a second round of workgroups) the first 3 go by before the codes are there and the last 2 in
// adding up.  For small layers it is the launches and the first pass through the code, 53 to 65
// KB, two bodies for each width: steps that are there whole, which need no bounds, and others.
// Registers are all in use: the variants of up to 16 tokens keep 9 to 12 vector registers in
// memory outside the loops.
#include "lut_gemm.h"
#include <limits.h>

namespace {

typedef _Float16 Half8 __attribute__((ext_vector_type(8)));
typedef float Float4 __attribute__((ext_vector_type(4)));
typedef uint32_t Word4 __attribute__((ext_vector_type(4)));

constexpr int kRowsPerStep = 32;
constexpr int kOuts = 16;                    // outputs of a lane = operands of a wavefront per step
constexpr int kTileOuts = 16 * kOuts;        // outputs of a wavefront
constexpr int kThreads = 256, kWaves = kThreads / CMPQ_WAVE;
constexpr int kMaxSegs = 5;                  // four widths and O_act
constexpr int kActBits = 16;
constexpr int kTok = 16;                     // tokens of an operand

// Rows of one width (or of O_act, bits = 16).
struct Seg {
    const uint32_t *packed;
    const uint16_t *lut;
    const int32_t *chan;
    int rows, words_per_row, bits, step0;    // step0: first step among all steps of the layer
    int steps, part0, parts;                 // few tokens: the parts (one a wavefront) that share the steps
};

struct Layer {
    Seg seg[kMaxSegs];
    const __half *X, *W_act;
    int64_t ldx, ld_act;
    const int32_t *colptr, *row_idx;
    const float *delta;
    float *Y;
    int64_t ldy;
    uint4 *xf;          // [token tile][step][lane]: X in operand order
    __half *xt;         // [token tile][channel][16 tokens]
    int32_t *pos;       // [channel]: its row among all steps (many tokens)
    float *partial;     // [slab][token][d_out]
    uint4 *dense;       // [step][tile][operand][lane]: W_hat in operand order (many tokens)
    int d_in, d_out, n_seg, steps, tiles, slabs;  // slabs: kWaves parts each
    int span;           // steps of the fullest slab
};

constexpr int kMaxLayers = CMPQ_MAX_GROUP;
struct Group {
    int wg0[kMaxLayers];  // first workgroup of each layer in the launch (past the last layer: INT_MAX)
    int n_layers, m, token_tiles;
    Layer l[kMaxLayers];
};
static_assert(sizeof(Group) + 64 <= 4096, "travels in the kernel arguments");

// The layer that workgroup `wg` of the launch belongs to; `wg` becomes its number among that layer's.
__device__ __forceinline__ const Layer &layer_of(const Group &g, const int (&wg0)[kMaxLayers], int &wg) {
    int l = 0;
#pragma unroll
    for (int i = 1; i < kMaxLayers; ++i) l += wg >= wg0[i];
    wg -= wg0[l];
    return g.l[l];
}
__device__ __forceinline__ const Layer &layer_of(const Group &g, int &wg) {
    wg = (int)blockIdx.x;
    return layer_of(g, g.wg0, wg);
}

// Workgroups are dealt out to the 8 XCDs in turn.  This renumbering gives each XCD a contiguous
// range of work, so that neighbouring tiles, which share cache lines of the packed rows (or whole
// operands), meet in one L2.
__device__ __forceinline__ int xcd_order(int i, int n) {
    const int q = n >> 3, r = n & 7, x = i & 7;
    return x * q + min(x, r) + (i >> 3);
}

// ---- X as the product reads it

// Inputs of channel `chan` (-1: none) of the tokens t0 .. t0 + 15, zero past the last token.  What is not there is
// read from channel 0 or the last token and dropped: loads under a condition each waited for the one before
// (8000 channels, 16 tokens: 8.6 us for the launch, now 4.8).
__device__ __forceinline__ void load_tokens(const __half *__restrict__ X, int64_t ldx, int chan, int t0, int m, __half (&v)[kTok]) {
    const __half *x = X + max(chan, 0);
#pragma unroll
    for (int t = 0; t < kTok; ++t) v[t] = x[(int64_t)min(t0 + t, m - 1) * ldx];
#pragma unroll
    for (int t = 0; t < kTok; ++t) v[t] = chan >= 0 && t0 + t < m ? v[t] : __ushort_as_half(0);
}

// Workgroups of a layer: per token tile, blocks of 256 rows (8 steps) of the operand order, then
// blocks of 256 channels.
constexpr int kTokensLds = kTok * (kThreads + 8) * 2;
__device__ __forceinline__ void order_tokens(const Group &g, const Layer &L, int b, unsigned char *smem) {
    const int tid = threadIdx.x;
    const int row_blocks = (L.steps + 7) / 8, chan_blocks = L.xt ? (L.d_in + kThreads - 1) / kThreads : 0;
    const int tt = b / (row_blocks + chan_blocks);
    b -= tt * (row_blocks + chan_blocks);
    const int t0 = tt * kTok;
    if (b >= row_blocks) {
        const int c = (b - row_blocks) * kThreads + tid;
        if (c >= L.d_in) return;
        __half v[kTok];
        load_tokens(L.X, L.ldx, c, t0, g.m, v);
        uint4 *dst = reinterpret_cast<uint4 *>(L.xt + ((int64_t)tt * L.d_in + c) * kTok);
        dst[0] = reinterpret_cast<const uint4 *>(v)[0];
        dst[1] = reinterpret_cast<const uint4 *>(v)[1];
        return;
    }
    __half(*s)[kThreads + 8] = reinterpret_cast<__half(*)[kThreads + 8]>(smem);
    const int k = b * kThreads + tid, step = k / kRowsPerStep;
    int chan = -1;
    if (step < L.steps) {
#pragma unroll
        for (int j = 0; j < kMaxSegs; ++j) {  // segments that are not there have no rows
            const int row = k - L.seg[j].step0 * kRowsPerStep;
            if (row >= 0 && row < L.seg[j].rows) chan = L.seg[j].chan[row];
        }
    }
    if (L.pos && tt == 0 && chan >= 0) L.pos[chan] = k;
    __half v[kTok];
    load_tokens(L.X, L.ldx, chan, t0, g.m, v);
#pragma unroll
    for (int t = 0; t < kTok; ++t) s[t][tid] = v[t];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int unit = u * kThreads + tid, st = unit / CMPQ_WAVE, lane = unit % CMPQ_WAVE;
        if (b * 8 + st < L.steps)
            L.xf[((int64_t)tt * L.steps + b * 8 + st) * CMPQ_WAVE + lane] =
                *reinterpret_cast<const uint4 *>(&s[lane % 16][st * kRowsPerStep + (lane / 16) * 8]);
    }
}

__global__ __launch_bounds__(kThreads) void tokens_kernel(Group g) {
    __shared__ __align__(16) unsigned char smem[kTokensLds];
    int b;
    const Layer &L = layer_of(g, b);
    order_tokens(g, L, b, smem);
}

// What the decoding of a tile needs of its layer, copied out of the kernel arguments once.
struct TileArgs {
    uint4 *xf;
    const __half *X, *W_act;
    int64_t ldx;
    int64_t ld_act;
    float *partial;
    int steps, d_out;
};

// ---- decoding one step: 32 rows x 256 outputs -> 16 operands

// LDS of a wavefront: the level tables of a step's 32 rows, twice.  Widths 1 and 4:
// [row % 8][row / 8][16 levels]; width 2: pairs of rows, [row / 2 % 4][row / 8][16 pairs of codes],
// an entry the two rows' levels side by side, so that one look-up decodes two weights; width 3: the
// tables twice over, [row % 8][row / 8][8 levels] with a level every 2 bytes and
// [row / 2 % 4][8 levels][row / 8][row % 2] with one every 16, so that two neighbouring codes of a
// shifted word are both in place as the bits of an address (bits 1-3 and 4-6): three instructions
// for two weights instead of four.  The tables that a half-wavefront reads at once lie in different
// banks.
constexpr int kTableBytes = kRowsPerStep * 16 * 2;

// (v << 1) + base in one instruction.
__device__ __forceinline__ uint32_t shl1_add(uint32_t v, uint32_t base) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(r) : "v"(v), "v"(base));
    return r;
}

template <int B>
struct Decoder {
    static constexpr bool kAct = B == kActBits, kPairs = B == 2;
    static constexpr int kWords = kAct ? 4 : (B >= 3 ? 2 : 1);  // words fetched per row: 16 outputs (O_act: 8)
    static constexpr int kLevels = kAct ? 0 : 1 << B;
    static constexpr int kEntries = kLevels / 2;               // levels a lane fetches per step (not for pairs)
    static constexpr int kRaw = kPairs ? 4 : 8;                // look-ups per operand
    static constexpr int kTable3 = kTableBytes / 2;            // width 3: the tables with a level every 16 bytes
    uint32_t w[8][kWords];
    uint32_t e[4];

    // The words of this lane's outputs in its 8 rows of the step that starts at `row`, and its share
    // of the step's tables.  Rows past the end are read again from the last one; their tables are
    // zero, so they add nothing.
    // WHOLE (uniform): all 32 rows and all 256 outputs are there.
    template <bool WHOLE>
    __device__ __forceinline__ void fetch(const TileArgs &L, const Seg &s, int row, int out0, int half = 0) {
        const bool full = WHOLE || out0 + kTileOuts <= L.d_out;
        const int lane = threadIdx.x & 63, kg = lane >> 4;
        const int unit = (out0 >> 4) + (lane & 15);        // which 16 outputs of a row
        if constexpr (kAct) {
            const int o = unit * kOuts + half * 8;
            with_act_mode(L.d_out, full, [&](auto mode) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int r = row + 8 * kg + j;
                    const uint4 a = act_outputs8<decltype(mode)::value>(L.W_act + (int64_t)min(r, s.rows - 1) * L.ld_act, o, L.d_out);
                    const bool ok = r < s.rows;
                    w[j][0] = ok ? a.x : 0, w[j][1] = ok ? a.y : 0, w[j][2] = ok ? a.z : 0, w[j][3] = ok ? a.w : 0;
                }
            });
        } else {
            const int first = B == 4 ? 2 * unit : (B == 3 ? 3 * (unit >> 1) + (unit & 1) : (B == 2 ? unit : unit >> 1));
            const uint32_t wpr = (uint32_t)s.words_per_row;
            // a uniform base and a 32-bit offset per lane (the packed rows of a width stay below 2^30 bytes)
            const char *base = reinterpret_cast<const char *>(s.packed) + (uint64_t)row * wpr * 4u;
            typedef uint32_t WordsN __attribute__((ext_vector_type(kWords), aligned(4)));
            if (WHOLE || (full && row + kRowsPerStep <= s.rows)) {
                const uint32_t at = ((uint32_t)(8 * kg) * wpr + (uint32_t)first) * 4u;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const WordsN v = __builtin_nontemporal_load(reinterpret_cast<const WordsN *>(base + (uint64_t)(j * wpr) * 4u + at));
#pragma unroll
                    for (int q = 0; q < kWords; ++q) w[j][q] = v[q];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // past the end of a row its last word again: outputs that are not there are not written
                    const uint32_t r = (uint32_t)min(8 * kg + j, s.rows - 1 - row) * wpr;
#pragma unroll
                    for (int q = 0; q < kWords; ++q)
                        w[j][q] = *reinterpret_cast<const uint32_t *>(base + (uint64_t)((r + min((uint32_t)(first + q), wpr - 1u)) * 4u));
                }
            }
            const uint16_t *lut = s.lut + (int64_t)row * kLevels;
            const int left = WHOLE ? kRowsPerStep : s.rows - row;  // rows of the step
            if constexpr (kPairs) {
                // lane: rows 2 p, 2 p + 1 with p = lane / 4; the upper row's code lane % 4
                const int r0 = lane >> 2 << 1;
                const uint16_t *lo = lut + min(r0, left - 1) * kLevels;
                uint16_t t[kLevels], h = lut[min(r0 + 1, left - 1) * kLevels + (lane & 3)];
                __builtin_memcpy(t, lo, sizeof(t));
                const uint32_t hi = r0 + 1 < left ? (uint32_t)h << 16 : 0u;
#pragma unroll
                for (int q = 0; q < kLevels; ++q) e[q] = (r0 < left ? (uint32_t)t[q] : 0u) | hi;
            } else {
                // lane: row lane / 2, half lane % 2 of its table
                const int r = lane >> 1;
                uint16_t t[8];
                __builtin_memcpy(t, lut + min(r, left - 1) * kLevels + (lane & 1) * kEntries, kEntries * 2);
#pragma unroll
                for (int q = 0; q < (kEntries + 1) / 2; ++q)
                    e[q] = r < left ? (uint32_t)t[2 * q] | (kEntries > 1 ? (uint32_t)t[2 * q + 1] << 16 : 0u) : 0u;
            }
        }
    }

    // Puts this lane's share of the tables into the wavefront's table buffer, and moves the codes
    // of widths 1 and 3 to the start of their words (odd units start in the middle of one).
    __device__ __forceinline__ void settle(unsigned char *buf) {
        const int lane = threadIdx.x & 63;
        if constexpr (kPairs) {
            const int p = lane >> 2;
            *reinterpret_cast<uint4 *>(buf + (p & 3) * 256 + (p >> 2) * 64 + (lane & 3) * 16) = make_uint4(e[0], e[1], e[2], e[3]);
        } else if constexpr (!kAct) {
            const int row = lane >> 1;
            unsigned char *p = buf + ((row & 7) * 4 + (row >> 3)) * (B == 3 ? 16 : 32) + (lane & 1) * kEntries * 2;
            if constexpr (B == 4) *reinterpret_cast<uint4 *>(p) = make_uint4(e[0], e[1], e[2], e[3]);
            else if constexpr (B == 3) {
                *reinterpret_cast<uint2 *>(p) = make_uint2(e[0], e[1]);
                uint16_t *q = reinterpret_cast<uint16_t *>(buf + kTable3 + ((row >> 1) & 3) * 128 + (lane & 1) * 64 + (row >> 3) * 4 + (row & 1) * 2);
                q[0] = (uint16_t)e[0], q[8] = (uint16_t)(e[0] >> 16), q[16] = (uint16_t)e[1], q[24] = (uint16_t)(e[1] >> 16);
            }
            else *reinterpret_cast<uint16_t *>(p) = (uint16_t)e[0];
            const int shift = 16 * (lane & 1);  // out0 is a whole number of units of 16 outputs, an even one
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (B == 3) {
                    w[j][0] = __builtin_amdgcn_alignbit(w[j][1], w[j][0], shift);
                    w[j][1] >>= shift;
                }
                if constexpr (B == 1) w[j][0] >>= shift;
            }
        }
    }

    // LDS address of this lane's tables.
    static __device__ __forceinline__ uint32_t tables_at(const unsigned char *tables) {
        return (uint32_t)reinterpret_cast<uintptr_t>(tables) + ((threadIdx.x & 63) >> 4) * (kPairs ? 64 : (B == 3 ? 16 : 32));
    }

    // What operand k (output k of this lane in its 8 rows) is made of, and the operand.  Two parts,
    // so that the look-ups of the next operands can be under way while these are packed and multiplied.
    struct Raw {
        uint32_t v[kRaw];
    };
    __device__ __forceinline__ Raw look_up(int k, uint32_t at) const {
        Raw r;
#pragma unroll
        for (int j = 0; j < kRaw; ++j) {
            if constexpr (kAct) {
                r.v[j] = w[j][k >> 1];
            } else if constexpr (kPairs) {
                // nibbles of a pair of rows' codes (even outputs | odd outputs), times 4, a byte each
                const uint32_t a = w[2 * j][0], b = w[2 * j + 1][0];
                const uint32_t n = k & 1 ? ((a >> 2) & 0x33333333u) | (b & 0xccccccccu) : (a & 0x33333333u) | ((b << 2) & 0xccccccccu);
                const uint32_t t = (k & 2 ? n >> 2 : n << 2) & 0x3c3c3c3cu;
                r.v[j] = lds_read<uint32_t>(add_byte(at, t, k >> 2) + j * 256);
            } else if constexpr (B == 4) {
                // every other code, times 2, a byte each
                const uint32_t t = (k & 1 ? w[j][k >> 3] >> 3 : w[j][k >> 3] << 1) & 0x1e1e1e1eu;
                r.v[j] = lds_read<uint16_t>(add_byte(at, t, (k & 7) >> 1) + j * 128);
            } else if constexpr (B == 3) {
                // codes k (even) and k + 1 at bits 1-3 and 4-6 of the row's words, shifted
                const int sh = 3 * (k & ~1) - 1;
                const uint32_t u = sh < 0 ? w[j][0] << 1 : (sh < 32 ? __builtin_amdgcn_alignbit(w[j][1], w[j][0], sh) : w[j][1] >> (sh - 32));
                if (k & 1) {
                    const uint32_t at3 = at + kTable3 - ((threadIdx.x & 63) >> 4) * 12;  // bits 2-3: row / 8
                    r.v[j] = lds_read<uint16_t>(((u & 0x70u) | at3) + (j >> 1) * 128 + (j & 1) * 2);
                } else {
                    r.v[j] = lds_read<uint16_t>(((u & 0xeu) | at) + j * 64);
                }
            } else {
                r.v[j] = lds_read<uint16_t>(shl1_add(code(j, k), at) + j * 128);
            }
        }
        return r;
    }
    static __device__ __forceinline__ Half8 operand(const Raw &r, int k) {
        Word4 v;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            if constexpr (kPairs) v[d] = r.v[d];
            else if constexpr (kAct) v[d] = __builtin_amdgcn_perm(r.v[2 * d + 1], r.v[2 * d], k & 1 ? 0x07060302u : 0x05040100u);
            else v[d] = r.v[2 * d] | (r.v[2 * d + 1] << 16);
        }
        return __builtin_bit_cast(Half8, v);
    }

    __device__ __forceinline__ uint32_t code(int j, int k) const {
        const int bit = k * B, q = bit >> 5, sh = bit & 31;
        if (sh + B <= 32) return __builtin_amdgcn_ubfe(w[j][q], sh, B);
        return __builtin_amdgcn_alignbit(w[j][q + 1 < kWords ? q + 1 : q], w[j][q], sh) & ((1u << B) - 1u);
    }
};

// ---- few tokens: decode and multiply

__device__ __forceinline__ Float4 mfma(Half8 a, Half8 b, Float4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// ND > 0: a workgroup fetches the inputs of its slab's rows, of up to ND tokens, into LDS itself,
// [token][row], instead of reading operands that tokens_kernel made: a launch less, which is what
// counts for short products.
constexpr int kTablesBytes = kWaves * 2 * kTableBytes;
constexpr int kSlabLds = kWaves * (kOuts / 2) * 4 * CMPQ_WAVE * 4;   // 32 KB: tables and inputs, then sums
constexpr int direct_steps(int nd) { return ((kSlabLds - kTablesBytes) / (nd * 2) - 8) / kRowsPerStep; }  // most steps of a slab

// The steps of a part, and its segment.  A slab is kWaves parts, one a wavefront; a part is of one
// width, and at the end of the last slab there may be parts that are empty.
__host__ __device__ __forceinline__ int part_of(const Layer &L, int part, int &lo, int &hi) {
    int j = 0;
#pragma unroll
    for (int i = 1; i < kMaxSegs; ++i) j += i < L.n_seg && part >= L.seg[i].part0;
    const Seg &s = L.seg[j];
    const int p = part - s.part0 < s.parts ? part - s.part0 : s.parts, next = p < s.parts ? p + 1 : p;
    lo = s.step0 + share_of(s.steps, p, s.parts);
    hi = s.step0 + share_of(s.steps, next, s.parts);
    return j;
}

template <int B, int MT, int ND, bool WHOLE>
__device__ __forceinline__ void multiply_steps(const TileArgs &L, const Seg &s, int lo, int hi, int out0, int tt,
                                               unsigned char *tables, const __half *xs, int xs_step0, int xs_rows,
                                               Float4 (&acc)[MT][kOuts]) {
    using D = Decoder<B>;
    const int lane = threadIdx.x & 63;
    const uint32_t at0 = D::tables_at(tables);
    const uint4 *xf = L.xf + ((int64_t)tt * L.steps) * CMPQ_WAVE + lane;
    auto load_x = [&](int step, Word4 (&x)[MT]) {
        if constexpr (ND > 0) {
            const int token = lane & 15;
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const Word4 v = *reinterpret_cast<const Word4 *>(xs + ((t * kTok + token) & (ND - 1)) * (xs_rows + 8) +
                                                                 (step - xs_step0) * kRowsPerStep + (lane >> 4) * 8);
                x[t] = t * kTok + token < ND ? v : Word4{0u, 0u, 0u, 0u};
            }
        } else {
#pragma unroll
            for (int t = 0; t < MT; ++t) x[t] = *reinterpret_cast<const Word4 *>(xf + ((int64_t)t * L.steps + step) * CMPQ_WAVE);
        }
    };
    if constexpr (D::kAct) {  // few steps, many words: one at a time
#pragma unroll 1
        for (int step = lo; step < hi; ++step) {
            Word4 x[MT];
            load_x(step, x);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                D d;
                d.template fetch<false>(L, s, (step - s.step0) * kRowsPerStep, out0, h);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const Half8 a = D::operand(d.look_up(k, 0), k);
#pragma unroll
                    for (int t = 0; t < MT; ++t) acc[t][8 * h + k] = mfma(a, __builtin_bit_cast(Half8, x[t]), acc[t][8 * h + k]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return;
    }
    D cur, nxt;
    Word4 x[MT], xn[MT];
    cur.template fetch<WHOLE>(L, s, (lo - s.step0) * kRowsPerStep, out0);
    load_x(lo, x);
    cur.settle(tables);
    wave_fence();
    int buf = 0;
#pragma unroll 1
    for (int step = lo; step < hi; ++step) {
        // the last step fetches itself again, which nothing uses
        const int ahead = step + 1 < hi ? step + 1 : step;
        nxt.template fetch<WHOLE>(L, s, (ahead - s.step0) * kRowsPerStep, out0);
        load_x(ahead, xn);
        const uint32_t at = at0 + buf * kTableBytes;
        // Look-ups run one operand ahead of the products.  The fences keep the compiler from starting
        // all of them at once, for which the registers would not do; two ahead costs a wavefront per
        // SIMD and 10 %.
        typename D::Raw raw = cur.look_up(0, at), raw_n;
#pragma unroll
        for (int k = 0; k < kOuts; ++k) {
            if (k + 1 < kOuts) raw_n = cur.look_up(k + 1, at);
            __builtin_amdgcn_sched_barrier(0);
            const Half8 a = D::operand(raw, k);
#pragma unroll
            for (int t = 0; t < MT; ++t) acc[t][k] = mfma(a, __builtin_bit_cast(Half8, x[t]), acc[t][k]);
            __builtin_amdgcn_sched_barrier(0);
            raw = raw_n;
        }
        buf ^= 1;
        nxt.settle(tables + buf * kTableBytes);
        wave_fence();
        cur = nxt;
#pragma unroll
        for (int t = 0; t < MT; ++t) x[t] = xn[t];
    }
}

// One slab: 256 outputs x MT * 16 tokens x a share of the layer's steps, which 4 wavefronts split.  A
// wavefront's steps are of one width: with the widths one after the other in one wavefront, the sums
// would change registers between them.
template <int MT, int ND>
__device__ __forceinline__ void multiply_slab(const TileArgs &L, const Layer &layer, int slab, int tile, int tt, int m,
                                              unsigned char *smem) {
    const int lane = threadIdx.x & 63, wave = wave_index();
    const int out0 = tile * kTileOuts;
    Float4 acc[MT][kOuts];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int k = 0; k < kOuts; ++k) acc[t][k] = Float4{0.f, 0.f, 0.f, 0.f};
    int lo, hi;
    const Seg s = layer.seg[part_of(layer, slab * kWaves + wave, lo, hi)];
    __half *xs = reinterpret_cast<__half *>(smem + kTablesBytes);
    int first = 0, rows = 0;
    if constexpr (ND > 0) {
        int last, other;
        part_of(layer, slab * kWaves, first, other);
        part_of(layer, slab * kWaves + kWaves - 1, other, last);
        rows = (last - first) * kRowsPerStep;
        for (int r = threadIdx.x; r < rows; r += kThreads) {
            int chan = -1;
#pragma unroll
            for (int j = 0; j < kMaxSegs; ++j) {  // segments that are not there have no rows
                const int row = first * kRowsPerStep + r - layer.seg[j].step0 * kRowsPerStep;
                if (row >= 0 && row < layer.seg[j].rows) chan = layer.seg[j].chan[row];
            }
            __half v[ND];
#pragma unroll
            for (int t = 0; t < ND; ++t) v[t] = chan >= 0 && t < m ? L.X[(int64_t)t * L.ldx + chan] : __ushort_as_half(0);
#pragma unroll
            for (int t = 0; t < ND; ++t) xs[t * (rows + 8) + r] = v[t];
        }
        __syncthreads();
    }
    if (lo < hi) {
        unsigned char *tables = smem + wave * 2 * kTableBytes;
        if (s.bits == kActBits) {
            multiply_steps<kActBits, MT, ND, false>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
        } else if (out0 + kTileOuts <= L.d_out && (hi - s.step0) * kRowsPerStep <= s.rows) {
            if (s.bits == 1) multiply_steps<1, MT, ND, true>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else if (s.bits == 2) multiply_steps<2, MT, ND, true>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else if (s.bits == 3) multiply_steps<3, MT, ND, true>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else multiply_steps<4, MT, ND, true>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
        } else {
            if (s.bits == 1) multiply_steps<1, MT, ND, false>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else if (s.bits == 2) multiply_steps<2, MT, ND, false>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else if (s.bits == 3) multiply_steps<3, MT, ND, false>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
            else multiply_steps<4, MT, ND, false>(L, s, lo, hi, out0, tt, tables, xs, first, rows, acc);
        }
    }
    // The four wavefronts' sums, added in pairs.  Wavefront w takes the operands 4 w .. 4 w + 3, for a
    // lane four neighbouring outputs of one token in each of the 4 components; two of them at a time,
    // so that 32 KB do.
    Float4 *red = reinterpret_cast<Float4 *>(smem);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        Float4 y[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kOuts / 2; ++k)
                red[(wave * (kOuts / 2) + k) * CMPQ_WAVE + lane] = acc[t][4 * (k >> 1) + 2 * h + (k & 1)];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const Float4 *v = red + (2 * wave + k) * CMPQ_WAVE + lane;
                constexpr int kNext = (kOuts / 2) * CMPQ_WAVE;
                y[2 * h + k] = (v[0] + v[kNext]) + (v[2 * kNext] + v[3 * kNext]);
            }
        }
        const int token = (tt + t) * kTok + (lane & 15);
        if (token < m) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = out0 + kOuts * (4 * (lane >> 4) + r) + 4 * wave;
                float *dst = L.partial + ((int64_t)slab * m + token) * L.d_out + o;
                if (L.d_out % 4 == 0) {
                    if (o < L.d_out) *reinterpret_cast<float4 *>(dst) = make_float4(y[0][r], y[1][r], y[2][r], y[3][r]);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (o + k < L.d_out) dst[k] = y[k][r];
                }
            }
        }
    }
}

template <int MT, int ND>
__global__ __launch_bounds__(kThreads, MT == 1 ? 3 : 2) void lut_tokens_kernel(Group g) {
    __shared__ __align__(kTableBytes) unsigned char smem[kSlabLds];
    int wg;
    const Layer &L = layer_of(g, wg);
    wg = xcd_order(wg, L.tiles * L.slabs * (g.token_tiles / MT));
    // the slabs of a tile one after the other, so that every XCD and compute unit gets slabs of all
    // widths (two 13824x5120 layers, 16 tokens: with the tiles innermost those of the widest codes took
    // 25 us, the others 15)
    const int slab = wg % L.slabs, rest = wg / L.slabs, tile = rest % L.tiles, tt = (rest / L.tiles) * MT;
    const TileArgs a{L.xf, L.X, L.W_act, L.ldx, L.ld_act, L.partial, L.steps, L.d_out};
    multiply_slab<MT, ND>(a, L, slab, tile, tt, g.m, smem);
}

// Slabs and entries of O_q: 16 outputs x NT tokens per workgroup.  16 lanes per column take its
// entries l, l + 16, ... with all NT tokens of the entry's channel at once; per output and token the
// slabs are added in 64 bits, then the 16 lanes' sums in lane order.
constexpr int kFinCols = 16;
template <int NT, bool DIRECT>
__global__ __launch_bounds__(kThreads) void tokens_finish_kernel(Group g) {
    int wg;
    const Layer &L = layer_of(g, wg);
    // a column's sums: odd distances between lanes and between columns, so that neither the writes
    // (one lane per entry) nor the reads (one lane per output) meet in a bank
    constexpr int kLane = NT + 1, kCol = 16 * kLane + 1;
    __shared__ float sp[kFinCols * kCol];
    const int hi = threadIdx.x >> 4, lo = threadIdx.x & 15;
    const int col_blocks = (L.d_out + kFinCols - 1) / kFinCols;
    const int tt = wg / col_blocks, o0 = (wg - tt * col_blocks) * kFinCols;
    const int d_out = L.d_out, slabs = L.slabs, m = g.m;
    const int32_t *colptr = L.colptr;
    // the slabs of output o0 + lo, token hi: on their way while the entries of O_q are worked on
    const int token = tt * kTok + hi, o = o0 + lo;
    const bool mine = hi < NT && token < m && o < d_out;
    constexpr int kInFlight = 8;
    const float *p = L.partial + (int64_t)token * d_out + o;
    float v[kInFlight];
#pragma unroll
    for (int q = 0; q < kInFlight; ++q) v[q] = mine && q < slabs ? p[(int64_t)q * m * d_out] : 0.f;
    if (colptr) {
        float t[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) t[u] = 0.f;
        if (o0 + hi < d_out) {
            const int e1 = colptr[o0 + hi + 1];
            const __half *xt = L.xt + (int64_t)tt * L.d_in * kTok, *X = L.X;
            const int64_t ldx = L.ldx;
            const int32_t *row_idx = L.row_idx;
            const float *delta = L.delta;
            constexpr int U = NT > 4 ? 4 : 8;  // entries in flight
            for (int e = colptr[o0 + hi] + lo; e < e1; e += 16 * U) {
                int r[U];
                float d[U];
                uint4 x[U][(NT + 7) / 8];
                __half xd[U][NT];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ok = e + 16 * u < e1;
                    r[u] = ok ? row_idx[e + 16 * u] : -1;
                    d[u] = ok ? delta[e + 16 * u] : 0.f;
                }
                if constexpr (DIRECT) {  // straight from X
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int w = 0; w < NT; ++w) xd[u][w] = r[u] >= 0 && tt * kTok + w < m ? X[(int64_t)(tt * kTok + w) * ldx + r[u]] : __ushort_as_half(0);
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int w = 0; w < NT; ++w) t[w] = fmaf(__half2float(xd[u][w]), d[u], t[w]);
                    continue;
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int q = 0; q < (NT + 7) / 8; ++q)
                        x[u][q] = r[u] >= 0 ? reinterpret_cast<const uint4 *>(xt + (int64_t)r[u] * kTok)[q] : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const __half *h = reinterpret_cast<const __half *>(x[u]);
#pragma unroll
                    for (int w = 0; w < NT; ++w) t[w] = fmaf(__half2float(h[w]), d[u], t[w]);
                }
            }
        }
#pragma unroll
        for (int w = 0; w < NT; ++w) sp[hi * kCol + lo * kLane + w] = t[w];
        __syncthreads();
    }
    if (!mine) return;
    // (in 64 bits: what the longer runs of width 2 lose this gains back.  Widened no earlier than here, or the
    // entries of O_q would wait for the slabs)
    auto sum = [&] {
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) asm volatile("" : "+v"(v[q]));
        return (((double)v[0] + v[1]) + ((double)v[2] + v[3])) + (((double)v[4] + v[5]) + ((double)v[6] + v[7]));
    };
    static_assert(kInFlight == 8, "");
    double y = sum();
    for (int s = kInFlight; s < slabs; s += kInFlight) {
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) v[q] = s + q < slabs ? p[(int64_t)(s + q) * m * d_out] : 0.f;
        y += sum();
    }
    if (colptr) {
        float z = 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) z += sp[lo * kCol + u * kLane + hi];
        y += z;
    }
    L.Y[(int64_t)token * L.ldy + o] = (float)y;
}

// ---- many tokens: decode once, then multiply

template <int B>
__device__ __forceinline__ void decode_step(const TileArgs &L, const Seg &s, Word4 *dense, int step, int out0, unsigned char *tables) {
    const int lane = threadIdx.x & 63;
    Word4 *dst = dense + lane;
    const uint32_t at = Decoder<B>::tables_at(tables);
    constexpr int kHalves = B == kActBits ? 2 : 1, kOps = kOuts / kHalves;
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
        Decoder<B> d;
        d.template fetch<false>(L, s, (step - s.step0) * kRowsPerStep, out0, h);
        d.settle(tables);
        wave_fence();
#pragma unroll
        for (int k = 0; k < kOps; ++k) dst[(h * kOps + k) * CMPQ_WAVE] = __builtin_bit_cast(Word4, Decoder<B>::operand(d.look_up(k, at), k));
    }
}

// X in operand order (the first workgroups) and W_hat in operand order, a wavefront for one step of one
// tile: neither needs the other, and as launches of their own the inputs took 13 us beside the 41 of
// the decoding (a 4096-wide group of two MLP layers, 512 tokens).
struct DecodeWgs {
    int wg0[kMaxLayers];  // first workgroup of each layer among those that decode
    int first;            //   and the first of those in the launch
};
// (Held to 6 wavefronts a SIMD, 79 registers: the rows of O_act alone would have it take 101.)
__global__ __launch_bounds__(kThreads, 6) void lut_decode_kernel(Group g, DecodeWgs d) {
    __shared__ __align__(kTableBytes) unsigned char smem[kTokensLds > kWaves * kTableBytes ? kTokensLds : kWaves * kTableBytes];
    int wg = (int)blockIdx.x;
    if (wg < d.first) {
        const Layer &L = layer_of(g, g.wg0, wg);
        order_tokens(g, L, wg, smem);
        return;
    }
    wg -= d.first;
    const Layer &L = layer_of(g, d.wg0, wg);
    const int wave = wave_index();
    const int unit = wg * kWaves + wave, tiles = L.tiles;
    const int step = unit / tiles, tile = unit - step * tiles;
    if (step >= L.steps) return;
    unsigned char *tables = smem + wave * kTableBytes;
    int j = 0;
#pragma unroll
    for (int i = 1; i < kMaxSegs; ++i) j += i < L.n_seg && step >= L.seg[i].step0;
    const Seg s = L.seg[j];
    const TileArgs a{L.xf, L.X, L.W_act, L.ldx, L.ld_act, L.partial, L.steps, L.d_out};
    Word4 *dense = reinterpret_cast<Word4 *>(L.dense) + (int64_t)unit * kOuts * CMPQ_WAVE;
    switch (s.bits) {
        case 1: decode_step<1>(a, s, dense, step, tile * kTileOuts, tables); break;
        case 2: decode_step<2>(a, s, dense, step, tile * kTileOuts, tables); break;
        case 3: decode_step<3>(a, s, dense, step, tile * kTileOuts, tables); break;
        case 4: decode_step<4>(a, s, dense, step, tile * kTileOuts, tables); break;
        default: decode_step<kActBits>(a, s, dense, step, tile * kTileOuts, tables); break;
    }
}

// Entries of O_q override their level: W_hat = FP16(level + delta), which is the FP16 weight.
// A wavefront per column.
__global__ __launch_bounds__(kThreads) void override_kernel(Group g) {
    int wg;
    const Layer &L = layer_of(g, wg);
    const int lane = threadIdx.x & 63;
    const int o = wg * kWaves + wave_index();
    if (!L.colptr || o >= L.d_out) return;
    const int in = o % kTileOuts, tile = o / kTileOuts, tiles = L.tiles;
    const uint32_t depth = (uint32_t)L.steps * kRowsPerStep;
    const int32_t *row_idx = L.row_idx, *pos = L.pos;
    const float *delta = L.delta;
    __half *dense = reinterpret_cast<__half *>(L.dense);
    for (int e = L.colptr[o] + lane, e1 = L.colptr[o + 1]; e < e1; e += CMPQ_WAVE) {
        const uint32_t k = (uint32_t)pos[row_idx[e]];
        if (k >= depth) continue;
        const int row = (int)(k % kRowsPerStep), ln = (row / 8) * 16 + in / kOuts;
        const int64_t at = ((((int64_t)(k / kRowsPerStep) * tiles + tile) * kOuts + in % kOuts) * CMPQ_WAVE + ln) * 8 + row % 8;
        dense[at] = __float2half_rn(__half2float(dense[at]) + delta[e]);
    }
}

// A workgroup: 128 outputs (operands 8 h .. 8 h + 7 of a tile) x 128 tokens.  Each of the 4
// wavefronts 4 operands x 4 token tiles.  Operands reach LDS by direct loads in the order in which
// they are read: 1 KB per operand, lane by lane, no conflicts.  A step's 16 operands are one
// buffer; kBuffers - 1 steps are on their way while one is multiplied.
constexpr int kGemmOps = 8;                           // operands of W and of X per step
constexpr int kBufBytes = 2 * kGemmOps * 1024, kBuffers = 4;
constexpr int kRun = 4;                               // steps whose sums are kept apart

__device__ __forceinline__ void load_lds16(const uint4 *src, unsigned char *dst) {
    __builtin_amdgcn_global_load_lds(reinterpret_cast<const __attribute__((address_space(1))) uint32_t *>(reinterpret_cast<uintptr_t>(src)),
                                     reinterpret_cast<__attribute__((address_space(3))) uint32_t *>((uint32_t)reinterpret_cast<uintptr_t>(dst)), 16, 0, 0);
}

__global__ __launch_bounds__(kThreads, 2) void weight_gemm_kernel(Group g) {
    __shared__ __align__(16) unsigned char smem[kBuffers * kBufBytes];
    int wg;
    const Layer &L = layer_of(g, wg);
    const int lane = threadIdx.x & 63, wave = wave_index();
    const int token_blocks = (g.token_tiles + kGemmOps - 1) / kGemmOps;
    const int steps = L.steps, tiles = L.tiles, d_out = L.d_out, m = g.m;
    float *Y = L.Y;
    const int64_t ldy = L.ldy;
    wg = xcd_order(wg, 2 * tiles * token_blocks);
    const int tb = wg % token_blocks, half = wg / token_blocks;
    const int tile = half >> 1, op0 = (half & 1) * kGemmOps, tt0 = tb * kGemmOps;
    // wavefront w brings operands 4 (w % 2) .. + 3 of W (w < 2) or of X
    const bool weights = wave < 2;
    const uint4 *src[4];
    unsigned char *dst = smem + wave * 4096;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = 4 * (wave & 1) + q;
        src[q] = (weights ? L.dense + ((int64_t)tile * kOuts + op0 + k) * CMPQ_WAVE
                          : L.xf + (int64_t)min(tt0 + k, g.token_tiles - 1) * steps * CMPQ_WAVE) + lane;
    }
    const int64_t stride = weights ? (int64_t)tiles * kOuts * CMPQ_WAVE : CMPQ_WAVE;
    auto load = [&](int step, int buf) {  // past the last step: that one again, which nothing reads
        const int64_t at = (int64_t)min(step, steps - 1) * stride;
#pragma unroll
        for (int q = 0; q < 4; ++q) load_lds16(src[q] + at, dst + buf * kBufBytes + q * 1024);
    };
    const int wn = (wave & 1) * 4, wt = (wave >> 1) * 4;  // this wavefront's operands of W and token tiles
    // The matrix cores add one step after the other into fp32; over a whole depth of thousands of
    // rows that loses more than the short runs of the other kernels (4.5e-7 against 1.4e-7 relative
    // at 4096 rows), so runs of kRun steps are added up apart, and kRun of those again.
    Float4 acc[4][4], sum[4][4], total[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = sum[a][b] = total[a][b] = Float4{0.f, 0.f, 0.f, 0.f};
    auto add_up = [](Float4 (&from)[4][4], Float4 (&to)[4][4]) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                to[p][q] += from[p][q];
                from[p][q] = Float4{0.f, 0.f, 0.f, 0.f};
            }
    };
#pragma unroll
    for (int u = 0; u < kBuffers - 1; ++u) load(u, u);
    for (int step = 0; step < steps; ++step) {
        // The oldest step's 4 loads of this wavefront have landed (two later steps, 8 loads, are under
        // way; any other load between them would only make the wait longer) and its LDS reads of the
        // step before have returned.  After the barrier both hold for every wavefront: this step's
        // buffer is full, and the one read a step ago, which is loaded next, is free.
        static_assert(kBuffers == 4, "the count of loads still under way");
        asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        load(step + kBuffers - 1, (step + kBuffers - 1) % kBuffers);
        const unsigned char *buf = smem + (step % kBuffers) * kBufBytes + lane * 16;
        Half8 a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = *reinterpret_cast<const Half8 *>(buf + (wn + q) * 1024);
            b[q] = *reinterpret_cast<const Half8 *>(buf + (kGemmOps + wt + q) * 1024);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[p][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[p], b[q], acc[p][q], 0, 0, 0);
        if (step % kRun == kRun - 1 || step == steps - 1) {
            add_up(acc, sum);
            if (step % (kRun * kRun) == kRun * kRun - 1 || step == steps - 1) add_up(sum, total);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads that nothing reads end before the LDS does
    // operand p, component r: output 16 (4 (lane / 16) + r) + op0 + wn + p of the tile
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int token = (tt0 + wt + q) * kTok + (lane & 15);
        if (token >= m) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = tile * kTileOuts + kOuts * (4 * (lane >> 4) + r) + op0 + wn;
            float *dst = Y + (int64_t)token * ldy + o;
            if (o + 4 <= d_out && (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0) {
                *reinterpret_cast<float4 *>(dst) = make_float4(total[0][q][r], total[1][q][r], total[2][q][r], total[3][q][r]);
            } else {
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (o + p < d_out) dst[p] = total[p][q][r];
            }
        }
    }
}

// ---- host

constexpr int kMaxSlabs = 16, kMaxRun = 8, kLeastCost = 6;
constexpr int64_t kDirectWeights = 4 << 20;

int64_t max_steps(int64_t d_in) { return cdiv(d_in, (int64_t)kRowsPerStep) + kMaxSegs; }

// Token tiles of a launch that multiplies while it decodes, and how many a wavefront takes at a time.
int tiles_at_once(int64_t m) { return m > kTok ? 2 : 1; }
int64_t padded_token_tiles(int64_t m) { return align_up((size_t)cdiv(m, (int64_t)kTok), tiles_at_once(m)); }

// Slabs of a tile and token tile: up to 384 workgroups in all, half of what the chip holds at once of
// them, so that two layers of that size run side by side in one go (two 13824x5120 layers in 756
// workgroups; 972 left a second round with a quarter of the chip busy).  Depends on the layer and m
// alone, so that a layer gives the same bits in any group.
int64_t wanted_slabs(int64_t d_out, int64_t m) {
    const int64_t want = 384 / (cdiv(d_out, (int64_t)kTileOuts) * (padded_token_tiles(m) / tiles_at_once(m)));
    return want < 1 ? 1 : (want < kMaxSlabs ? want : kMaxSlabs);
}
// Each width's steps in parts of even cost, the cheapest that need no more slabs than wanted.  A step of
// width 2 takes a wavefront two thirds of the time of one of width 3 or 4 (1.4 and 2.2 us with 3
// wavefronts a SIMD; half as many look-ups).  A part has at most 8 steps: longer runs of fp32 sums lose
// more than the token-by-token kernel.
int64_t part_steps(int bits, int64_t cost) {
    const int64_t n = bits <= 2 ? cost / 2 : cost / 3;
    return n < kMaxRun ? n : kMaxRun;
}
// At least what choose_slabs gives for any widths.
int64_t most_slabs(int64_t d_in, int64_t d_out, int64_t m) {
    const int64_t n = wanted_slabs(d_out, m) + kMaxSegs - 1, least = cdiv(cdiv(max_steps(d_in), (int64_t)kMaxRun) + kMaxSegs, (int64_t)kWaves);
    return n < least ? least : n;
}
// Up to 8 tokens a part has at most 4 steps of width 3 or 4, or as few more as the scratch of most_slabs takes, whatever is
// wanted: longer ones are a chain of latencies in a workgroup, with a third of the chip's places taken (widths 3 and 4 at
// 3.3 bits, 2 tokens: 8192 -> 10240 34.9 us in 360 workgroups of 8 steps, 29.2 in 480 of 6; 7936 -> 10821 35.2 and 30.3;
// 4096 -> 11008 24.5 with 5 steps, 21.8 with 4; 5248 -> 10496 25.2 and 21.9).  Two layers of that size side by side lose the
// round that they shared (4617 -> twice 10583 31.1 and 36.1; 4096 -> twice 11008 30.4 and 32.2; 5535 -> twice 12608
// level), and with more tokens they would lose more (5756 -> 11456 twice, 16 tokens 51.0 us with 6 steps, 54.9 with 5)
// than one alone gains.
constexpr int64_t kShortCost = 12, kShortTokens = 8;
// Parts of one step instead of at least two of width 3 or 4 (three of width 2) in layers of up to 16 steps and 32 tokens,
// which have few workgroups otherwise: 256x15296, 10 tokens 16.7 us, now 14.9; 450x6000 15.6 and 13.8; 256x4096, 24 tokens
// 19.2 and 16.5; smaller ones level.  (Many outputs and tokens lose, 480x16384, 32 tokens 22.7 and 24.2; past 16 steps
// many more do: 512x16384, 16 tokens 18.3 and 19.4; 1024x8192 17.2 and 18.7.)
constexpr int kThinSteps = 16;
void choose_slabs(Layer &L, int64_t m) {
    // (where there are few tiles, widths with few rows get their parts on top)
    const int64_t slabs = wanted_slabs(L.d_out, m), want = kWaves * (slabs + (slabs == kMaxSlabs && L.n_seg > 1 ? L.n_seg - 1 : 0));
    int64_t cost = L.steps <= kThinSteps && m <= 2 * kTok ? 3 : kLeastCost, parts = 0;
    for (;; ++cost) {
        parts = 0;
        for (int j = 0; j < L.n_seg; ++j) parts += cdiv(L.seg[j].steps, part_steps(L.seg[j].bits, cost));
        if (parts <= want || cost == 3 * kMaxRun) break;
        if (m <= kShortTokens && cost >= kShortCost && parts <= kWaves * most_slabs(L.d_in, L.d_out, m)) break;
    }
    int part = 0;
    for (int j = 0; j < L.n_seg; ++j) {
        L.seg[j].part0 = part;
        L.seg[j].parts = (int)cdiv(L.seg[j].steps, part_steps(L.seg[j].bits, cost));
        part += L.seg[j].parts;
    }
    L.slabs = (int)cdiv(parts, (int64_t)kWaves);
    L.span = 0;
    for (int s = 0; s < L.slabs; ++s) {
        int first, last, other;
        part_of(L, s * kWaves, first, other);
        part_of(L, s * kWaves + kWaves - 1, other, last);
        if (last - first > L.span) L.span = last - first;
    }
}

// Whether the workgroups of a layer take the inputs of m tokens straight from X.  They keep those of all
// their rows in LDS, so the fullest slab decides, not the mean: parts are of even cost, and four of width 2 hold up
// to 1.8 times the mean.  It is done where a launch less (3 to 4 us of the host's time, which bounds calls of less than
// 20 us) is worth more than the scattered reads, which grow with the tokens and the entries of O_q in a column.
// Straight | in order, us a call:
//   * up to 4 tokens always (13824x5120 twice, 4 tokens: 41 | 45), up to 8 in layers of up to 64 million weights (4099 and
//     513 of 3001, 5 tokens: 18 | 23; 4096x4096, 6 tokens: 17 | 20; 4096 -> 11008 twice, 8 tokens: level; 8192x28672: 65 | 62);
//   * up to 16 in layers of up to 4 million weights (4096x1024, 0.5 % of the weights in O_q, 12 tokens 17.8 | 18.7; 1 %, 16
//     tokens 21.4 | 19.5), and of up to 12 million up to 40960 tokens times channels (1024x8192, 1 %, 10 tokens 16.0 |
//     16.9; 2048x4096, 16 tokens 19.6 | 18.1 to 19.6, as fast as the host is; 4096x2048, 9 tokens 18.8 | 19.8;
//     3072x3072, 16 tokens 21.1 | 18.2 to 19.3; 4096x4096, 10 tokens 22.7 | 20.0);
//   * up to 32 in layers of up to 16 steps with up to 8192 outputs in the call, more than which the finish kernel takes in
//     two rounds (256x4096, 24 tokens 16.5 | 17.2 to 18.7; 340x9000 22.2 | 18.7; 1000x1000, 32 tokens 19.5 | 19.3;
//     4000x1000, 1 % 24.8 | 20.4).
// Either way the same numbers in the same order.
constexpr int64_t kDirectReads = 40 << 10, kThinOutputs = 8192;
int direct_tokens(int64_t m) { return m <= 4 ? 4 : (m <= 8 ? 8 : (m <= 16 ? 16 : 32)); }
bool direct_inputs(const Layer &L, int64_t m) {
    if (m > 32 || (m > 16 && (L.steps > kThinSteps || L.d_out > kThinOutputs))) return false;
    const int64_t most = kDirectWeights * (m <= 8 ? 16 : (m * L.d_in <= kDirectReads ? 3 : 1));
    if (m > 4 && (int64_t)L.d_in * L.d_out > most) return false;
    return L.span <= direct_steps(direct_tokens(m));
}

// Whether to decode the weight once into memory and multiply from there.  That costs 4 bytes of
// traffic per weight and two launches, multiplying while decoding costs a decoding per 32 tokens;
// measured (us, decode once | while decoding): 4096x4096, 256 tokens 74 | 66; 13824x5120 twice,
// 96 tokens 169 | 152, each 32 tokens more 4 | 39.  Every channel has to have a row, so that an
// entry of O_q always finds the weight it overrides.
constexpr int64_t kManyTokens = 96, kManyProducts = (int64_t)8 << 30;
bool enough_for_many(int64_t d_in, int64_t d_out, int64_t m) {
    return m >= kManyTokens && m * d_in >= kManyProducts / d_out;
}
bool many_tokens(const cmpq_deployed_layer &L, int64_t m) {
    int64_t rows = L.k_act;
    for (int j = 0; j < L.n_set; ++j) rows += L.counts_host[j];
    return rows > 0 && rows == L.d_in && enough_for_many(L.d_in, L.d_out, m);
}

// Tokens of a launch that multiplies while it decodes.  Past the line above (layers that are not
// stored whole) the tokens go in parts of about the line, so that the partial results stay the size
// they have there; and no grid or row of partial results grows past 2^28 for one layer.
int64_t part_tokens(int64_t d_in, int64_t d_out, int64_t m) {
    int64_t c = m;
    if (enough_for_many(d_in, d_out, m)) {
        c = (int64_t)align_up((size_t)cdiv(cdiv(kManyProducts, d_in), d_out), 32);
        if (c < kManyTokens) c = kManyTokens;
    }
    int64_t most = ((int64_t)1 << 28) / (d_in > d_out ? d_in : d_out) / 32 * 32;
    if (most < 32) most = 32;
    if (c > most) c = most;
    return c < m ? c : m;
}

size_t piece(size_t bytes) { return align_up(bytes, 256); }

}  // namespace

// All in us, this way | token by token.  A launch of this kind costs 1 to 6 us more to get going
// (bigger kernels, colder code), a token in it next to nothing; so the line lies where the tokens'
// work outweighs the start.  It is drawn by d_in first, without d_out, so that the layers of a group,
// which read the same input, go the same way: a group split over both ways pays for both
// (2048 -> 2048, 512, 512, 12 tokens: 42 split, 20 | 37; 1000 -> 1024, 300, 32 tokens: 42, 23 | 30).
//   * up to 8 tokens (one answer for all of them, so that a token's bits do not depend on how many
//     come with it) from 960 channels: 300x2048, 4 tokens 15.5 | 12.6; 700x700 16.2 | 14.5;
//     600 -> 600, 700, 800 16.8 | 16.0.  Above the line a layer of its own still loses 1 to 3 us
//     (1000x1024, 4 tokens 15.4 | 13.5; 2048x2048 15.9 | 14.0), groups win (2048 -> 2048, 512, 512
//     16.5 | 18.2; 4096 -> 4096, 512, 512, 2 tokens 20 | 27), and so do outputs that are no multiple
//     of 32 beside rows of O_act (3001x513, 2 tokens 17 | 25).  Below it from 4 million weights:
//     700 -> 3000, 200, 8 tokens 17.2 | 17.9; 300x8192 16.2 | 16.6.
//   * up to 16 tokens, m * d_in from 16384: 2048x512, 9 tokens 18.0 | 15.4; 2048 -> 2048, 512, 512
//     19 | 29.
//   * more, with kernels of 32 tokens, from 24576: 512x512, 32 tokens 19 | 15, 64 tokens 20.5 | 21.3;
//     1024 -> 1024, 256, 256, 24 tokens 19 | 32.
//   * or, past 8 tokens, 24 million weight-token products: 300x8192, 16 tokens 19 | 26.
bool lut_gemm_takes(int64_t d_in, int64_t d_out, int64_t m) {
    if (m < 2) return false;
    if (m <= 8) return d_in >= 960 || d_in >= ((int64_t)4 << 20) / d_out;
    return m * d_in >= (m <= 16 ? 16384 : 24576) || m * d_in >= ((int64_t)24 << 20) / d_out;
}

size_t lut_gemm_ws_bytes(int64_t d_in, int64_t d_out, int64_t m) {
    const int64_t steps = max_steps(d_in), tiles = cdiv(d_out, (int64_t)kTileOuts), part = part_tokens(d_in, d_out, m);
    auto few = [&](int64_t n) -> size_t {
        if (n == 0) return 0;
        const int64_t tt = padded_token_tiles(n);
        return piece((size_t)tt * steps * 1024) + piece((size_t)tt * d_in * kTok * 2) +
               piece((size_t)most_slabs(d_in, d_out, n) * n * d_out * 4);
    };
    size_t b = few(part), last = few(m % part);
    if (last > b) b = last;
    if (enough_for_many(d_in, d_out, m)) {
        const size_t dense = piece((size_t)cdiv(m, (int64_t)kTok) * steps * 1024) + piece((size_t)d_in * 4) +
                             piece((size_t)steps * tiles * kOuts * 1024);
        if (dense > b) b = dense;
    }
    return b;
}

namespace {

// A layer as the kernels see it, its scratch from `base` on; returns the bytes of that.
size_t plan_layer(const cmpq_deployed_layer &S, int64_t m, bool dense, char *base, Layer &L) {
    L = Layer{};
    int64_t steps = 0;
    auto add = [&](const uint32_t *packed, const uint16_t *lut, const int32_t *chan, int64_t rows, int bits) {
        if (rows <= 0) return;
        Seg &g = L.seg[L.n_seg++];
        g.packed = packed;
        g.lut = lut;
        g.chan = chan;
        g.rows = (int)rows;
        g.words_per_row = bits == kActBits ? 0 : (int)cdiv(S.d_out * bits, 32);
        g.bits = bits;
        g.step0 = (int)steps;
        g.steps = (int)cdiv(rows, (int64_t)kRowsPerStep);
        steps += g.steps;
    };
    for (int b = 1; b <= 4; ++b)  // ascending widths
        for (int j = 0; j < S.n_set; ++j)
            if (S.bit_set[j] == b) add(S.packed[j], S.lut[j], S.chan_idx[j], S.counts_host[j], b);
    add(nullptr, nullptr, S.act_idx, S.k_act, kActBits);
    L.X = static_cast<const __half *>(S.X);
    L.ldx = S.ldx;
    L.W_act = reinterpret_cast<const __half *>(S.W_act);
    L.ld_act = S.ld_act;
    L.colptr = S.colptr;
    L.row_idx = S.row_idx;
    L.delta = S.delta;
    L.Y = S.Y;
    L.ldy = S.ldy;
    L.d_in = (int)S.d_in;
    L.d_out = (int)S.d_out;
    L.steps = (int)steps;
    L.tiles = (int)cdiv(S.d_out, (int64_t)kTileOuts);
    size_t used = 0;
    auto take = [&](size_t bytes) {
        char *p = base + used;
        used += piece(bytes);
        return p;
    };
    if (dense) {
        L.xf = reinterpret_cast<uint4 *>(take((size_t)cdiv(m, (int64_t)kTok) * steps * 1024));
        if (S.colptr) L.pos = reinterpret_cast<int32_t *>(take((size_t)S.d_in * 4));
        L.dense = reinterpret_cast<uint4 *>(take((size_t)steps * L.tiles * kOuts * 1024));
    } else {
        const int64_t tts = padded_token_tiles(m);
        L.xf = reinterpret_cast<uint4 *>(take((size_t)tts * steps * 1024));
        if (S.colptr) L.xt = reinterpret_cast<__half *>(take((size_t)tts * S.d_in * kTok * 2));
        choose_slabs(L, m);
        L.partial = reinterpret_cast<float *>(take((size_t)L.slabs * m * S.d_out * 4));
    }
    return used;
}

}  // namespace

size_t lut_gemm_need(const cmpq_deployed_layer &S, int64_t m) {
    Layer L;
    if (many_tokens(S, m)) return plan_layer(S, m, true, nullptr, L);
    const int64_t part = part_tokens(S.d_in, S.d_out, m);
    const size_t first = plan_layer(S, part, false, nullptr, L);
    const size_t last = m % part ? plan_layer(S, m % part, false, nullptr, L) : 0;
    return first > last ? first : last;
}

void lut_gemm_shape(const cmpq_deployed_layer &S, int64_t m, int64_t *shape, int64_t *parts, int64_t room) {
    Layer L;
    if (many_tokens(S, m)) {
        plan_layer(S, m, true, nullptr, L);
        shape[0] = 2, shape[1] = m, shape[2] = L.tiles;
        return;
    }
    const int64_t at_once = part_tokens(S.d_in, S.d_out, m);
    plan_layer(S, at_once, false, nullptr, L);
    shape[0] = 1, shape[1] = at_once, shape[2] = L.slabs;
    const int nd = direct_tokens(at_once), n = L.n_seg ? L.seg[L.n_seg - 1].part0 + L.seg[L.n_seg - 1].parts : 0;
    for (int part = 0; part < n && part < room; ++part) {
        int lo, hi;
        const Seg &s = L.seg[part_of(L, part, lo, hi)];
        const int64_t row = (int64_t)(lo - s.step0) * kRowsPerStep, rows = (int64_t)(hi - lo) * kRowsPerStep;
        parts[3 * part] = s.bits, parts[3 * part + 1] = row;
        parts[3 * part + 2] = row + rows < s.rows ? rows : s.rows - row;
    }
    shape[3] = n;
    shape[4] = direct_inputs(L, at_once) ? (int64_t)nd * (L.span * kRowsPerStep + 8) * (int64_t)sizeof(__half) : 0;
    shape[5] = kSlabLds - kTablesBytes;
}

int launch_lut_gemm(const cmpq_deployed_layer *const *layers, int n_layers, int64_t m, void *ws, hipStream_t s) {
    Group few, many;
    few.n_layers = many.n_layers = 0;
    const int MT = tiles_at_once(m);
    const int64_t tts = padded_token_tiles(m);
    char *base = static_cast<char *>(ws);
    for (int i = 0; i < n_layers; ++i) {
        const cmpq_deployed_layer &S = *layers[i];
        const bool dense = many_tokens(S, m);
        const int64_t part = dense ? m : part_tokens(S.d_in, S.d_out, m);
        if (part < m) {  // on its own, a part of the tokens after the other in the same scratch
            for (int64_t t = 0; t < m; t += part) {
                cmpq_deployed_layer P = S;
                P.X = static_cast<const __half *>(S.X) + t * S.ldx;
                P.Y = S.Y + t * S.ldy;
                const cmpq_deployed_layer *one = &P;
                const int rc = launch_lut_gemm(&one, 1, m - t < part ? m - t : part, base, s);
                if (rc != CMPQ_OK) return rc;
            }
            base += lut_gemm_need(S, m);
            continue;
        }
        Group &G = dense ? many : few;
        base += plan_layer(S, m, dense, base, G.l[G.n_layers++]);
    }
    for (Group *G : {&few, &many}) {
        if (G->n_layers == 0) continue;
        const int n = G->n_layers;
        G->m = (int)m;
        G->token_tiles = (int)(G == &few ? tts : cdiv(m, (int64_t)kTok));
        auto number = [&](auto &&count) {
            int64_t w = 0;
            for (int i = 0; i < kMaxLayers; ++i) G->wg0[i] = INT_MAX;
            for (int i = 0; i < n; ++i) {
                G->wg0[i] = (int)w;
                w += count(G->l[i]);
            }
            return (unsigned)w;
        };
        const unsigned wx = number([&](const Layer &L) {
            return G->token_tiles * (cdiv(L.steps, 8) + (L.xt ? cdiv(L.d_in, (int64_t)kThreads) : 0)); });
        const int nd = direct_tokens(m);
        bool direct = G == &few;
        // (past 8 tokens by the weights of all layers: the launch left out is one, the scattered reads are each layer's;
        // 542 -> three times 13568, 12 tokens: 28.9 us with inputs straight from X, 24.1 without)
        int64_t weights = 0, outputs = 0;
        for (int i = 0; i < n; ++i) weights += (int64_t)G->l[i].d_in * G->l[i].d_out, outputs += G->l[i].d_out;
        if (m > 8 && weights > 4 * kDirectWeights) direct = false;
        if (m > 16 && outputs > kThinOutputs) direct = false;
        for (int i = 0; direct && i < n; ++i) direct = direct_inputs(G->l[i], m);
        if (wx && !direct && G == &few) tokens_kernel<<<wx, kThreads, 0, s>>>(*G);
        if (G == &few) {
            const unsigned w = number([&](const Layer &L) { return (int64_t)L.tiles * L.slabs * (tts / MT); });
            if (w > 0) {
                const int d = direct ? nd : 0;
                if (d == 4) lut_tokens_kernel<1, 4><<<w, kThreads, 0, s>>>(*G);
                else if (d == 8) lut_tokens_kernel<1, 8><<<w, kThreads, 0, s>>>(*G);
                else if (d == 16) lut_tokens_kernel<1, 16><<<w, kThreads, 0, s>>>(*G);
                else if (d == 32) lut_tokens_kernel<2, 32><<<w, kThreads, 0, s>>>(*G);
                else if (MT == 1) lut_tokens_kernel<1, 0><<<w, kThreads, 0, s>>>(*G);
                else lut_tokens_kernel<2, 0><<<w, kThreads, 0, s>>>(*G);
            }
            const unsigned f = number([&](const Layer &L) { return cdiv(L.d_out, (int64_t)kFinCols) * tts; });
            if (direct && nd == 4) tokens_finish_kernel<4, true><<<f, kThreads, 0, s>>>(*G);
            else if (direct && nd == 8) tokens_finish_kernel<8, true><<<f, kThreads, 0, s>>>(*G);
            else if (direct) tokens_finish_kernel<16, true><<<f, kThreads, 0, s>>>(*G);
            else if (m <= 8) tokens_finish_kernel<8, false><<<f, kThreads, 0, s>>>(*G);
            else tokens_finish_kernel<16, false><<<f, kThreads, 0, s>>>(*G);
        } else {
            DecodeWgs d;
            int64_t w = 0;
            for (int i = 0; i < kMaxLayers; ++i) {
                d.wg0[i] = i < n ? (int)w : INT_MAX;
                if (i < n) w += cdiv((int64_t)G->l[i].steps * G->l[i].tiles, (int64_t)kWaves);
            }
            d.first = (int)wx;
            lut_decode_kernel<<<(unsigned)(wx + w), kThreads, 0, s>>>(*G, d);
            bool any = false;
            for (int i = 0; i < n; ++i) any = any || G->l[i].colptr;
            if (any) {
                const unsigned o = number([&](const Layer &L) { return L.colptr ? cdiv(L.d_out, (int64_t)kWaves) : 0; });
                override_kernel<<<o, kThreads, 0, s>>>(*G);
            }
            const int64_t tb = cdiv((int64_t)G->token_tiles, (int64_t)kGemmOps);
            const unsigned q = number([&](const Layer &L) { return 2 * L.tiles * tb; });
            weight_gemm_kernel<<<q, kThreads, 0, s>>>(*G);
        }
    }
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}
