// Bucket k-means for the common case of cmpq_kmeans_quantize: fp16 weights, unit
// importance (Sec. 3.2.1 of arXiv 2410.13056; entries of O_q removed as in Sec. 3.2.2).
//
// A Lloyd round on a line only needs, for each boundary between two neighbouring
// levels, how many weights lie below it and what they sum to.  Three kernels:
//
//   * kmeans_build_kernel arranges a channel once so that a round reads these numbers instead of
//     recounting them.  Every weight becomes its 16-bit order key (unsigned order = value order); the
//     top bits name a bucket (1024 of 64 places for long channels, 512 of 128 otherwise), the low bits
//     the place inside it.  One pass counts the buckets and sums the places, a scan turns this into
//     exclusive prefixes of the count and of the exact integer sum of x*2^24 (inside a bucket x*2^24 is
//     affine in the place: sign, exponent and top mantissa bits are shared), a second pass scatters the
//     places into an LDS byte array ordered by bucket (any order inside a bucket; a bucket's stretch
//     starts on a whole word and its unused tail holds a filler above every place).  The tables go to
//     memory;
//   * kmeans_rounds_kernel runs start-up and rounds from the tables: per boundary the prefix of its
//     bucket plus a scan of that one bucket; a cell is the difference of two boundaries, and the new
//     level is the exact integer sum divided in fp64 and rounded once to fp32 - the value an fp64
//     reference computes.  When no boundary moved the iteration has reached its fixed point and the
//     remaining rounds, which would repeat it, are skipped;
//   * kmeans_code_kernel codes the weights with the final boundaries, and writes the stored format and
//     the error where they are asked for.
//
// Few channels, short ones and few rounds go through all three in one workgroup each, with their tables in LDS
// (kmeans_channel_kernel).
//
// A quantization without entries of O_q can leave its tables to a later one with them.  That one has
// kmeans_removed_kernel arrange the removed entries alone, in the same form, and its rounds take
// (all) - (removed) at every boundary.
//
// Why three kernels.  A round is a chain of some 200 dependent instructions and two table look-ups, 20
// times over, which one wavefront can run for several channels at once - while a channel's tables take
// 5 to 36 KB to build in LDS.  In one kernel the rounds, half of a channel's time, hold that LDS and all
// wavefronts of the channel, and leave a compute unit with 3 to 16 channels to hide the chain behind (2400
// cycles a round at 28672 weights, where a wavefront alone needs 1400).  On their own they hold 4.4 to 10.2 KB a
// channel and one wavefront for 1 to 4.  Both quantizations of a layer, widths 2 to 4 at 3.5 on average, 1 %
// in O_q, us in one kernel -> now (first + final):
//   8192 x 28672  471 + 594 -> 318 + 411      4096 x 11008  192 + 244 -> 102 + 156
//   28672 x 8192  574 + 751 -> 446 + 578      8192 x 1024    98 + 133 ->  58 + 95
//   4096 x 4096    82 + 112 ->  64 + 94
// Tried on the way, same results: rounds of 4 / 2 / 1 channels on one wavefront inside the one kernel (1024
// weights 98 -> 70, 8192 weights 574 -> 630), all tables of the rounds in LDS (28672 x 8192 528: too few
// channels at a time), none of them (gate-shaped 373, the records' lines do not stay in L2).
//
// All sums are integers, so the result is reproducible bit for bit and identical to the
// brute-force kernels.  Boundaries are exact: between distinct neighbouring levels
// lo < hi the boundary key is that of the largest fp16 value below the real midpoint (or
// equal to it when the tie rule gives the midpoint to lo).  Levels are ranked by (value,
// index) whenever their order may have changed; they need not stay ascending because a
// level without members keeps a stale value.
//
// A channel with NaN or infinity raises the status flag and gets levels 0 and codes 0.
#include <type_traits>

#include "kmeans_args.h"
#include "kmeans_keys.h"

namespace {

// Bytes of the place array: one per weight plus up to 3 of filler per non-empty bucket.
__host__ __device__ inline size_t bucket_arr_bytes(int64_t d_out, int lb) {
    const int64_t buckets = (int64_t)1 << (16 - lb);
    const int64_t pad = 3 * (d_out < buckets ? d_out : buckets);
    return ((size_t)(d_out + pad) + 15) & ~(size_t)15;
}

// RAGGED: rows that are no whole number of groups of 4 weights, or do not start on 8 bytes.  A
// group is then fetched and its codes are stored at any alignment; the last one may hold 1 to 3
// weights, and what fills it up is marked as removed.
template <bool RAGGED>
__device__ __forceinline__ uint2 load_group(const __half *row, int g, int n_groups, int d_out) {
    uint2 v = make_uint2(0, 0);
    if (g >= n_groups) return v;
    if constexpr (!RAGGED) return reinterpret_cast<const uint2 *>(row)[g];
    const __half *p = row + 4 * (int64_t)g;
    const int n = d_out - 4 * g;
    if (n >= 4) {
        __builtin_memcpy(&v, p, 8);
    } else {
        v.x = __half_as_ushort(p[0]);
        if (n > 1) v.x |= (uint32_t)__half_as_ushort(p[1]) << 16;
        if (n > 2) v.y = __half_as_ushort(p[2]);
    }
    return v;
}
template <bool RAGGED>
__device__ __forceinline__ void store_codes(uint8_t *row, int g, int d_out, uint32_t word) {
    if constexpr (!RAGGED) {
        reinterpret_cast<uint32_t *>(row)[g] = word;
    } else {
        const int n = d_out - 4 * g;
        if (n >= 4) __builtin_memcpy(row + 4 * (int64_t)g, &word, 4);
        else for (int e = 0; e < n; ++e) row[4 * (int64_t)g + e] = (uint8_t)(word >> (8 * e));
    }
}
template <bool RAGGED, int T>
__device__ __forceinline__ void zero_codes(uint8_t *row, int tid, int n_groups, int d_out) {
    if (!row) return;
    for (int g = tid; g < n_groups; g += T) store_codes<RAGGED>(row, g, d_out, 0);
}

// A channel's tables in memory: head | one record per bucket | the place array.
struct TableHead {
    uint32_t magic;          // kTableMagic + 1: tables follow; + 2: the channel held a non-finite weight
    uint32_t kept;           // weights that take part
    uint32_t d_out, unused;  // row length
    // exact sum of x * 2^24 over the keys below key k << 10 (64 runs of 1024 keys: one sign and exponent
    // each); [64] is the sum over all
    long long base[65];
    uint32_t unused2[2];
    uint32_t fill[4];        // filler
};
constexpr uint32_t kTableMagic = 0xC3A77B00u;
// Record of a bucket: .x = word of the place array where its stretch begins | weights below it << 16; .y =
// sum over the buckets below it that share its sign and exponent, in units of that exponent's spacing
// (|.y| <= 2047 * 32768).  A stretch ends where the next one begins.
static_assert(sizeof(TableHead) == 560, "records start on 16 bytes");
// 16 bytes more than the place array: scans read whole groups of 4 words.
__host__ __device__ inline size_t table_bytes(int64_t d_out, int lb) {
    return sizeof(TableHead) + ((size_t)8 << (16 - lb)) + bucket_arr_bytes(d_out, lb) + 16;
}

// Of bucket b: mantissa of its first key with the sign, and the exponent's shift: x * 2^24 = (mantissa + place) << sh.
template <int LB>
__device__ __forceinline__ void bucket_scale(uint32_t b, int &mant, uint32_t &sh) {
    const uint32_t h = half_of_key(b << LB);
    const uint32_t e = (h >> 10) & 31u;
    const int mag = (int)((e ? 1024u : 0u) + (h & 1023u));
    sh = (e > 1 ? e : 1) - 1;
    mant = (h & 0x8000u) ? -mag : mag;
}

template <int G>
__device__ __forceinline__ uint32_t elem_key(const uint32_t (&keys)[2 * G], int k, int e) {
    return (keys[2 * k + (e >> 1)] >> (16 * (e & 1))) & 0xffffu;
}

// Counts the buckets and sums the places of the kept weights with packed LDS atomics: `n << kShift |
// sum of places`.  In 32 bits the sum of a bucket may run over into its count (channels of more than
// 4096 weights); every such carry makes the counts add up to more than the weights, which is how the
// caller finds out that it has to count again in 64 bits.
//
// Low bits of the word that the sum of places has: the count's need room for all 4 * G * T weights that a
// workgroup can take.
template <int G, int T>
constexpr int count_shift() {
    int shift = 31;
    for (int n = 4 * G * T; n > 1; n >>= 1) --shift;
    return shift;
}
template <int G, int T, int LB>
constexpr bool kMayCarry = (int64_t)4 * G * T * ((1 << LB) - 1) >= (int64_t)1 << count_shift<G, T>();
// LDS of the place array.  The 64-bit count lies there before the places do, and the bitmap behind it has to
// outlive that count.
template <int G, int T, int LB>
__host__ __device__ inline size_t place_area_bytes(int64_t d_out) {
    const size_t arr = bucket_arr_bytes(d_out, LB), wide = kMayCarry<G, T, LB> ? (size_t)8 << (16 - LB) : 0;
    return arr > wide ? arr : wide;
}
template <int G, int T, int LB, bool MASKED, int kShift, typename Word>
__device__ __forceinline__ void count_buckets(const uint32_t (&keys)[2 * G], const uint32_t *removed, Word *table,
                                              int tid, int n_groups) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int g = k * T + tid;
        if (g < n_groups) {
            uint32_t kept = 0xfu;  // 4 bits of the bitmap per group of 4 weights
            if constexpr (MASKED) kept = ~(removed[g >> 3] >> ((g & 7) * 4)) & 0xfu;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!MASKED || ((kept >> e) & 1u)) {
                    const uint32_t key = elem_key<G>(keys, k, e);
                    atomicAdd(&table[key >> LB], ((Word)1 << kShift) | (key & ((1u << LB) - 1)));
                }
            }
        }
    }
}

// Keeps what one pass over the keys works out (bucket and bitmap addresses) from being held for the next: of 64
// registers, the 32 keys of a lane of the longest channels leave no room for it.
template <int G>
__device__ __forceinline__ int next_pass(uint32_t (&keys)[2 * G], int tid) {
#pragma unroll
    for (int k = 0; k < 2 * G; ++k) asm("" : "+v"(keys[k]));
    asm("" : "+v"(tid));
    return tid;
}

// Puts the place of every kept weight into its bucket's stretch of the byte array.
template <int G, int T, int LB, bool MASKED>
__device__ __forceinline__ void scatter_places(const uint32_t (&keys)[2 * G], const uint32_t *removed,
                                               uint32_t *cursor, unsigned char *arr, int tid, int n_groups) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int g = k * T + tid;
        if (g < n_groups) {
            uint32_t kept = 0xfu;
            if constexpr (MASKED) kept = ~(removed[g >> 3] >> ((g & 7) * 4)) & 0xfu;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!MASKED || ((kept >> e) & 1u)) {
                    const uint32_t key = elem_key<G>(keys, k, e);
                    const uint32_t pos = atomicAdd(&cursor[key >> LB], 1u);
                    arr[pos] = (unsigned char)(key & ((1u << LB) - 1));
                }
            }
        }
    }
}

// The exclusive prefix over the kBuckets buckets of a channel: every lane hands over the counts n and sums of
// places l of its `per` buckets from b0 on (lanes past the buckets: none).  Writes the records and the head's
// sums to memory; start[r] becomes the byte where the bucket's stretch begins.  Returns the number of weights
// counted.  All T lanes call it; contains barriers.
template <int T>
struct PrefixShared {
    uint32_t wave_n[T / CMPQ_WAVE + 1];
    long long run[64];  // per sign and exponent: sum of x * 2^24
};
template <int T, int LB>
__device__ __forceinline__ uint32_t write_records(PrefixShared<T> &sm, const uint32_t *n, const uint32_t *l,
                                                  uint32_t *start, TableHead *head, uint2 *rec, uint32_t *total_n) {
    constexpr int kBuckets = 1 << (16 - LB), kPer = kBuckets / T > 0 ? kBuckets / T : 1;
    constexpr int kSeg = T >= 64 ? (T / 64 < kBuckets / 64 ? T / 64 : kBuckets / 64) : 1;  // lanes that share a sign and exponent
    static_assert(kBuckets >= T, "a lane owns whole buckets");
    constexpr int kWaves = T / CMPQ_WAVE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b0 = tid * kPer;
    uint32_t n_loc = 0;  // count | padded count << 16: both stay below 2^16
    int u_loc = 0, mant;
    uint32_t sh;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        n_loc += n[r] | (((n[r] + 3) & ~3u) << 16);
        bucket_scale<LB>((uint32_t)(b0 + r), mant, sh);
        u_loc += __mul24(mant, (int)n[r]) + (int)l[r];
    }
    // sums inside a run of equal sign and exponent (its kSeg lanes are neighbours)
    int u_incl = u_loc;
    static_assert(kSeg <= 8, "inside a row of 16 lanes");
    auto from_below = [&](auto d) {
        const int up = __builtin_amdgcn_update_dpp(0, u_incl, 0x110 + d, 0xF, 0xF, true);  // row_shr:d
        if ((lane & (kSeg - 1)) >= d) u_incl += up;
    };
    if constexpr (kSeg > 1) from_below(std::integral_constant<int, 1>{});
    if constexpr (kSeg > 2) from_below(std::integral_constant<int, 2>{});
    if constexpr (kSeg > 4) from_below(std::integral_constant<int, 4>{});
    if ((lane & (kSeg - 1)) == kSeg - 1) {
        bucket_scale<LB>((uint32_t)b0, mant, sh);
        sm.run[(b0 << LB) >> 10] = (long long)((unsigned long long)(long long)u_incl << sh);
    }
    uint32_t n_incl = wave_scan_incl_u32(n_loc);
    if (lane == 63) sm.wave_n[wave] = n_incl;
    __syncthreads();
    uint32_t n_run = n_incl - n_loc, n_tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t t = sm.wave_n[w];
        if (w < wave) n_run += t;
        n_tot += t;
    }
    if (wave == 0) {
        const unsigned long long v = (unsigned long long)sm.run[lane];
        const unsigned long long incl = wave_scan_incl_u64(v);
        head->base[lane] = (long long)(incl - v);
        if (lane == 63) head->base[64] = (long long)incl;
        if (lane < 4) head->fill[lane] = kFill4;
    }
    int u_run = u_incl - u_loc;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        start[r] = n_run >> 16;
        rec[b0 + r] = make_uint2((n_run >> 18) | (n_run << 16), (uint32_t)u_run);
        bucket_scale<LB>((uint32_t)(b0 + r), mant, sh);
        n_run += n[r] | (((n[r] + 3) & ~3u) << 16);
        u_run += __mul24(mant, (int)n[r]) + (int)l[r];
    }
    *total_n = n_tot;
    return n_tot & 0xffffu;
}

// Tables of channel i: head and records where the caller wants them, the place array at the start of `dyn`.  Dynamic
// LDS: places of the kept weights, ordered by bucket | removed-entry bitmap (one bit per weight; MASKED) | a word per
// bucket: count and sum of places, then the cursor of its stretch.  Returns the bytes of the place array that hold
// stretches, -1 for a channel with a non-finite weight (the same for all lanes); ends in a barrier.
template <int T>
struct BuildShared {
    PrefixShared<T> prefix;
    uint32_t flag[T / CMPQ_WAVE];
};
template <int G, int T, int LB, bool MASKED, bool RAGGED>
__device__ __forceinline__ int build_tables(const KmArgs &a, int64_t i, unsigned char *dyn, BuildShared<T> &sm,
                                            TableHead *head, uint2 *rec) {
    constexpr int kBuckets = 1 << (16 - LB), kPer = kBuckets / T, kShift = count_shift<G, T>();
    const int tid = threadIdx.x;
    const int d_out = (int)a.d_out, n_groups = RAGGED ? (d_out + 3) >> 2 : d_out >> 2;
    const size_t arr_bytes = bucket_arr_bytes(d_out, LB);
    const int n_words = MASKED ? (d_out + 31) >> 5 : 0;
    unsigned char *arr = dyn;
    uint32_t *removed = reinterpret_cast<uint32_t *>(dyn + place_area_bytes<G, T, LB>(d_out));
    uint32_t *cursor = removed + ((n_words + 3) & ~3);
    const __half *wrow = static_cast<const __half *>(a.W) + i * a.ldw;

    // lane owns groups g = k*T + tid of 4 weights, kept as packed 16-bit keys
    uint32_t keys[2 * G];
    uint32_t nonfinite = 0;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const uint2 raw = load_group<RAGGED>(wrow, k * T + tid, n_groups, d_out);
        keys[2 * k] = raw.x;
        keys[2 * k + 1] = raw.y;
    }
    const uint4 fill = make_uint4(kFill4, kFill4, kFill4, kFill4);
    for (int s = tid; s < (int)(arr_bytes >> 4); s += T) reinterpret_cast<uint4 *>(arr)[s] = fill;
#pragma unroll
    for (int r = 0; r < kPer; ++r) cursor[r * T + tid] = 0;
    for (int s = tid; s < n_words; s += T)  // what fills up the last group counts as removed
        removed[s] = RAGGED && s == d_out >> 5 && (d_out & 3) ? ((1u << (4 - (d_out & 3))) - 1u) << (d_out & 31) : 0u;
#pragma unroll
    for (int k = 0; k < 2 * G; ++k) {
        nonfinite |= nonfinite_of_half2(keys[k]);
        keys[k] = keys_of_half2(keys[k]);
    }
    const bool bad = __ballot((nonfinite & 0x80008000u) != 0u) != 0ull;
    if ((tid & 63) == 0) sm.flag[tid >> 6] = bad;
    __syncthreads();
    {
        uint32_t any = 0;
#pragma unroll
        for (int w = 0; w < T / CMPQ_WAVE; ++w) any |= sm.flag[w];
        if (any) {
            if (tid == 0) head->magic = kTableMagic + 2u, head->d_out = (uint32_t)d_out;
            return -1;
        }
    }
    int n_ex = 0;
    if constexpr (MASKED) {  // entries of O_q do not take part in the clustering
        const int lo = a.seg ? a.seg[i] : 0;
        n_ex = a.seg ? a.seg[i + 1] - lo : 0;
        const int32_t chan_base = (int32_t)(i * a.d_out);
        for (int e = tid; e < n_ex; e += T) {
            const int o = a.out_idx[lo + e] - chan_base;
            atomicOr(&removed[o >> 5], 1u << (o & 31));
        }
        __syncthreads();
    }
    count_buckets<G, T, LB, MASKED, kShift>(keys, removed, cursor, next_pass<G>(keys, tid), n_groups);
    __syncthreads();
    uint32_t n[kPer], l[kPer], start[kPer], total;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const uint32_t w = cursor[tid * kPer + r];
        n[r] = w >> kShift;
        l[r] = w & ((1u << kShift) - 1u);
    }
    uint32_t kept = write_records<T, LB>(sm.prefix, n, l, start, head, rec, &total);
    if constexpr (kMayCarry<G, T, LB>) {
        if (kept != (uint32_t)(d_out - n_ex)) {  // a sum of places ran over into a count (the same for all lanes):
            unsigned long long *wide = reinterpret_cast<unsigned long long *>(arr);  // again, in 64 bits
            __syncthreads();
            for (int s = tid; s < kBuckets; s += T) wide[s] = 0;
            __syncthreads();
            count_buckets<G, T, LB, MASKED, 32>(keys, removed, wide, next_pass<G>(keys, tid), n_groups);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                const unsigned long long w = wide[tid * kPer + r];
                n[r] = (uint32_t)(w >> 32);
                l[r] = (uint32_t)w;
            }
            __syncthreads();
            for (int s = tid; s < (int)(arr_bytes >> 4); s += T) reinterpret_cast<uint4 *>(arr)[s] = fill;
            kept = write_records<T, LB>(sm.prefix, n, l, start, head, rec, &total);
        }
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) cursor[tid * kPer + r] = start[r];
    __syncthreads();
    scatter_places<G, T, LB, MASKED>(keys, removed, cursor, arr, next_pass<G>(keys, tid), n_groups);
    __syncthreads();
    if (tid == 0) {
        head->magic = kTableMagic + 1u;
        head->kept = kept;
        head->d_out = (uint32_t)d_out;
    }
    return (int)(total >> 16);
}

// The stretches to memory, up to the last one's end; what a scan may read past it is defined too.
template <int T>
__device__ __forceinline__ void store_places(void *to, const unsigned char *arr, int bytes, size_t arr_bytes) {
    const int quads = min(((bytes + 15) >> 4) + 1, (int)(arr_bytes >> 4));
    for (int s = threadIdx.x; s < quads; s += T)
        reinterpret_cast<uint4 *>(to)[s] = reinterpret_cast<const uint4 *>(arr)[s];
}

// The tables of one channel, built in LDS.  Bound by LDS (an atomic, a returning atomic and a byte store to
// scattered addresses per weight: 6.7 clocks a wavefront instruction, two thirds of them bank conflicts) and
// by what it reads and writes: 2 B a weight in, 1.1 B and 8 B a bucket out.  8192 x 28672 in 208 us, 220 with removed
// entries.  64 registers: 8 wavefronts a SIMD, so that one workgroup's fetch runs beside the others' LDS passes; nothing
// may spill (231 and 307 us with 32 and 80 bytes of scratch a lane, written and read with the tables).  Counting in 32
// bits where that is enough halves the LDS words of a count.
template <int G, int T, int LB, bool MASKED, bool RAGGED>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(8, 8))) void kmeans_build_kernel(KmArgs a, int64_t i0, unsigned char *tables, int64_t stride) {
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ BuildShared<T> sm;
    const int64_t i = i0 + blockIdx.x;
    const int b = a.bits[i];
    if (b < 1 || b > 4) return;
    TableHead *head = reinterpret_cast<TableHead *>(tables + blockIdx.x * stride);
    uint2 *rec = reinterpret_cast<uint2 *>(head + 1);
    const int bytes = build_tables<G, T, LB, MASKED, RAGGED>(a, i, dyn, sm, head, rec);
    if (bytes >= 0) store_places<T>(rec + (1 << (16 - LB)), dyn, bytes, bucket_arr_bytes((int)a.d_out, LB));
}

// The removed entries of one channel (slice of out_idx), in the form of the tables above.  About 1 % of the
// channel: bound by latency (a gather of their weights) and by the records.
constexpr int kRemovedLanes = 256;
template <int LB>
__global__ __launch_bounds__(kRemovedLanes) void kmeans_removed_kernel(KmArgs a, int64_t i0, unsigned char *tables,
                                                                      int64_t stride) {
    constexpr int T = kRemovedLanes, kBuckets = 1 << (16 - LB), kPer = kBuckets / T;
    __shared__ PrefixShared<T> sm;
    __shared__ unsigned long long count[kBuckets];  // count << 32 | sum of places, then the cursors
    const int64_t i = i0 + blockIdx.x;
    const int b = a.bits[i];
    if (b < 1 || b > 4) return;
    const int tid = threadIdx.x;
    const __half *wrow = static_cast<const __half *>(a.W) + i * a.ldw;
    TableHead *head = reinterpret_cast<TableHead *>(tables + blockIdx.x * stride);
    uint2 *rec = reinterpret_cast<uint2 *>(head + 1);
    const int lo = a.seg[i], n_ex = min(a.seg[i + 1] - lo, (int)a.d_out);
    if (n_ex <= 0) {
        if (tid == 0) head->kept = 0;
        return;
    }
    const int32_t chan_base = (int32_t)(i * a.d_out);
    constexpr int kHeld = 2;  // entries whose keys a lane keeps for the second visit
    uint32_t held[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int e = u * T + tid;
        held[u] = e < n_ex ? key_of_half(__half_as_ushort(wrow[a.out_idx[lo + e] - chan_base])) : 0u;
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) count[r * T + tid] = 0;
    __syncthreads();
    auto each = [&](auto &&visit) {
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if (u * T + tid < n_ex) visit(held[u]);
        for (int e = kHeld * T + tid; e < n_ex; e += T) visit(key_of_half(__half_as_ushort(wrow[a.out_idx[lo + e] - chan_base])));
    };
    each([&](uint32_t key) { atomicAdd(&count[key >> LB], (1ull << 32) | (key & ((1u << LB) - 1))); });
    __syncthreads();
    uint32_t n[kPer], l[kPer], start[kPer], total;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const unsigned long long w = count[tid * kPer + r];
        n[r] = (uint32_t)(w >> 32);
        l[r] = (uint32_t)w;
    }
    write_records<T, LB>(sm, n, l, start, head, rec, &total);
    unsigned char *arr = reinterpret_cast<unsigned char *>(rec + kBuckets);
    uint32_t *cursor = reinterpret_cast<uint32_t *>(count);
#pragma unroll
    for (int r = 0; r < kPer; ++r) {  // (a lane's words lie in its own entries of `count`)
        cursor[2 * (tid * kPer + r)] = start[r];
        for (uint32_t s = start[r] + n[r]; s < ((start[r] + n[r] + 3) & ~3u); ++s) arr[s] = 0x80;
    }
    if (tid < 4) reinterpret_cast<uint32_t *>(arr + (total >> 16))[tid] = kFill4;  // a scan may read past the last stretch
    __syncthreads();
    each([&](uint32_t key) { arr[atomicAdd(&cursor[2 * (key >> LB)], 1u)] = (unsigned char)(key & ((1u << LB) - 1)); });
    if (tid == 0) head->kept = total & 0xffffu;
}

// What the rounds leave for the coding pass.
struct ChannelFinal {
    uint16_t tk[CMPQ_KMAX];      // boundary keys by sorted position
    uint8_t code_of[CMPQ_KMAX];  // level index that each sorted position stands for
    uint32_t ok;                 // 0: the channel was flagged, its codes are zero
    uint32_t unused[3];
};
static_assert(sizeof(ChannelFinal) == 64, "one line of memory");

// Sum over the R = 1, 2 or 4 rows of 16 lanes that share a channel; every row gets it.
template <int R>
__device__ __forceinline__ uint32_t row_group_sum(uint32_t v) {
    if constexpr (R >= 2) {
        const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = s[0] + s[1];
    }
    if constexpr (R >= 4) {
        const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = s[0] + s[1];
    }
    return v;
}

// Value that lane `l` of the caller's row of 16 lanes holds.
__device__ __forceinline__ float from_row_lane(float v, int l) {
    return __shfl(v, (threadIdx.x & 48) | l, CMPQ_WAVE);
}
__device__ __forceinline__ int from_row_lane(int v, int l) {
    return __shfl(v, (threadIdx.x & 48) | l, CMPQ_WAVE);
}

// Value of lane L of the caller's row of 16 lanes, on the DPP path.
template <int L>
__device__ __forceinline__ float row_bcast(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x150 + L, 0xF, 0xF, true));  // row_newbcast:L
}
// Hands v to lane `to` of the caller's row; the lanes of a row name different ones.
__device__ __forceinline__ int to_row_lane(int v, int to) {
    return __builtin_amdgcn_ds_permute(((threadIdx.x & 48) | to) << 2, v);
}
__device__ __forceinline__ float to_row_lane(float v, int to) {
    return __uint_as_float((uint32_t)to_row_lane((int)__float_as_uint(v), to));
}

// Number of lanes of the row before lane j in the order (value, lane): lanes L on.
template <int L>
__device__ __forceinline__ int rank_in_row(float c, int j) {
    const float cl = row_bcast<L>(c);
    const int before = (cl < c) || (cl == c && L < j) ? 1 : 0;
    if constexpr (L + 1 < CMPQ_KMAX) return before + rank_in_row<L + 1>(c, j);
    else return before;
}

// Levels by level index (lane j of a row of 16 lanes holds c for j < K, infinity above) -> per sorted
// position p (lane p): value, owning level, next distinct value above and the owners for the tie rule.
// Handles repeated values and any order.  K may differ from row to row.  Levels that no weight is nearest to repeat
// one another round after round where a channel has few different values, so this counts: as 48 exchanges through
// LDS one after the other, 3000 channels of 8 weights took 53 us (26 now, in the three kernels), 4096 x 4096 with all of
// one row's weights removed 149 (73).
__device__ __forceinline__ void rank_levels_in_rows(float c, int K, float &sorted, int &own, float &hi, int &owner_lo,
                                                    int &owner_hi, bool &have_hi) {
    const int j = threadIdx.x & 15;
    const int rank = rank_in_row<0>(c, j);
    sorted = to_row_lane(c, rank);
    own = to_row_lane(j, rank);
    // positions whose neighbour above is larger: the next of them from j on, and the one before j, end j's run of
    // equal values
    const float above = __uint_as_float(row_from_above(__float_as_uint(sorted)));
    const uint64_t ends = __ballot(j < K - 1 && sorted < above);
    const uint32_t mine = (uint32_t)(ends >> (threadIdx.x & 48)) & 0xffffu;
    const uint32_t up = mine >> j, down = mine & ((1u << j) - 1u);
    have_hi = up != 0;
    const int next = (j + __ffs(up)) & 15, first = 32 - __clz(down);
    const float larger = from_row_lane(sorted, next);  // (by all lanes: one left out would have nothing to give)
    hi = have_hi ? larger : INFINITY;
    owner_hi = from_row_lane(own, next);
    owner_lo = from_row_lane(own, first);
}

__device__ __forceinline__ uint4 load_words4(const uint32_t *p) {  // 4-byte aligned
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
// Keeps the compiler from moving the load of v past this point: it would otherwise wait for one group of
// words, or put a load under the condition of its use, and pay several trips to memory for one.
__device__ __forceinline__ void loaded(uint4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

// A channel's sums per run and records in LDS (what the removed entries add to both taken off), and where its
// place arrays lie in memory; with removed entries, also where the stretches of theirs begin.
// No key that is looked up lies in the first or the last 8 * 128 keys but one: those buckets are left out.
template <int LB, bool REM>
struct ChannelView {
    static constexpr int kLB = LB;
    static constexpr bool kRem = REM;
    static constexpr uint32_t kBuckets = 1u << (16 - LB), kFirst = (0x0400u >> LB) - 1u, kLast = (0xfbffu >> LB) + 1u;
    static constexpr uint32_t kRecs = (kLast - kFirst + 2u) & ~1u;
    static constexpr uint32_t kBytes = (520 + 8 * kRecs + (REM ? 2 * kRecs : 0) + 15u) & ~15u;
    unsigned char *at;
    const uint32_t *arr, *rem_arr, *fill;  // memory
    __device__ __forceinline__ long long *base() const { return reinterpret_cast<long long *>(at); }
    __device__ __forceinline__ uint2 *rec() const { return reinterpret_cast<uint2 *>(at + 520); }  // [bucket - kFirst]
    __device__ __forceinline__ uint16_t *rem_start() const { return reinterpret_cast<uint16_t *>(at + 520 + 8 * kRecs); }
};

// Sums of absolute differences of the bytes of a stretch of the place array (`len` words) to pl and to pl + 1,
// over the words that row r of the channel's R rows takes: whole groups of 4 words in turn, then the 0 to 3
// words after them; what a row lacks is filler, so that no lane has a condition to pass.  AHEAD groups are on
// their way at a time.
template <int R, int AHEAD>
struct Stretch {
    const uint32_t *src, *fill;
    uint32_t len, r;
    uint4 tail, x[AHEAD];
    __device__ __forceinline__ const uint32_t *group(uint32_t q) const { return q < (len >> 2) ? src + 4 * q : fill; }
    __device__ __forceinline__ void fetch(const uint32_t *from, uint32_t n_words, uint32_t row, const uint32_t *filler) {
        src = from, len = n_words, r = row, fill = filler;
        tail = load_words4((len & 3u) ? src + (len & ~3u) : fill);
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; ++u) x[u] = load_words4(group(r + u * R));
    }
    __device__ __forceinline__ void wait() {
        loaded(tail);
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; ++u) loaded(x[u]);
    }
    // N bytes are looked at in all rows together.  Leaves the first groups in place: the sums can be taken again
    // for another pl.
    __device__ __forceinline__ void sums(uint32_t pl, uint32_t &A, uint32_t &B, uint32_t &N) const {
        const uint32_t pl4 = pl * 0x01010101u, pu4 = pl4 + 0x01010101u;
        const uint32_t m = (R == 1 || ((len >> 2) & (R - 1)) == r) ? len & 3u : 0u;
        const uint32_t end[3] = {m > 0 ? tail.x : kFill4, m > 1 ? tail.y : kFill4, m > 2 ? tail.z : kFill4};
        A = B = 0;
        auto add = [&](uint32_t v) {
            A = __builtin_amdgcn_sad_u8(v, pl4, A);
            B = __builtin_amdgcn_sad_u8(v, pu4, B);
        };
#pragma unroll
        for (int e = 0; e < 3; ++e) add(end[e]);
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; ++u) add(x[u].x), add(x[u].y), add(x[u].z), add(x[u].w);
        N = (16 * AHEAD + 12) * R;
        for (uint32_t q = AHEAD * R; __ballot(q < (len >> 2)) != 0ull; q += AHEAD * R) {
            uint4 y[AHEAD];
#pragma unroll
            for (uint32_t u = 0; u < AHEAD; ++u) y[u] = load_words4(group(q + r + u * R));
#pragma unroll
            for (uint32_t u = 0; u < AHEAD; ++u) loaded(y[u]);
#pragma unroll
            for (uint32_t u = 0; u < AHEAD; ++u) add(y[u].x), add(y[u].y), add(y[u].z), add(y[u].w);
            N += 16 * AHEAD * R;
        }
    }
};

// The stretch of one bucket, less that of the removed entries in it.
template <int R, int AHEAD, typename View>
struct BucketPlaces {
    static constexpr bool REM = View::kRem;
    Stretch<R, AHEAD> all;
    Stretch<R, 1> rem;
    bool any_rem;
    // b: the bucket, counted from kFirst
    __device__ __forceinline__ void fetch(const View &ch, uint32_t b, uint32_t x0, uint32_t x1, bool in, uint32_t r) {
        const uint32_t w0 = x0 & 0xffffu;
        all.fetch(ch.arr + (in ? w0 : 0u), in ? (x1 & 0xffffu) - w0 : 0u, r, ch.fill);
        if constexpr (REM) {
            const uint32_t v0 = ch.rem_start()[b], v1 = ch.rem_start()[b + 1];
            const uint32_t len = in ? v1 - v0 : 0u;
            any_rem = __ballot(len != 0) != 0ull;
            rem.fetch(ch.rem_arr + (len ? v0 : 0u), len, r, ch.fill);
        }
        // a copy of what was loaded first, moved up among the loads, would wait for it before the rest go out
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (REM) rem.wait();
        all.wait();
    }
    // N + D = twice the number of places at or below pl; A as in below_key.
    __device__ __forceinline__ void sums(uint32_t pl, int &A, int &D, int &N) const {
        uint32_t a, b, n;
        all.sums(pl, a, b, n);
        A = (int)a, D = (int)(b - a), N = (int)n;
        if constexpr (REM) {
            if (any_rem) {
                rem.sums(pl, a, b, n);
                A -= (int)a, D -= (int)(b - a), N -= (int)n;
            }
        }
        if constexpr (R > 1) {
            A = (int)row_group_sum<R>((uint32_t)A);
            D = (int)row_group_sum<R>((uint32_t)D);
        }
    }
};

// How many of a channel's weights have a key up to tk, and their exact sum of x * 2^24 (nothing to look up
// and both 0 where `inside` is false).  Called by all lanes.
//
// The part of a bucket at or below place pl comes from two sums of absolute differences over the
// stretch's bytes x (v_sad_u8, four bytes an instruction): with A = sum |x - pl| and B = sum |x - pl - 1|
// over N bytes, B - A = #(x <= pl) - #(x > pl), and A gives the sum of the places at or below pl once the
// sum of all bytes is known - which the records tell, filler included.  (Places and pl are at most 127, the
// filler is 128.)  Every term is linear in the bytes, so what the removed entries add is taken off term by
// term.
template <int R, int AHEAD, typename View>
__device__ __forceinline__ void below_key(const View &ch, uint32_t tk, bool inside, uint32_t r, uint32_t &n_below,
                                          long long &s_below) {
    constexpr int LB = View::kLB;
    constexpr uint32_t kPerRun = 1u << (10 - LB);  // buckets that share sign and exponent
    // a boundary key is that of a finite value: its bucket is not the last one, nor is its run of buckets
    const uint32_t b = inside ? tk >> LB : ch.kFirst, run = b / kPerRun;
    const uint2 r0 = ch.rec()[b - ch.kFirst], r1 = ch.rec()[b - ch.kFirst + 1];
    const long long base0 = ch.base()[run], base1 = ch.base()[run + 1];
    BucketPlaces<R, AHEAD, View> places;
    places.fetch(ch, b - ch.kFirst, r0.x, r1.x, inside, r);
    const int pl = (int)(tk & ((1u << LB) - 1));
    int A, D, N;
    places.sums((uint32_t)pl, A, D, N);
    const int n_b = (int)((r1.x >> 16) - (r0.x >> 16));  // places in the bucket
    const int n = (N + D) >> 1;                          // those at or below pl
    int mant;
    uint32_t sh;
    bucket_scale<LB>(b, mant, sh);
    const int u0 = (int)r0.y;
    const int u1 = (b & (kPerRun - 1)) == kPerRun - 1 ? (int)((base1 - base0) >> sh) : (int)r1.y;
    const int bytes = u1 - u0 - __mul24(mant, n_b) + 128 * (N - n_b);  // sum of all bytes
    const int l = (bytes + __mul24(pl, 2 * n - N) - A) >> 1;
    n_below = inside ? (r0.x >> 16) + (uint32_t)n : 0u;
    s_below = inside ? base0 + (long long)((unsigned long long)(long long)(u0 + __mul24(mant, n) + l) << sh) : 0ll;
}

// Start-up: level j = order statistic floor((2j+1)M/(2K)) of the kept weights.  The bucket by bisection on
// the counts below, then the place by bisection with counting scans of that bucket.
template <int R, int AHEAD, typename View>
__device__ __forceinline__ float quantile_start(const View &ch, int K, uint32_t M, uint32_t r) {
    constexpr int LB = View::kLB;
    const int p = threadIdx.x & 15;
    const bool mine = p < K && M > 0;
    const uint32_t rank = mine ? (uint32_t)(2 * p + 1) * M >> __ffs(K) : 0u;  // K is a power of two
    uint32_t b = 0;  // largest bucket with at most `rank` weights below it
#pragma unroll 1
    for (uint32_t s = View::kBuckets / 2; s > 0; s >>= 1)
        if ((ch.rec()[min(max(b + s, View::kFirst), View::kLast) - View::kFirst].x >> 16) <= rank) b += s;
    b = mine ? min(max(b, View::kFirst), View::kLast - 1u) : View::kFirst;
    const uint32_t x0 = ch.rec()[b - View::kFirst].x, x1 = ch.rec()[b - View::kFirst + 1].x, in = rank - (x0 >> 16);
    BucketPlaces<R, AHEAD, View> places;
    places.fetch(ch, b - View::kFirst, x0, x1, mine, r);
    uint32_t pl = 0;  // smallest place with more than `in` weights at or below it
#pragma unroll 1
    for (uint32_t s = (1u << LB) / 2; s > 0; s >>= 1) {
        int A, D, N;
        places.sums(pl + s - 1, A, D, N);
        if ((uint32_t)((N + D) >> 1) <= in) pl += s;
    }
    const float c = mine ? value_of_key((b << LB) | pl) : 0.0f;
    return c == 0.0f ? 0.0f : c;  // a level never starts as -0
}

// (s * 2^-24) / n in fp64, rounded once more to fp32.  The quotient by Markstein's method (Computation of elementary
// functions on the IBM RISC System/6000 processor, 1990): the reciprocal by two Newton steps from an estimate, the
// quotient from it, corrected by its remainder, exact in a fused multiply-add.  No |s| < 2^56 and 1 <= n <= 32768
// leaves the normal range (with n = 0 the value is not used).  The reciprocal is ready before the sum is.
__device__ __forceinline__ float mean_of_cell(long long s, uint32_t n) {
    const double d = ldexp((double)n, 24);
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double x = (double)s, q = x * r;
    return (float)fma(fma(-d, q, x), r, q);
}

// What the rounds leave in lane p of a row: the level at sorted position p, which level that is, the key of the
// boundary above it.
struct Rounds {
    float c_sorted;
    int own;
    uint32_t tk;
};
// Start-up (unless the caller gave the levels: lane p's is c0) and rounds of the channels whose rows of 16 lanes these
// are.  M weights take part, their sum of x * 2^24 is s_all.
template <int R, int AHEAD, typename View>
__device__ __forceinline__ Rounds run_rounds(const View &ch, int K, uint32_t M, long long s_all, bool start_given, float c0,
                                             int iters, uint32_t r) {
    const int p = threadIdx.x & 15;
    if (!start_given) {
        const float start = quantile_start<R, AHEAD>(ch, K, M, r);
        c0 = p < K ? start : INFINITY;
    }

    // lane p of a row: the level at sorted position p, which level that is, the next distinct level above it
    // (there is none for have_hi = false) and whether a weight half way belongs to the upper one
    float c_sorted, hi;
    int own;
    bool have_hi, tie_up;
    auto rank = [&](float c_level) {
        int owner_lo, owner_hi;
        rank_levels_in_rows(c_level, K, c_sorted, own, hi, owner_lo, owner_hi, have_hi);
        tie_up = owner_hi < owner_lo;
    };
    {
        // starting levels that ascend strictly (the usual outcome of the quantile start) are
        // in sorted order already: each level's upper neighbour sits one lane up
        const float c0_up = __uint_as_float(row_from_above(__float_as_uint(c0)));
        if (__ballot(p < K - 1 && !(c0 < c0_up)) == 0ull) {
            c_sorted = c0;
            own = p;
            hi = c0_up;
            have_hi = p < K - 1;
            tie_up = false;
        } else {
            rank(c0);
        }
    }
    uint32_t tk = 0xffffffffu;
#pragma unroll 1
    for (int round = 0;; ++round) {
        const uint32_t tk_prev = tk;
        tk = boundary_key(c_sorted, hi, __ballot(have_hi && tie_up) != 0ull && tie_up);
        if (!have_hi) tk = kKeyInf;
        // no boundary moved: the iteration sits on its fixed point
        if (round == iters || __ballot(p < K - 1 && tk != tk_prev) == 0ull) break;
        // cumulative count and sum at each boundary; the last position takes everything
        uint32_t n_below;
        long long s_below;
        below_key<R, AHEAD>(ch, tk, have_hi, r, n_below, s_below);
        if (!have_hi) {
            n_below = M;
            s_below = s_all;
        }
        // sorted positions live in one DPP row: neighbours come by row shifts
        const uint32_t n_cell = n_below - row_from_below(n_below);
        const long long s_cell = s_below - (long long)(((unsigned long long)row_from_below((uint32_t)((unsigned long long)s_below >> 32)) << 32) |
                                                       row_from_below((uint32_t)s_below));
        const float mean = mean_of_cell(s_cell, n_cell);
        const float c = p < K && n_cell > 0 ? mean : c_sorted;
        // usual case: the levels are still strictly ascending in the old order
        const float c_up = __uint_as_float(row_from_above(__float_as_uint(c)));
        const int own_up = (int)row_from_above((uint32_t)own);
        if (__ballot(p < K - 1 && !(c < c_up)) == 0ull) {
            c_sorted = c;
            hi = c_up;
            have_hi = p < K - 1;
            tie_up = own_up < own;
        } else {
            // bring the values back to level order and rank them again
            const float c_level = to_row_lane(c, own);
            rank(c_level);
        }
    }
    return {c_sorted, own, tk};
}
// The levels of a channel, lane p's share: why != 0 is the status of a flagged one.
__device__ __forceinline__ void store_levels(const KmArgs &a, int64_t i, int K, uint32_t why, const Rounds &res) {
    const int p = threadIdx.x & 15;
    float *crow = a.centroids + i * CMPQ_KMAX;
    if (why && p == 0 && a.status) atomicOr(a.status, (int)why);
    if (p >= K) crow[p] = INFINITY;
    else if (why) crow[p] = 0.0f;
    else crow[res.own] = res.c_sorted;
}
__device__ __forceinline__ void store_final(ChannelFinal &fin, uint32_t why, const Rounds &res) {
    const int p = threadIdx.x & 15;
    fin.tk[p] = (uint16_t)res.tk;
    fin.code_of[p] = (uint8_t)res.own;
    if (p == 0) fin.ok = why == 0;
}

// The caller's level p of channel i in lane p (infinity: no such level; -0 is taken as +0); a non-finite one raises
// `why`.
__device__ __forceinline__ float given_level(const KmArgs &a, int64_t i, int K, uint32_t &why) {
    const int p = threadIdx.x & 15;
    float c = INFINITY;
    if (a.start_given) {
        if (p < K) c = a.centroids[i * CMPQ_KMAX + p];
        const uint64_t odd = __ballot(p < K && !isfinite(c));
        if (((odd >> (threadIdx.x & 48)) & 0xffffu) && !why) why = CMPQ_STATUS_NONFINITE;
        c = c == 0.0f ? 0.0f : c;
    }
    return c;
}

// Wavefronts a SIMD that this much LDS each leaves room for (160 KiB a CU): registers are not saved for more.
constexpr int rounds_waves(uint32_t lds) { return (int)((160 * 1024 / lds + 3) / 4); }

// Start-up and rounds of 4 / R channels on one wavefront.  A channel has R rows of 16 lanes; lane p of a
// row carries the level at sorted position p and the boundary above it.  All rows of a channel hold the same
// state; they share out the words of a boundary's bucket.  Sharing a wavefront is what makes a round
// cheap: its ~200 dependent instructions per boundary key and level cost the same for one channel and for four.
// REM: `removed` holds the tables of the entries that do not take part.
// Bound by that chain: about 1400 cycles of instructions and a trip to memory for the words of a bucket (800
// cycles; the records come from LDS, 150).
template <int R, int LB, int AHEAD, bool REM>
__global__ __launch_bounds__(CMPQ_WAVE) __attribute__((amdgpu_waves_per_eu(1, rounds_waves(4 / R * ChannelView<LB, REM>::kBytes)))) void kmeans_rounds_kernel(KmArgs a, int64_t i0, int64_t n_chan,
                                                                 const unsigned char *tables, int64_t stride,
                                                                 const unsigned char *removed, ChannelFinal *fin) {
    const int lane = threadIdx.x;
    const uint32_t r = (uint32_t)((lane >> 4) & (R - 1));
    // Channels 8 apart: workgroups go to the 8 XCDs in turn, and a channel's tables are best read on the XCD that
    // built them, whose L2 may still hold them.  First and final quantization, us, neighbouring channels together
    // and 8 apart: 3001 x 1031 51 + 69 and 45 + 63, 3001 x 2049 58 + 79 and 52 + 72, 28672 x 8192 459 + 606 and
    // 455 + 595.
    const int64_t at = (int64_t)(blockIdx.x >> 3) * (8 * (4 / R)) + (blockIdx.x & 7) + (lane >> 4) / R * 8;
    const bool exists = at < n_chan;
    const int64_t j = exists ? at : n_chan - 1, i = i0 + j;
    const int b = exists ? a.bits[i] : 0;
    const bool coded = b >= 1 && b <= 4;
    if (__ballot(coded) == 0ull) {  // all kept whole in FP16
        if (exists && r == 0) a.centroids[i * CMPQ_KMAX + (lane & 15)] = INFINITY;
        return;
    }
    const TableHead *head = reinterpret_cast<const TableHead *>(tables + j * stride);
    const TableHead *rem = reinterpret_cast<const TableHead *>(REM ? removed + j * stride : nullptr);
    // ---- sums per run and records into LDS, what the removed entries add taken off.  All loads go out before
    //      the first is looked at: each trip to another kernel's output costs about 2000 cycles.
    extern __shared__ __align__(16) unsigned char dyn[];
    using View = ChannelView<LB, REM>;
    constexpr int kLanes = 16 * R, kPairs = (int)View::kRecs / 2, kHeld = (kPairs + kLanes - 1) / kLanes;
    constexpr int kRuns = (65 + kLanes - 1) / kLanes;
    const int at0 = lane & (kLanes - 1);
    View ch;
    ch.at = dyn + (lane >> 4) / R * View::kBytes;
    const uint2 *src = reinterpret_cast<const uint2 *>(head + 1), *src_rem = reinterpret_cast<const uint2 *>(rem + 1);
    ch.arr = reinterpret_cast<const uint32_t *>(src + View::kBuckets);
    ch.rem_arr = REM ? reinterpret_cast<const uint32_t *>(src_rem + View::kBuckets) : nullptr;
    ch.fill = head->fill;
    uint4 two[kHeld], two_rem[REM ? kHeld : 1];
    long long run[kRuns], run_rem[REM ? kRuns : 1];
    const uint32_t magic = head->magic, len = head->d_out, kept_all = head->kept, n_rem = REM ? rem->kept : 0u;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int s = min(at0 + u * kLanes, kPairs - 1);
        __builtin_memcpy(&two[u], src + View::kFirst + 2 * s, 16);
        if constexpr (REM) __builtin_memcpy(&two_rem[u], src_rem + View::kFirst + 2 * s, 16);
    }
#pragma unroll
    for (int u = 0; u < kRuns; ++u) {
        const int s = min(at0 + u * kLanes, 64);
        run[u] = head->base[s];
        if constexpr (REM) run_rem[u] = rem->base[s];
    }
    const bool has_rem = n_rem > 0;  // without, the removed entries' records were not written
    if (!has_rem) ch.rem_arr = ch.arr;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int s = at0 + u * kLanes;
        uint4 v = two[u];
        loaded(v);
        if constexpr (REM) {
            uint4 w = two_rem[u];
            loaded(w);
            if (!has_rem) w = make_uint4(0, 0, 0, 0);
            v.x -= w.x & 0xffff0000u, v.z -= w.z & 0xffff0000u;
            v.y -= w.y, v.w -= w.w;
            if (s < kPairs) ch.rem_start()[2 * s] = (uint16_t)w.x, ch.rem_start()[2 * s + 1] = (uint16_t)w.z;
        }
        if (s < kPairs) ch.rec()[2 * s] = make_uint2(v.x, v.y), ch.rec()[2 * s + 1] = make_uint2(v.z, v.w);
    }
#pragma unroll
    for (int u = 0; u < kRuns; ++u) {
        const int s = at0 + u * kLanes;
        if (s < 65) ch.base()[s] = REM && has_rem ? run[u] - run_rem[u] : run[u];
    }
    int K = coded ? 1 << b : 0;
    // a non-finite weight or starting level, or no usable tables: the caller's status word says so; the
    // channel gets defined outputs (all levels 0, all codes 0) instead of a clustering of NaNs
    uint32_t why = 0;
    if (coded && (magic != kTableMagic + 1u || len != (uint32_t)a.d_out))
        why = magic == kTableMagic + 2u ? CMPQ_STATUS_NONFINITE : CMPQ_STATUS_ARRANGEMENT;
    const float c0 = given_level(a, i, K, why);
    const int K_out = K;
    if (why) K = 0;
    const uint32_t M = K ? kept_all - n_rem : 0u;
    __syncthreads();
    const long long s_all = K ? ch.base()[64] : 0ll;
    const Rounds res = run_rounds<R, AHEAD>(ch, K, M, s_all, a.start_given, c0, a.iters, r);
    if (!exists || r != 0) return;
    store_levels(a, i, K_out, why, res);
    if (fin && coded) store_final(fin[j], why, res);
}

// The coding table over the buckets (many levels, long channels): a bucket with no boundary
// inside has one code; with one boundary, a code on either side of it; with more (rare) the
// entry sends the weight to the search.  An entry: byte 0 the code at or below the boundary,
// byte 1 the low byte of the boundary's key (0xff: nothing lies above it), byte 2 the code
// above it, bit 24 the flag for more than one boundary.  A key and a boundary of the same
// bucket share all bits above the place, so their low bytes compare like their places.
constexpr uint32_t kTblMulti = 0x1000000u;

template <int K, int T, int LB>
__device__ __forceinline__ int build_code_table(const uint32_t (&thr)[CMPQ_KMAX], const uint32_t *code_of,
                                                const uint32_t *tk, uint32_t *tbl, int tid) {
    constexpr int kLows = 1 << LB, kBuckets = 1 << (16 - LB);
    int multi = 0;
    for (int bk = tid; bk < kBuckets; bk += T) {
        const uint32_t first = (uint32_t)bk << LB;
        const uint32_t p0 = cell_of<K>(first, thr), p1 = cell_of<K>(first + kLows - 1, thr);
        uint32_t ent = code_of[p0] | (code_of[p1] << 16);
        if (p1 == p0) {
            ent |= 0xff00u;
        } else {
            ent |= (tk[p0] & 0xffu) << 8;
            if (p1 > p0 + 1) {
                ent |= kTblMulti;
                multi = 1;
            }
        }
        tbl[bk] = ent;
    }
    return multi;
}

// (v << 2) + base in one instruction (the compiler's own form of extract-shift-add is a
// shift, a mask and an add); base is the same in every lane.
__device__ __forceinline__ uint32_t shl2_add(uint32_t v, uint32_t base) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(r) : "v"(v), "s"(base));
    return r;
}

// LDS address (byte offset inside the workgroup's LDS) of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)reinterpret_cast<uintptr_t>(p);
}

// The table entry of the key in half `half` (0: low, 1: high) of the packed pair kk; the
// table starts at LDS address tbl_at.
template <int LB>
__device__ __forceinline__ uint32_t table_entry(uint32_t tbl_at, uint32_t kk, int half) {
    typedef const uint32_t __attribute__((address_space(3))) *LdsWord;
    const uint32_t bucket = __builtin_amdgcn_ubfe(kk, 16 * half + LB, 16 - LB);
    return *(LdsWord)(uintptr_t)shl2_add(bucket, tbl_at);
}

// The code that entry `ent` gives the same key (when its flag for several boundaries is clear).
__device__ __forceinline__ uint32_t code_from_entry(uint32_t ent, uint32_t kk, int half) {
    const uint32_t low = (kk >> (16 * half)) & 0xffu;
    return low > ((ent >> 8) & 0xffu) ? (ent >> 16) & 0xffu : ent & 0xffu;
}

// Words of the coding table (0: no number of levels uses one).
constexpr int code_table_words(int T, int G, int LB) { return G * T >= 2 * (1 << (16 - LB)) ? 1 << (16 - LB) : 0; }

struct CodeShared {
    float cent[CMPQ_KMAX];        // levels by level index
    uint32_t tk[CMPQ_KMAX];       // final boundary keys by sorted position
    uint32_t code_of[CMPQ_KMAX];  // level index that each sorted position stands for
    uint32_t flag[8];             // per wavefront
    double cent64[CMPQ_KMAX];     // levels by level index, as the error sum reads them
    double red[8];
};

// A table over the buckets replaces the search in the coding pass where there are many levels; worth it
// for long channels only.
template <int G, int K, int T, int LB>
constexpr bool kCodeTable = K >= 8 && G * T >= 2 * (1 << (16 - LB));

// The final boundaries as wave-uniform values.
template <int K>
__device__ __forceinline__ void final_boundaries(const CodeShared &sm, uint32_t (&thr)[CMPQ_KMAX]) {
    const uint32_t tk_fin = sm.tk[threadIdx.x & (CMPQ_KMAX - 1)];
#pragma unroll
    for (int p = 0; p < K - 1; ++p) thr[p] = (uint32_t)__builtin_amdgcn_readlane((int)tk_fin, p);
}

// What the coding pass needs before the channel's lanes may start on their groups: the coding table, the
// levels in fp64, zeros in the bytes of the row of the bit stream that no group writes.
template <int G, int K, int T, int LB, bool FUSED>
__device__ __forceinline__ void coding_prepare(const KmArgs &a, CodeShared &sm, unsigned char *arr, uint32_t *tbl,
                                               int tid, int n_groups) {
    if constexpr (FUSED) {
        constexpr int B = K == 2 ? 1 : (K == 4 ? 2 : (K == 8 ? 3 : 4));
        const int row_bytes = (int)(((int64_t)a.d_out * B + 31) / 32) * 4;
        const int coded = B == 4 ? 2 * n_groups : (B == 2 ? n_groups : (B == 3 ? 3 * ((n_groups + 1) >> 1) : (n_groups + 1) >> 1));
        for (int x = coded + tid; x < row_bytes; x += T) arr[x] = 0;
    }
    if constexpr (kCodeTable<G, K, T, LB>) {
        uint32_t thr[CMPQ_KMAX];
        final_boundaries<K>(sm, thr);
        const int multi = build_code_table<K, T, LB>(thr, sm.code_of, sm.tk, tbl, tid);
        const bool any = __ballot(multi) != 0ull;
        if ((tid & 63) == 0) sm.flag[tid >> 6] = any;
    }
}
template <int T>
__device__ __forceinline__ bool any_flag(const CodeShared &sm) {
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < T / CMPQ_WAVE; ++w) any |= sm.flag[w];
    return __builtin_amdgcn_readfirstlane((int)any) != 0;
}

// The coding pass with the stored format and the error folded in (Sec. 5.1; App. B.3): every
// lane takes groups g = tid, tid + T, ... of 4 weights (fetched again: the place array cannot
// give a weight's position back), finds their codes, adds (w - level)^2 in fp64 - nothing for an
// entry of O_q, whose FP16 weight is restored - and puts the group's 4 * B code bits into the
// channel's row of the bit stream, which is built in the place array the rounds no longer need.
// A rolled loop: its fp64 temporaries would not fit the register budget of the unrolled one.
// Returns the lane's share of the error.
template <int G, int K, int T, int LB, bool RAGGED>
__device__ __forceinline__ double coding_pass_fused(const KmArgs &a, int64_t i, CodeShared &sm,
                                                    unsigned char *arr, uint32_t *tbl, const uint32_t *removed,
                                                    int n_ex, int tid, int n_groups) {
    constexpr int B = K == 2 ? 1 : (K == 4 ? 2 : (K == 8 ? 3 : 4));
    constexpr bool kTable = kCodeTable<G, K, T, LB>;
    uint32_t thr[CMPQ_KMAX];
    final_boundaries<K>(sm, thr);
    const bool any_multi = kTable && any_flag<T>(sm);
    const uint32_t tbl_at = lds_address(tbl);
    const __half *wrow = static_cast<const __half *>(a.W) + i * a.ldw;
    const int d_out = (int)a.d_out;
    uint8_t *crow = a.codes ? a.codes + i * a.d_out : nullptr;
    double err = 0.0;
    const int n_steps = (n_groups + T - 1) / T;  // the same for every lane: the neighbour exchange below needs all of them
    // the weights of the next few groups are fetched while the current ones are worked on: this
    // pass may be the first to touch the row (when the tables came from an earlier run)
    constexpr int kAhead = 4;
    // two copies of the loop: only a channel that has a bucket with several boundaries (rare)
    // pays for looking at each entry's flag
    auto all_groups = [&](auto with_search) {
    constexpr bool kSearch = decltype(with_search)::value;
    uint2 nxt[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        nxt[u] = load_group<RAGGED>(wrow, u * T + tid, n_groups, d_out);
    }
#pragma unroll 1
    for (int step0 = 0; step0 < n_steps; step0 += kAhead) {
        uint2 chunk[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            chunk[u] = nxt[u];
            nxt[u] = load_group<RAGGED>(wrow, (step0 + kAhead + u) * T + tid, n_groups, d_out);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (step0 + u >= n_steps) break;  // uniform over the workgroup
            const int g = (step0 + u) * T + tid;
            const bool in = g < n_groups;
            const uint2 cur = chunk[u];
            const uint32_t kk[2] = {keys_of_half2(cur.x), keys_of_half2(cur.y)};
            uint32_t code[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (kTable) {
                    const uint32_t ent = table_entry<LB>(tbl_at, kk[e >> 1], e & 1);
                    code[e] = code_from_entry(ent, kk[e >> 1], e & 1);
                    if (kSearch && (ent & kTblMulti))
                        code[e] = sm.code_of[cell_of<K>((kk[e >> 1] >> (16 * (e & 1))) & 0xffffu, thr)];
                } else {
                    code[e] = sm.code_of[cell_of<K>((kk[e >> 1] >> (16 * (e & 1))) & 0xffffu, thr)];
                }
            }
            uint32_t word = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);  // one code per byte
            if (RAGGED && d_out - 4 * g < 4) word &= (1u << (8 * (d_out & 3))) - 1u;  // the stream ends in zeros
            if (in && crow) store_codes<RAGGED>(crow, g, d_out, word);
            // (w - level)^2 of the four entries; an entry of O_q (restored to its FP16 weight) and a
            // lane past the end add an exact zero: their difference is masked bit by bit
            uint32_t kept = in ? 0xfu : 0u;
            if ((RAGGED || n_ex > 0) && in) kept = ~(removed[g >> 3] >> ((g & 7) * 4)) & 0xfu;
            const uint32_t hw[2] = {cur.x, cur.y};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = __half2float(__ushort_as_half((unsigned short)(hw[e >> 1] >> (16 * (e & 1)))));
                const double d = (double)w - sm.cent64[code[e]];
                const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)kept, e, 1);  // all ones or zero
                const unsigned long long db = (unsigned long long)__double_as_longlong(d);
                const double dm = __longlong_as_double((long long)(((unsigned long long)(m & (uint32_t)(db >> 32)) << 32) |
                                                                   (m & (uint32_t)db)));
                err = fma(dm, dm, err);
            }
            const uint32_t f = in ? squeeze4<B>(word) : 0u;
            if constexpr (B == 4) {
                if (in) reinterpret_cast<uint16_t *>(arr)[g] = (uint16_t)f;
            } else if constexpr (B == 2) {
                if (in) arr[g] = (unsigned char)f;
            } else {
                // 12 (4) bits: an even lane joins its own with those of the lane above it (the next
                // group: T is even, so a lane's groups keep its parity) into 3 (1) whole bytes
                const uint32_t v = f | (row_from_above(f) << (4 * B));
                if (in && (tid & 1) == 0) {
                    if constexpr (B == 3) {
                        unsigned char *dst = arr + 3 * (g >> 1);
                        dst[0] = (unsigned char)v;
                        dst[1] = (unsigned char)(v >> 8);
                        dst[2] = (unsigned char)(v >> 16);
                    } else {
                        arr[g >> 1] = (unsigned char)v;
                    }
                }
            }
        }
    }
    };
    if (any_multi) all_groups(std::true_type{});
    else all_groups(std::false_type{});
    return err;
}

// Codes alone: 4 per lane and store.  The weights are fetched again (from cache) instead of being held in
// registers through the rounds.
template <int G, int K, int T, int LB, bool RAGGED>
__device__ __forceinline__ void coding_pass_plain(const KmArgs &a, int64_t i, CodeShared &sm, uint32_t *tbl,
                                                  int tid, int n_groups) {
    constexpr bool kTable = kCodeTable<G, K, T, LB>;
    uint32_t thr[CMPQ_KMAX];
    final_boundaries<K>(sm, thr);
    const bool any_multi = kTable && any_flag<T>(sm);
    const uint32_t tbl_at = lds_address(tbl);
    const __half *wrow = static_cast<const __half *>(a.W) + i * a.ldw;
    uint8_t *crow = a.codes + i * a.d_out;
    const int d_out = (int)a.d_out;
    auto all_groups = [&](auto with_search) {
        constexpr bool kSearch = decltype(with_search)::value;
#pragma unroll 4
        for (int k = 0; k < G; ++k) {
            const int g = k * T + tid;
            if (g >= n_groups) break;
            const uint2 raw = load_group<RAGGED>(wrow, g, n_groups, d_out);
            const uint32_t kk[2] = {keys_of_half2(raw.x), keys_of_half2(raw.y)};
            uint32_t word = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t key = (kk[e >> 1] >> (16 * (e & 1))) & 0xffffu;
                uint32_t code;
                if constexpr (kTable) {
                    const uint32_t ent = table_entry<LB>(tbl_at, kk[e >> 1], e & 1);
                    code = code_from_entry(ent, kk[e >> 1], e & 1);
                    if (kSearch && (ent & kTblMulti)) code = sm.code_of[cell_of<K>(key, thr)];
                } else {
                    code = sm.code_of[cell_of<K>(key, thr)];
                }
                word |= code << (8 * e);
            }
            store_codes<RAGGED>(crow, g, d_out, word);
        }
    };
    if (any_multi) all_groups(std::true_type{});
    else all_groups(std::false_type{});
}

// Codes of a channel's weights with its final boundaries, and, FUSED, the row of the stored format, the FP16
// table and the channel's error.
// tbl: LDS of the coding table; removed: of the removed-entry bitmap (MARKED: there already); arr: of the row.
template <int G, int T, int LB, bool FUSED, bool RAGGED, bool MARKED>
__device__ __forceinline__ void code_channel(const KmArgs &a, int64_t i, const ChannelFinal &f, CodeShared &sm, uint32_t *tbl,
                                             uint32_t *removed, unsigned char *arr) {
    const int tid = threadIdx.x;
    const int d_out = (int)a.d_out, n_groups = RAGGED ? (d_out + 3) >> 2 : d_out >> 2;
    const int b = a.bits[i];
    uint8_t *codes_row = a.codes ? a.codes + i * a.d_out : nullptr;
    if (b < 1 || b > 4) {  // a channel of O_act: no codes, no row; kept whole in FP16: no error
        zero_codes<RAGGED, T>(codes_row, tid, n_groups, d_out);
        if (FUSED && a.err_ch && tid == 0) a.err_ch[i] = 0.0;
        return;
    }
    const int K = 1 << b;
    // where the channel's row of the stored format goes
    uint32_t *row_dst = nullptr;
    uint16_t *lut_dst = nullptr;
    const int row_words = (int)(((int64_t)d_out * b + 31) / 32);
    if (FUSED) {
        const int32_t row = a.row_of[i];
        int j = 0;
        while (j < a.pack.n_set && a.pack.width[j] != b) ++j;
        if (row >= 0 && j < a.pack.n_set) {
            if (a.pack.packed[j]) row_dst = a.pack.packed[j] + (int64_t)row * row_words;
            if (a.pack.lut[j]) lut_dst = a.pack.lut[j] + ((int64_t)row << b);
        }
    }
    if (!f.ok) {
        zero_codes<RAGGED, T>(codes_row, tid, n_groups, d_out);
        if constexpr (FUSED) {  // the row of all-zero codes, the table of zero levels, no number for the error
            if (row_dst) for (int w = tid; w < row_words; w += T) row_dst[w] = 0;
            if (lut_dst && tid < K) lut_dst[tid] = 0;
            if (a.err_ch && tid == 0) a.err_ch[i] = __longlong_as_double(0x7ff8000000000000ll);
        }
        return;
    }
    if (tid < CMPQ_KMAX) {
        const float c = a.centroids[i * CMPQ_KMAX + tid];
        sm.tk[tid] = f.tk[tid];
        sm.code_of[tid] = f.code_of[tid];
        sm.cent[tid] = c;
        sm.cent64[tid] = (double)c;
    }
    int n_ex = 0;
    if constexpr (FUSED) {
        const int lo = a.seg ? a.seg[i] : 0;
        n_ex = a.seg ? a.seg[i + 1] - lo : 0;
        if constexpr (!MARKED) {
            if (RAGGED || n_ex > 0) {
                for (int s = tid; s < (d_out + 31) >> 5; s += T)  // what fills up the last group counts as removed
                    removed[s] = RAGGED && s == d_out >> 5 && (d_out & 3) ? ((1u << (4 - (d_out & 3))) - 1u) << (d_out & 31) : 0u;
            }
            __syncthreads();
            const int32_t chan_base = (int32_t)(i * a.d_out);
            for (int e = tid; e < n_ex; e += T) {  // entries of O_q are restored to their FP16 weight: no error
                const int o = a.out_idx[lo + e] - chan_base;
                atomicOr(&removed[o >> 5], 1u << (o & 31));
            }
        } else {
            __syncthreads();
        }
    } else {
        __syncthreads();
    }
    switch (K) {
        case 2: coding_prepare<G, 2, T, LB, FUSED>(a, sm, arr, tbl, tid, n_groups); break;
        case 4: coding_prepare<G, 4, T, LB, FUSED>(a, sm, arr, tbl, tid, n_groups); break;
        case 8: coding_prepare<G, 8, T, LB, FUSED>(a, sm, arr, tbl, tid, n_groups); break;
        default: coding_prepare<G, 16, T, LB, FUSED>(a, sm, arr, tbl, tid, n_groups); break;
    }
    __syncthreads();
    if constexpr (!FUSED) {
        switch (K) {
            case 2: coding_pass_plain<G, 2, T, LB, RAGGED>(a, i, sm, tbl, tid, n_groups); break;
            case 4: coding_pass_plain<G, 4, T, LB, RAGGED>(a, i, sm, tbl, tid, n_groups); break;
            case 8: coding_pass_plain<G, 8, T, LB, RAGGED>(a, i, sm, tbl, tid, n_groups); break;
            default: coding_pass_plain<G, 16, T, LB, RAGGED>(a, i, sm, tbl, tid, n_groups); break;
        }
    } else {
        double err;
        switch (K) {
            case 2: err = coding_pass_fused<G, 2, T, LB, RAGGED>(a, i, sm, arr, tbl, removed, n_ex, tid, n_groups); break;
            case 4: err = coding_pass_fused<G, 4, T, LB, RAGGED>(a, i, sm, arr, tbl, removed, n_ex, tid, n_groups); break;
            case 8: err = coding_pass_fused<G, 8, T, LB, RAGGED>(a, i, sm, arr, tbl, removed, n_ex, tid, n_groups); break;
            default: err = coding_pass_fused<G, 16, T, LB, RAGGED>(a, i, sm, arr, tbl, removed, n_ex, tid, n_groups); break;
        }
        // the lanes' error sums, added in a fixed order
        err = wave_sum_f64(err);
        if ((tid & 63) == 0) sm.red[tid >> 6] = err;
        __syncthreads();
        // the row is complete: copy it out, the table in FP16 beside it
        if (row_dst) {
            const uint32_t *stage = reinterpret_cast<const uint32_t *>(arr);
            for (int w = tid; w < row_words; w += T) row_dst[w] = stage[w];
        }
        if (lut_dst && tid < K) lut_dst[tid] = __half_as_ushort(__float2half_rn(sm.cent[tid]));
        if (tid == 0 && a.err_ch) {
            double t = 0.0;
            for (int w = 0; w < T / CMPQ_WAVE; ++w) t += sm.red[w];
            a.err_ch[i] = t;
        }
    }
}

template <int G, int T, int LB, bool FUSED, bool RAGGED>
__global__ __launch_bounds__(T) void kmeans_code_kernel(KmArgs a, int64_t i0, const ChannelFinal *fin) {
    // dynamic LDS: coding table | removed-entry bitmap | the row of the bit stream
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ CodeShared sm;
    uint32_t *tbl = reinterpret_cast<uint32_t *>(dyn), *removed = tbl + code_table_words(T, G, LB);
    const int n_words = FUSED ? ((int)a.d_out + 31) >> 5 : 0;
    code_channel<G, T, LB, FUSED, RAGGED, false>(a, i0 + blockIdx.x, fin[blockIdx.x], sm, tbl, removed,
                                                 reinterpret_cast<unsigned char *>(removed + ((n_words + 3) & ~3)));
}

// The same of a channel whose tables lie in LDS as they were built, nothing taken off.
template <int LB>
struct LocalView {
    static constexpr int kLB = LB;
    static constexpr bool kRem = false;
    static constexpr uint32_t kBuckets = ChannelView<LB, false>::kBuckets, kFirst = ChannelView<LB, false>::kFirst,
                              kLast = ChannelView<LB, false>::kLast;
    const TableHead *head;
    const uint32_t *arr, *fill;
    __device__ __forceinline__ const long long *base() const { return head->base; }
    __device__ __forceinline__ const uint2 *rec() const { return reinterpret_cast<const uint2 *>(head + 1) + kFirst; }
};

// Tables, start-up and rounds of a channel in one workgroup, nothing but its levels (and tables to be kept) to
// memory: for few channels or rounds, short rows, and scratch too small for the tables of many.  Kept tables are not
// taken: a channel's own are built without the removed entries, which gives the same.
//
// A round's latency is the bound, as in kmeans_rounds_kernel, but its words come from LDS and nothing has to be read
// first.  First and final quantization (with packing and error; 20 rounds), us, as three kernels and so: 1024 x 8192
// 35 + 61 -> 29 + 48, 1031 x 4099 40 + 53 -> 35 + 46, 3001 x 2049 49 + 63 -> 41 + 54, 1024 x 11008 40 + 69 -> 31 + 57,
// 512 x 28672 49 + 67 -> 38 + 65.
template <int G, int T, int LB, bool MASKED, bool RAGGED, bool FUSED>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(6))) void kmeans_channel_kernel(KmArgs a, int64_t stride) {
    // dynamic LDS: what build_tables wants (the coding pass has its row in the place array and its table in the
    // buckets' words) | head | records
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ union { BuildShared<T> build; CodeShared code; } sm;
    __shared__ ChannelFinal fin;
    constexpr int kBuckets = 1 << (16 - LB);
    static_assert(code_table_words(T, G, LB) <= kBuckets, "the coding table fits the buckets' words");
    const int64_t i = blockIdx.x;
    const int tid = threadIdx.x, b = a.bits[i];
    const int d_out = (int)a.d_out, n_words = MASKED ? (d_out + 31) >> 5 : 0;
    uint32_t *removed = reinterpret_cast<uint32_t *>(dyn + place_area_bytes<G, T, LB>(d_out));
    uint32_t *words = removed + ((n_words + 3) & ~3);
    TableHead *head = reinterpret_cast<TableHead *>(words + kBuckets);
    uint2 *rec = reinterpret_cast<uint2 *>(head + 1);
    const bool coded = b >= 1 && b <= 4;
    if (!coded && tid < CMPQ_KMAX) a.centroids[i * CMPQ_KMAX + tid] = INFINITY;
    uint32_t why = 0;  // the same for all lanes
    if (coded && a.arr_reuse) {
        const TableHead *kept = reinterpret_cast<const TableHead *>(static_cast<const unsigned char *>(a.arr_reuse) + i * stride);
        if (kept->magic != kTableMagic + 1u || kept->d_out != (uint32_t)d_out)
            why = kept->magic == kTableMagic + 2u ? CMPQ_STATUS_NONFINITE : CMPQ_STATUS_ARRANGEMENT;
    }
    if (coded && !why) {
        const int bytes = build_tables<G, T, LB, MASKED, RAGGED>(a, i, dyn, sm.build, head, rec);
        if (bytes < 0) why = CMPQ_STATUS_NONFINITE;
        __syncthreads();
        if (a.arr_keep) {
            unsigned char *to = static_cast<unsigned char *>(a.arr_keep) + i * stride;
            const int quads = (int)((why ? sizeof(TableHead) : sizeof(TableHead) + 8 * kBuckets) / 16);
            for (int s = tid; s < quads; s += T) reinterpret_cast<uint4 *>(to)[s] = reinterpret_cast<const uint4 *>(head)[s];
            if (!why) store_places<T>(to + sizeof(TableHead) + 8 * kBuckets, dyn, bytes, bucket_arr_bytes(d_out, LB));
        }
    }
    if (coded && tid < CMPQ_WAVE) {
        const int K_out = 1 << b;
        const float c0 = given_level(a, i, K_out, why);
        const int K = why ? 0 : K_out;
        const LocalView<LB> ch = {head, reinterpret_cast<const uint32_t *>(dyn), head->fill};
        // Groups of 4 words at a time: a stretch is a few words where the channel is short, and a trip to LDS is short.
        // First + final quantization with 1 / 2 / 4, us: 2000 x 300 58 / 60 / 64, 3001 x 2049 94 / 97 / 103, 2500 x 4096
        // 104 / 100 / 104, 1024 x 8192 88 / 83 / 77, 512 x 28672 116 / 107 / 101.
        constexpr int kAhead = T == 64 ? 1 : (T == 128 ? 2 : 4);
        const Rounds res = run_rounds<4, kAhead>(ch, K, K ? head->kept : 0u, K ? head->base[64] : 0ll, a.start_given, c0, a.iters,
                                            (uint32_t)(tid >> 4));
        if (tid < 16) {
            store_levels(a, i, K_out, why, res);
            store_final(fin, why, res);
        }
    }
    if (!FUSED && !a.codes) return;
    __syncthreads();  // the places are read, the levels written
    code_channel<G, T, LB, FUSED, RAGGED, MASKED>(a, i, fin, sm.code, words, removed, dyn);
}

// Dynamic LDS of a table build; the channel kernel has head and records behind it.
template <int G, int T, int LB>
size_t build_lds(int64_t d_out, bool masked) {
    size_t b = place_area_bytes<G, T, LB>(d_out);
    if (masked) b += (size_t)((((d_out + 31) >> 5) + 3) & ~3) * 4;
    return b + ((size_t)4 << (16 - LB));
}
template <int T>
constexpr size_t kChannelShared = (sizeof(BuildShared<T>) > sizeof(CodeShared) ? sizeof(BuildShared<T>) : sizeof(CodeShared)) + sizeof(ChannelFinal);
template <int LB>
constexpr size_t kLocalTables = sizeof(TableHead) + ((size_t)8 << (16 - LB));

template <typename Kern>
int allow_lds(Kern kern, size_t lds) {
    if (lds <= 64 * 1024) return CMPQ_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return CMPQ_EHIP;
    }
    return CMPQ_OK;
}

// Rows of 16 lanes per channel in the rounds (1 for channels built by 64 lanes, 2 by 128 and 256, 4 by 512).  More
// rows shorten the scan of a bucket and put more wavefronts on the chip, fewer share the rest of the chain: first
// quantization with 1 / 2 / 4 rows, us: 8192 x 1024 62 / 76 / 100, 4096 x 4096 69 / 63 / 76, 28672 x 8192 552 / 459
// / 456, 8192 x 28672 433 / 395 / 360.
// Parts of fewer channels than this leave the chip idle between their launches: the tables stay in LDS then.
constexpr int64_t kLeastPart = 2048;
template <int R, int LB, int AHEAD>
int launch_rounds(const KmArgs &a, int64_t i0, int64_t n, const unsigned char *tables, int64_t stride,
                   const unsigned char *removed, ChannelFinal *fin, hipStream_t s) {
    const unsigned grid = (unsigned)cdiv(n, 8 * (4 / R)) * 8;
    const size_t lds = 4 / R * (removed ? ChannelView<LB, true>::kBytes : ChannelView<LB, false>::kBytes);
    auto kern = removed ? kmeans_rounds_kernel<R, LB, AHEAD, true> : kmeans_rounds_kernel<R, LB, AHEAD, false>;
    if (const int rc = allow_lds(kern, lds)) return rc;
    kern<<<grid, CMPQ_WAVE, lds, s>>>(a, i0, n, tables, stride, removed, fin);
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

// Codes of channels i0 .. i0 + n from what the rounds left.
template <int G, int T, int LB>
int launch_codes(const KmArgs &a, int64_t i0, int64_t n, const ChannelFinal *fin, hipStream_t s) {
    auto kern = a.fused ? (a.ragged ? kmeans_code_kernel<G, T, LB, true, true> : kmeans_code_kernel<G, T, LB, true, false>)
                        : (a.ragged ? kmeans_code_kernel<G, T, LB, false, true> : kmeans_code_kernel<G, T, LB, false, false>);
    size_t lds = (size_t)code_table_words(T, G, LB) * 4;
    if (a.fused) lds += (size_t)((((a.d_out + 31) >> 5) + 3) & ~3) * 4 + (size_t)(a.d_out / 2 + 16);
    if (const int rc = allow_lds(kern, lds)) return rc;
    kern<<<(unsigned)n, T, lds, s>>>(a, i0, fin);
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

bool wants_codes(const KmArgs &a) { return a.codes || a.fused; }
// The removed entries have tables of their own where those of all weights are kept ones.
bool wants_removed(const KmArgs &a) { return a.arr_reuse && a.n_out > 0; }
// Scratch per channel: tables of all weights, or of the removed ones beside kept tables; what the rounds leave.
size_t scratch_per_channel(const KmArgs &a, size_t stride) {
    return ((!a.arr_keep && !a.arr_reuse) || wants_removed(a) ? stride : 0) + (wants_codes(a) ? sizeof(ChannelFinal) : 0);
}

// One quantization, `step` channels at a time.
template <int G, int T, int LB, int R>
int launch_variant(const KmArgs &a, unsigned char *scratch, int64_t step, hipStream_t s) {
    const int64_t stride = (int64_t)table_bytes(a.d_out, LB);
    ChannelFinal *fin = wants_codes(a) ? reinterpret_cast<ChannelFinal *>(scratch) : nullptr;
    unsigned char *side = scratch + (fin ? step * (int64_t)sizeof(ChannelFinal) : 0);
    for (int64_t i0 = 0; i0 < a.d_in; i0 += step) {
        const int64_t n = a.d_in - i0 < step ? a.d_in - i0 : step;
        unsigned char *tables = a.arr_keep ? static_cast<unsigned char *>(a.arr_keep) + i0 * stride : side;
        const unsigned char *src = tables;
        if (a.arr_reuse) {
            src = static_cast<const unsigned char *>(a.arr_reuse) + i0 * stride;
            if (wants_removed(a)) {
                kmeans_removed_kernel<LB><<<(unsigned)n, kRemovedLanes, 0, s>>>(a, i0, side, stride);
                CMPQ_LAUNCH_CHECK();
            }
        } else {
            const bool masked = a.n_out > 0 || a.ragged;
            auto kern = a.ragged ? kmeans_build_kernel<G, T, LB, true, true>
                                 : (masked ? kmeans_build_kernel<G, T, LB, true, false> : kmeans_build_kernel<G, T, LB, false, false>);
            const size_t lds = build_lds<G, T, LB>(a.d_out, masked);
            if (const int rc = allow_lds(kern, lds)) return rc;
            kern<<<(unsigned)n, T, lds, s>>>(a, i0, tables, stride);
            CMPQ_LAUNCH_CHECK();
        }
        if (const int rc = launch_rounds<R, LB, G == 16 ? 8 : 4>(a, i0, n, src, stride, wants_removed(a) ? side : nullptr, fin, s)) return rc;
        if (!fin) continue;
        if (const int rc = launch_codes<G, T, LB>(a, i0, n, fin, s)) return rc;
    }
    return CMPQ_OK;
}

// The same with a channel's tables in LDS alone, in one launch.
template <int G, int T, int LB, bool FUSED>
int launch_channels(const KmArgs &a, hipStream_t s) {
    const bool masked = a.n_out > 0 || a.ragged;
    auto kern = a.ragged ? kmeans_channel_kernel<G, T, LB, true, true, FUSED>
                         : (masked ? kmeans_channel_kernel<G, T, LB, true, false, FUSED> : kmeans_channel_kernel<G, T, LB, false, false, FUSED>);
    const size_t lds = build_lds<G, T, LB>(a.d_out, masked) + kLocalTables<LB>;
    if (const int rc = allow_lds(kern, lds)) return rc;
    kern<<<(unsigned)a.d_in, T, lds, s>>>(a, (int64_t)table_bytes(a.d_out, LB));
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

}  // namespace

#ifndef CMPQ_LB512
#define CMPQ_LB512 6
#endif
#ifndef CMPQ_LB256
#define CMPQ_LB256 7
#endif
namespace {

// A shape of the launches: groups of 4 weights per lane, lanes per workgroup, low bits of a key that name the
// place inside a bucket, rows of 16 lanes per channel in the rounds.
template <int G_, int T_, int LB_, int R_>
struct Shape {
    static constexpr int G = G_, T = T_, LB = LB_, R = R_;
};

// Calls f with the shape for channels of d_out weights (rows of any length: up to whole groups of 4).  A
// power-of-two workgroup of at most 512 lanes: up to 32 weights per lane, 64 for the longest channels.  LOCAL: for
// the channel kernel, whose rounds have a wavefront per channel.  CMPQ_ESHAPE: too long.
template <bool LOCAL, typename F>
int with_shape(int64_t d_out, F &&f) {
    const int64_t groups = (d_out + 3) / 4;
    int64_t T = 64;
    while (T < 512 && T * 8 < groups) T <<= 1;
    const int64_t per_lane = cdiv(groups, T);
    if (per_lane > 16) return CMPQ_ESHAPE;
    if (per_lane > 8) return f(Shape<16, 512, CMPQ_LB512, 4>{});
    if (T == 512) return f(Shape<8, 512, CMPQ_LB512, 4>{});
    if (T == 256) return f(Shape<8, 256, CMPQ_LB256, LOCAL ? 4 : 2>{});
    if (T == 128) return f(Shape<8, 128, 7, LOCAL ? 4 : 2>{});
    if (per_lane > 4) return f(Shape<8, 64, 7, LOCAL ? 4 : 1>{});
    if (per_lane > 2) return f(Shape<4, 64, 7, LOCAL ? 4 : 1>{});
    if (per_lane > 1) return f(Shape<2, 64, 7, LOCAL ? 4 : 1>{});
    return f(Shape<1, 64, 7, LOCAL ? 4 : 1>{});
}

// Bytes of a channel's tables.  0: too long.
size_t table_bytes_of(int64_t d_out) {
    size_t bytes = 0;
    (void)with_shape<false>(d_out, [&](auto s) {
        bytes = table_bytes(d_out, s.LB);
        return CMPQ_OK;
    });
    return bytes;
}

// Rows of up to this many weights are shorter than their tables' records: 262144 x 128 1121 us in three kernels, 1001 in
// the channel kernel, x 64 963 and 734, x 16 807 and 531; x 256 1309 and 1311.
constexpr int64_t kShortRow = 128;

// Whether the channel kernel takes these: few channels, all of whose workgroups the chip holds at once - 256 CUs
// of 2048 lanes (1536 where a lane takes 64 weights, by its registers) and 160 KiB of LDS, a tenth of it to spare.
// The rounds then leave wavefronts free in any case, and what the three kernels cost beyond their work - tables
// out and in again, two launches - is what counts.  Rows of up to 2048 weights share a wavefront of the rounds
// between 4 channels there and turn at 3 wavefronts a SIMD here.
//
// First and final quantization, us, three kernels and this one:
//   3000 x 300   27 + 41, 28 + 40      3300 x 2052  44 + 69, 39 + 61      2880 x 4096  47 + 75, 47 + 79
//   3500 x 300   28 + 43, 33 + 47      2500 x 4096  45 + 72, 39 + 64      2048 x 8192  49 + 74, 41 + 69
//   3000 x 1024  30 + 48, 30 + 44      672 x 28672  56 + 75, 45 + 76      1024 x 28672 64 + 88, 65 + 115
bool tables_stay_in_lds(int64_t d_in, int64_t d_out) {
    bool stay = false;
    (void)with_shape<true>(d_out, [&](auto s) {
        const size_t lds = build_lds<s.G, s.T, s.LB>(d_out, true) + kLocalTables<s.LB> + kChannelShared<s.T>;
        stay = d_in <= 256 * (s.G == 16 ? 1536 : 2048) / s.T && d_in <= 230 * (int64_t)(160 * 1024 / lds) && (s.T > 64 || d_in <= 3072);
        return CMPQ_OK;
    });
    return stay || d_out <= kShortRow;
}

// And, where tables are neither kept nor taken, up to this many rounds: what a round costs less in the three kernels
// has to make up for the tables' way out and in.  Final quantization, us, three kernels and the channel kernel:
//   4096 x 4096   5 rounds 58, 55; 10: 64, 65        4000 x 6000   10 rounds 82, 77; 20: 99, 100
//   8192 x 2048   2 rounds 65, 63;  5: 69, 72        8192 x 8192   10 rounds 163, 144; 20: 186, 188; 60: 277, 322
//   8192 x 11008  2 rounds 195, 185; 5: 206, 210     28672 x 8192   5 rounds 471, 387; 20: 584, 584
int64_t few_rounds(int64_t d_out) { return d_out > 4096 && d_out <= 8192 ? d_out / 400 : 5; }

template <typename S>
int report_shape(S, bool local, int64_t d_out, int64_t *shape) {
    constexpr int G = S::G, T = S::T, LB = S::LB;
    shape[0] = T;
    shape[1] = G;
    shape[2] = LB;
    shape[3] = (int64_t)bucket_arr_bytes(d_out, LB);
    shape[4] = (int64_t)(build_lds<G, T, LB>(d_out, true) + (local ? kLocalTables<LB> : 0));
    shape[5] = (int64_t)(local ? kChannelShared<T> : sizeof(BuildShared<T>));
    shape[6] = (int64_t)place_area_bytes<G, T, LB>(d_out);
    shape[7] = count_shift<G, T>();
    shape[8] = local ? (int64_t)kLocalTables<LB> : 0;
    return CMPQ_OK;
}

}  // namespace

size_t kmeans_hist_arrangement_stride(int64_t d_out) {
    return d_out < 4 || d_out % 4 != 0 ? 0 : table_bytes_of(d_out);
}

size_t kmeans_hist_scratch(int64_t d_in, int64_t d_out) {
    const size_t tables = d_in < 1 || d_out < 1 ? 0 : table_bytes_of(d_out);
    if (!tables) return 0;
    return tables_stay_in_lds(d_in, d_out) ? 0 : (size_t)d_in * (tables + sizeof(ChannelFinal));
}

extern "C" int cmpq_kmeans_build_shape(int64_t d_in, int64_t d_out, int64_t *shape) {
    if (!shape || d_in < 1 || d_out < 1) return CMPQ_EINVAL;
    if (tables_stay_in_lds(d_in, d_out))
        return with_shape<true>(d_out, [&](auto s) { return report_shape(s, true, d_out, shape); });
    return with_shape<false>(d_out, [&](auto s) { return report_shape(s, false, d_out, shape); });
}

extern "C" int cmpq_kmeans_launch_shape(int64_t d_out, int64_t *shape) {
    if (!shape || d_out < 4 || d_out % 4 != 0) return CMPQ_EINVAL;
    int64_t all[9];
    const int rc = cmpq_kmeans_build_shape(INT64_MAX, d_out, all);
    for (int k = 0; rc == CMPQ_OK && k < 6; ++k) shape[k] = all[k];
    return rc;
}

int launch_kmeans_hist(const KmArgs &a, void *scratch, size_t scratch_bytes, hipStream_t s) {
    unsigned char *sc = static_cast<unsigned char *>(scratch);
    const size_t stride = table_bytes_of(a.d_out), per = scratch_per_channel(a, stride);
    if (!stride) return CMPQ_ESHAPE;
    const int64_t room = per ? (int64_t)(scratch_bytes / per) : a.d_in, step = room < a.d_in ? room : a.d_in;
    const bool local = tables_stay_in_lds(a.d_in, a.d_out) || (step < a.d_in && step < kLeastPart) ||
                       (!a.arr_keep && !a.arr_reuse && a.iters <= few_rounds(a.d_out));
    cmpq_timing_before(CMPQ_KERNEL_KMEANS, s);
    const int rc = local ? with_shape<true>(a.d_out, [&](auto v) {
        return a.fused ? launch_channels<v.G, v.T, v.LB, true>(a, s) : launch_channels<v.G, v.T, v.LB, false>(a, s);
    })
                         : with_shape<false>(a.d_out, [&](auto v) { return launch_variant<v.G, v.T, v.LB, v.R>(a, sc, step, s); });
    cmpq_timing_after(CMPQ_KERNEL_KMEANS, s);
    return rc;
}
