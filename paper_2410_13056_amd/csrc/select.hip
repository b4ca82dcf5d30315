// Rankings of the CMPQ path (arXiv 2410.13056): the activation outliers O_act and
// Algorithm 1 rank d_in channel statistics; the quantization-aware outliers O_q
// (Sec. 3.2.2) rank up to d_in*d_out residuals.  All three are "the k largest
// keys, equal keys by smaller index", done with a radix select on the fp32 bit
// pattern of the non-negative key: histogram a digit, locate the digit that holds
// the k-th key, descend.  Nothing is sorted; the selected set is then written in
// index order through ordered compaction (prefix sums), so the output is unique.
#include "common.h"

namespace {

// ------------------------------------------------------------------ one workgroup, d_in keys

constexpr int kSelThreads = 1024;

struct SelShared {
    uint32_t hist[256];
    uint32_t scan[34];
    uint32_t prefix, rem;
};

__device__ __forceinline__ uint32_t stat_key(float f) {
    return f == 0.0f ? 0u : __float_as_uint(f);  // -0 -> +0; the statistic is non-negative
}

// k-th largest key among entries with skip[i] == 0 (skip nullable).  After the
// call: select key > T, and of the keys == T the first `need` in index order.
__device__ void block_kth_largest(const float *__restrict__ keys, const uint8_t *__restrict__ skip,
                                  int64_t d, uint32_t k, SelShared &sh, uint32_t &T,
                                  uint32_t &need) {
    if (k == 0) {  // nothing: no key exceeds the all-ones pattern
        T = 0xffffffffu;
        need = 0;
        return;
    }
    if (threadIdx.x == 0) {
        sh.prefix = 0;
        sh.rem = k;
    }
    uint32_t have_mask = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int b = threadIdx.x; b < 256; b += blockDim.x) sh.hist[b] = 0;
        __syncthreads();
        const uint32_t prefix = sh.prefix;
        for (int64_t i = threadIdx.x; i < d; i += blockDim.x) {
            if (skip && skip[i]) continue;
            const uint32_t key = stat_key(keys[i]);
            if ((key & have_mask) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        {
            // walk the digits from the largest down, all at once: thread t looks at digit
            // 255 - t and owns it when the rank falls inside its count
            const uint32_t rem = sh.rem;
            const uint32_t v = threadIdx.x < 256 ? sh.hist[255 - threadIdx.x] : 0u;
            uint32_t total;
            const uint32_t before = block_scan_excl_u32(v, sh.scan, &total);
            if (threadIdx.x < 256 && v && before < rem && rem <= before + v) {
                sh.rem = rem - before;  // rank inside the chosen digit
                sh.prefix = prefix | ((uint32_t)(255 - threadIdx.x) << shift);
            }
        }
        have_mask |= 255u << shift;
        __syncthreads();
    }
    T = sh.prefix;
    need = sh.rem;
    __syncthreads();
}

__global__ __launch_bounds__(kSelThreads) void top_channels_kernel(
    const float *__restrict__ sumsq, int64_t d_in, uint32_t k, int32_t *__restrict__ idx_out,
    uint8_t *__restrict__ mask_out) {
    __shared__ SelShared sh;
    uint32_t T, need;
    block_kth_largest(sumsq, nullptr, d_in, k, sh, T, need);
    uint32_t tie_base = 0, out_base = 0;
    for (int64_t base = 0; base < d_in; base += blockDim.x) {
        const int64_t i = base + threadIdx.x;
        uint32_t key = 0;
        const bool in = i < d_in;
        if (in) key = stat_key(sumsq[i]);
        const uint32_t tie = in && key == T, gt = in && key > T;
        // ties are taken in index order until `need` are in, so the number of taken ties
        // before a position is min(ties before it, need): one scan gives both offsets
        uint32_t tie_excl, gt_excl, tie_total, gt_total;
        block_scan_excl_2xu32(tie, gt, sh.scan, tie_excl, gt_excl, tie_total, gt_total);
        const uint32_t tie_rank = tie_base + tie_excl;
        const uint32_t sel = gt || (tie && tie_rank < need);
        const uint32_t pos = out_base + gt_excl + (min(tie_rank, need) - min(tie_base, need));
        if (sel && idx_out) idx_out[pos] = (int32_t)i;
        if (in && mask_out) mask_out[i] = (uint8_t)sel;
        const uint32_t sel_total = gt_total + (min(tie_base + tie_total, need) - min(tie_base, need));
        tie_base += tie_total;
        out_base += sel_total;
    }
}

// bits[i] = w_hi for the k_hi most salient unprotected channels, w_mid for the
// next ones up to rank k_mid, w_lo for the rest; CMPQ_PROTECTED where chan_mask is set.
__global__ __launch_bounds__(kSelThreads) void allocate_bits_kernel(
    const float *__restrict__ sumsq, int64_t d_in, const uint8_t *__restrict__ chan_mask,
    uint32_t k_hi, uint32_t k_mid, int all_mid, int w_hi, int w_mid, int w_lo,
    uint8_t *__restrict__ bits) {
    __shared__ SelShared sh;
    uint32_t T1, need1, T2 = 0, need2 = 0;
    block_kth_largest(sumsq, chan_mask, d_in, k_hi, sh, T1, need1);
    if (!all_mid) block_kth_largest(sumsq, chan_mask, d_in, k_mid, sh, T2, need2);
    uint32_t tie1_base = 0, tie2_base = 0;
    for (int64_t base = 0; base < d_in; base += blockDim.x) {
        const int64_t i = base + threadIdx.x;
        const bool in = i < d_in;
        const bool prot = in && chan_mask && chan_mask[i];
        const bool live = in && !prot;
        uint32_t key = 0;
        if (live) key = stat_key(sumsq[i]);
        const uint32_t tie1 = live && key == T1, tie2 = live && !all_mid && key == T2;
        uint32_t t1_excl, t2_excl, t1_total, t2_total;
        block_scan_excl_2xu32(tie1, tie2, sh.scan, t1_excl, t2_excl, t1_total, t2_total);
        const uint32_t r1 = tie1_base + t1_excl, r2 = tie2_base + t2_excl;
        if (in) {
            int w;
            if (prot)
                w = CMPQ_PROTECTED;
            else if (key > T1 || (tie1 && r1 < need1))
                w = w_hi;
            else if (all_mid || key > T2 || (tie2 && r2 < need2))
                w = w_mid;
            else
                w = w_lo;
            bits[i] = (uint8_t)w;
        }
        tie1_base += t1_total;
        tie2_base += t2_total;
    }
}

// The same two rankings for up to 8192 channels: every thread keeps PER consecutive keys in
// registers, so the statistic is read once, a digit is 11 bits (three passes, and fewer lanes on one
// counter), and the output takes one scan instead of one per 1024 channels.  These kernels are one
// workgroup's chain of dependent steps: what counts is how many there are (8192 channels: top
// channels 16.4 -> 6.8 us, allocation 20.8 -> 7.4 us; 512 threads of 16 keys 7.9 and 11.1, 256 of 32
// keys 12.2 and 17.8).  1024 threads of 32 keys, for 32768 channels, need 116 registers and waited
// 0.8 ms for a compute unit that K-means on other streams had left empty, so larger counts stay with
// the kernels above.
constexpr int kRankThreads = 1024, kRankPer = 8;

struct RankShared {
    uint32_t hist[2048];
    uint32_t scan[34];
    uint32_t prefix, rem;
};

template <int PER>
struct RankKeys {
    uint32_t key[PER];
    uint32_t live;  // bit r: entry r takes part

    __device__ __forceinline__ void load(const float *__restrict__ stat, const uint8_t *__restrict__ skip, int d) {
        const int i0 = (int)threadIdx.x * PER;
        float f[PER];
        uint8_t m[PER];
        const bool whole = i0 + PER <= d;
        if (whole && reinterpret_cast<uintptr_t>(stat) % 16 == 0) {
#pragma unroll
            for (int q = 0; q < PER / 4; ++q) {
                const float4 v = reinterpret_cast<const float4 *>(stat + i0)[q];
                f[4 * q] = v.x, f[4 * q + 1] = v.y, f[4 * q + 2] = v.z, f[4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < PER; ++r) f[r] = i0 + r < d ? stat[i0 + r] : 0.f;
        }
        if (!skip) {
#pragma unroll
            for (int r = 0; r < PER; ++r) m[r] = 0;
        } else if (whole && reinterpret_cast<uintptr_t>(skip) % 8 == 0) {
#pragma unroll
            for (int q = 0; q < PER / 8; ++q) reinterpret_cast<uint2 *>(m)[q] = reinterpret_cast<const uint2 *>(skip + i0)[q];
        } else {
#pragma unroll
            for (int r = 0; r < PER; ++r) m[r] = i0 + r < d ? skip[i0 + r] : 0;
        }
        live = 0;
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            key[r] = stat_key(f[r]);
            live |= (uint32_t)(i0 + r < d && !m[r]) << r;
        }
    }

    // block_kth_largest over the live keys.
    __device__ __forceinline__ void kth_largest(uint32_t k, RankShared &sh, uint32_t &T, uint32_t &need) const {
        if (k == 0) {  // nothing: no key exceeds the all-ones pattern
            T = 0xffffffffu;
            need = 0;
            return;
        }
        uint32_t prefix = 0, have = 0, rem = k;
#pragma unroll
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
            const uint32_t digit_mask = pass == 2 ? 1023u : 2047u;
            constexpr int kBinsPer = 2048 / kRankThreads;
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) sh.hist[threadIdx.x + q * kRankThreads] = 0;
            // a rank past the last live key falls in no digit: digit 0 and the rank stay, and every live
            // key is taken in the end, as in block_kth_largest
            if (threadIdx.x == 0) {
                sh.rem = rem;
                sh.prefix = prefix;
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if (((live >> r) & 1u) && (key[r] & have) == prefix) atomicAdd(&sh.hist[(key[r] >> shift) & digit_mask], 1u);
            __syncthreads();
            // thread t looks at the digits 2047 - 2 t and 2046 - 2 t, and owns the one the rank falls in
            const int top = 2047 - kBinsPer * (int)threadIdx.x;
            uint32_t v[kBinsPer], sum = 0, total;
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) sum += v[q] = sh.hist[top - q];
            uint32_t before = block_scan_excl_u32(sum, sh.scan, &total);
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) {
                if (before < rem && rem <= before + v[q]) {
                    sh.rem = rem - before;
                    sh.prefix = prefix | ((uint32_t)(top - q) << shift);
                }
                before += v[q];
            }
            have |= digit_mask << shift;
            __syncthreads();
            prefix = sh.prefix;
            rem = sh.rem;
            __syncthreads();
        }
        T = prefix;
        need = rem;
    }
};

// PER bytes of this thread's channels, at any alignment and up to the last channel.
template <int PER>
__device__ __forceinline__ void store_bytes(uint8_t *__restrict__ dst, const uint8_t (&v)[PER], int d) {
    const int i0 = (int)threadIdx.x * PER;
    if (i0 + PER <= d && reinterpret_cast<uintptr_t>(dst) % 8 == 0) {
#pragma unroll
        for (int q = 0; q < PER / 8; ++q) reinterpret_cast<uint2 *>(dst + i0)[q] = reinterpret_cast<const uint2 *>(v)[q];
    } else {
#pragma unroll
        for (int r = 0; r < PER; ++r)
            if (i0 + r < d) dst[i0 + r] = v[r];
    }
}

template <int PER>
__global__ __launch_bounds__(kRankThreads) void top_channels_reg_kernel(const float *__restrict__ sumsq, int d_in,
                                                                        uint32_t k, int32_t *__restrict__ idx_out,
                                                                        uint8_t *__restrict__ mask_out) {
    __shared__ RankShared sh;
    RankKeys<PER> a;
    a.load(sumsq, nullptr, d_in);
    uint32_t T, need;
    a.kth_largest(k, sh, T, need);
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const uint32_t in = (a.live >> r) & 1u;
        gt += in && a.key[r] > T;
        eq += in && a.key[r] == T;
    }
    uint32_t gt_before, eq_before, gt_all, eq_all;
    block_scan_excl_2xu32(gt, eq, sh.scan, gt_before, eq_before, gt_all, eq_all);
    // equal keys are taken in index order until `need` are in
    uint32_t pos = gt_before + min(eq_before, need);
    __align__(8) uint8_t taken[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool in = (a.live >> r) & 1u, tie = in && a.key[r] == T;
        const bool sel = (in && a.key[r] > T) || (tie && eq_before < need);
        eq_before += tie;
        if (sel && idx_out) idx_out[pos] = (int)threadIdx.x * PER + r;
        pos += sel;
        taken[r] = sel;
    }
    if (mask_out) store_bytes<PER>(mask_out, taken, d_in);
}

template <int PER>
__global__ __launch_bounds__(kRankThreads) void allocate_bits_reg_kernel(
    const float *__restrict__ sumsq, int d_in, const uint8_t *__restrict__ chan_mask, uint32_t k_hi, uint32_t k_mid,
    int all_mid, int w_hi, int w_mid, int w_lo, uint8_t *__restrict__ bits) {
    __shared__ RankShared sh;
    RankKeys<PER> a;
    a.load(sumsq, chan_mask, d_in);
    uint32_t T1, need1, T2 = 0, need2 = 0;
    a.kth_largest(k_hi, sh, T1, need1);
    if (!all_mid) a.kth_largest(k_mid, sh, T2, need2);
    uint32_t eq1 = 0, eq2 = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const uint32_t in = (a.live >> r) & 1u;
        eq1 += in && a.key[r] == T1;
        eq2 += in && !all_mid && a.key[r] == T2;
    }
    uint32_t before1, before2, all1, all2;
    block_scan_excl_2xu32(eq1, eq2, sh.scan, before1, before2, all1, all2);
    __align__(8) uint8_t w[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool in = (a.live >> r) & 1u, tie1 = in && a.key[r] == T1, tie2 = in && !all_mid && a.key[r] == T2;
        if (!in) w[r] = CMPQ_PROTECTED;
        else if (a.key[r] > T1 || (tie1 && before1 < need1)) w[r] = (uint8_t)w_hi;
        else if (all_mid || a.key[r] > T2 || (tie2 && before2 < need2)) w[r] = (uint8_t)w_mid;
        else w[r] = (uint8_t)w_lo;
        before1 += tie1;
        before2 += tie2;
    }
    store_bytes<PER>(bits, w, d_in);
}

// Both rankings in one launch (d_in <= 8192).  O_act, the channels of the wider width and those of the middle
// one are the first k[0], k[1] and k[2] channels of one order (larger key first, equal keys by index), so
// the three threshold keys come out of the same three digit passes: one histogram for the first digit, one for
// each rank after that.  A pass is a chain of barriers, so what counts is their number: 5120 channels, 1.6 us a
// digit; as two launches of three and three passes 5.9 + 6.7 us and the gap between them, now 8.1.
struct MultiShared {
    uint32_t hist[3][2048];
    uint32_t scan[34];
    uint32_t prefix[3], rem[3];
};

// RANKS = 2: every channel that is not of the wider width is of the middle one.
template <int PER, int RANKS>
__global__ __launch_bounds__(kRankThreads) void rank_channels_kernel(const float *__restrict__ sumsq, int d_in, uint3 k,
                                                                     int w_hi, int w_mid, int w_lo, int32_t *__restrict__ idx_out,
                                                                     uint8_t *__restrict__ mask_out, uint8_t *__restrict__ bits) {
    __shared__ MultiShared sh;
    RankKeys<PER> a;
    a.load(sumsq, nullptr, d_in);
    const uint32_t kk[3] = {k.x, k.y, k.z};
    uint32_t T[RANKS], need[RANKS], have = 0;
#pragma unroll
    for (int h = 0; h < RANKS; ++h) T[h] = 0, need[h] = kk[h];
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
        const uint32_t digit_mask = pass == 2 ? 1023u : 2047u;
        constexpr int kBinsPer = 2048 / kRankThreads;
        const int hists = pass == 0 ? 1 : RANKS;
#pragma unroll
        for (int h = 0; h < hists; ++h)
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) sh.hist[h][threadIdx.x + q * kRankThreads] = 0;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int h = 0; h < RANKS; ++h) sh.rem[h] = need[h], sh.prefix[h] = T[h];  // (a rank of 0 falls in no digit)
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const uint32_t digit = (a.key[r] >> shift) & digit_mask;
#pragma unroll
            for (int h = 0; h < hists; ++h)
                if (((a.live >> r) & 1u) && (a.key[r] & have) == T[h]) atomicAdd(&sh.hist[h][digit], 1u);
        }
        __syncthreads();
        // thread t looks at the digits 2047 - 2 t and 2046 - 2 t, and owns the one a rank falls in.  Counts
        // stay below 2^16: two ranks to a word of the scan.
        const int top = 2047 - kBinsPer * (int)threadIdx.x;
        uint32_t v[RANKS][kBinsPer], before[RANKS], sum[3] = {0, 0, 0};
#pragma unroll
        for (int h = 0; h < RANKS; ++h)
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) sum[h] += v[h][q] = h < hists ? sh.hist[h][top - q] : v[0][q];
        if constexpr (RANKS == 2) {
            uint32_t total;
            const uint32_t both = block_scan_excl_u32(sum[0] | (sum[1] << 16), sh.scan, &total);
            before[0] = both & 0xffffu, before[1] = both >> 16;
        } else {
            uint32_t both, total, total2;
            block_scan_excl_2xu32(sum[0] | (sum[1] << 16), sum[2], sh.scan, both, before[2], total, total2);
            before[0] = both & 0xffffu, before[1] = both >> 16;
        }
#pragma unroll
        for (int h = 0; h < RANKS; ++h)
#pragma unroll
            for (int q = 0; q < kBinsPer; ++q) {
                if (before[h] < need[h] && need[h] <= before[h] + v[h][q]) {
                    sh.rem[h] = need[h] - before[h];
                    sh.prefix[h] = T[h] | ((uint32_t)(top - q) << shift);
                }
                before[h] += v[h][q];
            }
        have |= digit_mask << shift;
        __syncthreads();
#pragma unroll
        for (int h = 0; h < RANKS; ++h) T[h] = sh.prefix[h], need[h] = sh.rem[h];
        __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < RANKS; ++h)
        if (kk[h] == 0) T[h] = 0xffffffffu, need[h] = 0;  // nothing: no key exceeds the all-ones pattern
    uint32_t gt = 0, eq[3] = {0, 0, 0};
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const uint32_t in = (a.live >> r) & 1u;
        gt += in && a.key[r] > T[0];
#pragma unroll
        for (int h = 0; h < RANKS; ++h) eq[h] += in && a.key[r] == T[h];
    }
    uint32_t x, y, all_x, all_y;
    block_scan_excl_2xu32(gt | (eq[0] << 16), eq[1] | (eq[2] << 16), sh.scan, x, y, all_x, all_y);
    uint32_t ties[3] = {x >> 16, y & 0xffffu, y >> 16};
    uint32_t pos = (x & 0xffffu) + min(ties[0], need[0]);
    __align__(8) uint8_t taken[PER], w[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool in = (a.live >> r) & 1u;
        bool first[RANKS];  // among the first kk[h] channels: equal keys are taken in index order until `need` are in
#pragma unroll
        for (int h = 0; h < RANKS; ++h) {
            const bool tie = in && a.key[r] == T[h];
            first[h] = (in && a.key[r] > T[h]) || (tie && ties[h] < need[h]);
            ties[h] += tie;
        }
        if (first[0] && idx_out) idx_out[pos] = (int)threadIdx.x * PER + r;
        pos += first[0];
        taken[r] = first[0];
        w[r] = (uint8_t)(first[0] ? CMPQ_PROTECTED : (first[1] ? w_hi : (RANKS < 3 || first[RANKS - 1] ? w_mid : w_lo)));
    }
    if (mask_out) store_bytes<PER>(mask_out, taken, d_in);
    store_bytes<PER>(bits, w, d_in);
}

// ------------------------------------------------------------------ whole layer, d_in*d_out keys
//
// Top-k of the scores of a whole layer, written in ascending linear index.  The data is
// shared out in wave-chunks (512 consecutive entries of one channel, 8 per lane); a unit
// is one wavefront with a contiguous run of wave-chunks, four consecutive units make a
// workgroup.
//
// Exact chain: three histogram passes over the data fix the threshold key digit by digit
// (11 + 11 + 10 bits).  The last pass also sets aside, unit by unit and in index order,
// every entry whose top 22 bits reach the prefix known by then - a superset of the answer
// a little over k entries long - and the result is written from this staging list.  When
// a unit's share of the list does not fit (many equal scores, or an unusual
// concentration), a flag sends the call down the full path: per-workgroup tables from the
// last pass and one more pass over the data.
//
// Fast chain, tried first: one histogram pass over a sample (every s-th wave-chunk) gives a
// threshold that, by the sample, some ten percent more than k entries reach.  One pass over
// the data stages every entry that reaches it; the exact k-th key is then found inside the
// list (two histograms, the first of them counted from the guess upwards, which is where it
// lies) and the answer written from the list.  Where the scores fall off a cliff between the k-th
// and the guess (as many far weights planted as are asked for), the k-th key lies beyond twice the
// guess: the first histogram's bins are coarse there, and a third one, in a kernel of the exact
// chain that would return at once, settles the last 8 bits.  The sample only guides the guess: if
// the list turns out to hold fewer than k entries or overflows, a flag is raised and the exact
// chain, whose kernels otherwise return at once, does the work.  Either way the result is the same
// set.  (4096x4096 weights, 0.52 % of them far, k = 0.5 %: 78 us; with such keys left to the
// exact chain 178; keys near the guess 73.)
//
// What bounds the chain beside the one pass over the data is its launches, 4.5 us each, and counters
// that many workgroups add to.  Nine launches (ten in large layers): one sample pass, two of the list, the second of which is
// the exact chain's first where that one runs, and no scan of the units' counts in a kernel of its own, where
// it were thirteen; 4096x4096 weights, k = 0.5 %, all kernels but the pass over the data: 102 -> 56 us
// (sample 31 -> 11, list 25 -> 15, counts and output 29 -> 12).

constexpr int kWThreads = 256;
constexpr int kWaves = kWThreads / CMPQ_WAVE;
constexpr int kWPerLane = 8;
constexpr int kWaveChunk = CMPQ_WAVE * kWPerLane;
constexpr int kMaxBlocks = 2048;
constexpr int kMaxUnits = kMaxBlocks * kWaves;
constexpr int kBins = 2048;
// Histograms: the three digits of the exact chain; the sample's, 12 bits of the key (exponent and
// 4 mantissa bits) and the sums of 8 of those; the list's first (from the guess on 1024 bins of
// 2^13 keys, twice the guess, then bins of 2^21 keys, which reach every key there is), its second
// (2^13 bins of one bin of the first, and the sums of 8 of those), and the third (the 2^8 keys of one
// bin of the second, where the first one's was a coarse one).
constexpr int kSampleShift = 19, kSampleFine = 1 << (31 - kSampleShift);
constexpr int kListShift = 13, kListFine = 1 << kListShift;
constexpr uint32_t kListNear = 1024, kListFarShift = 8;
// Additions from many workgroups to one counter go one after the other (0.13 us each across the
// chip), so the sample's and the list's first histogram are kept in kSets sets, to be added up by
// the reader.
constexpr int kSets = 4, kSampleSet = kSampleFine + kSampleFine / 8;
constexpr int kHistSample = 3 * kBins, kHistList = kHistSample + kSets * kSampleSet;
constexpr int kHistList2 = kHistList + kSets * kBins;
constexpr int kHistList2Fine = kHistList2 + kListFine / 8, kHistList3 = kHistList2Fine + kListFine;
constexpr int kHistTop = kHistList3 + (1 << kListFarShift);  // the sample's largest key, in kSets sets too
constexpr int kHistWords = kHistTop + kSets;

struct WselState {
    uint32_t T;         // final threshold key
    uint64_t need;      // ties (key == T) to take, in index order
    uint32_t overflow;  // exact chain: a unit's staging share was too small: take the full path
    // fast chain
    uint32_t fast_overflow;  // a unit's staging share was too small
    uint32_t fast_failed;    // the list does not settle the answer: the exact chain runs
    uint32_t reach;          // staged: key >= reach
    uint32_t first_key;      // the k-th key lies in the kListFine << list_shift keys from here
    uint32_t list_shift;     //   (0 or kListFarShift)
    uint64_t rem;            //   and is the rem-th largest of the list there
};

struct WselArgs {
    const void *W;
    const float *centroids;
    const uint8_t *codes;
    const uint8_t *bits;
    int64_t d_in, d_out, ldw;
    int64_t wc_per_channel, total_wc, wc_per_unit;
    int score;
    int vec_ok;  // 16-byte loads of W and 8-byte loads of codes are aligned
    unsigned long long *stage_ik;  // per unit `cap` entries: linear index << 32 | key
    uint16_t *stage_val;           //   and the entry's value as fp16 bits
    uint32_t *stage_cnt;           // entries staged per unit
    uint32_t cap;
    int64_t sample_stride, n_sample;  // sampled wave-chunks: q = j * stride, j < n_sample
    uint64_t sample_rank;             // rank in the sample that the guess aims at
};

struct WselPlan {
    int64_t wc_per_channel, total_wc, wc_per_unit;
    int nunits, nblocks;
    uint32_t cap;
    int64_t sample_stride, n_sample;
    uint64_t sample_rank;
};

WselPlan wsel_plan(int64_t d_in, int64_t d_out, int64_t k) {
    WselPlan p;
    p.wc_per_channel = cdiv(d_out, kWaveChunk);
    p.total_wc = p.wc_per_channel * d_in;
    int64_t nu = p.total_wc < kMaxUnits ? p.total_wc : kMaxUnits;
    if (nu < 1) nu = 1;
    p.wc_per_unit = cdiv(p.total_wc, nu);
    if (p.wc_per_unit < 1) p.wc_per_unit = 1;
    nu = cdiv(p.total_wc, p.wc_per_unit);
    if (nu < 1) nu = 1;
    p.nblocks = (int)cdiv(nu, kWaves);
    p.nunits = p.nblocks * kWaves;
    // four times a unit's even share of k, plus room for small inputs
    int64_t cap = 4 * cdiv(k, nu) + 256;
    if (cap > p.wc_per_unit * kWaveChunk) cap = p.wc_per_unit * kWaveChunk;
    p.cap = (uint32_t)cap;
    // sample: 4096 wave-chunks or more, a prime stride that does not divide the chunks of a
    // channel (so that every part of a channel is met); aim a margin above the sample's share
    // of k: 15 % (channels differ, a chunk is of one channel, and keys are not spread evenly inside
    // a bin), or 8 standard deviations of a count of that size if that is more
    static const int primes[] = {1021, 761, 509, 383, 251, 191, 127, 97, 73, 61, 53, 47, 43, 37, 31, 23, 19, 17, 13, 11, 7, 5, 3};
    p.sample_stride = 1;
    for (int pr : primes) {
        if ((int64_t)pr * 4096 <= p.total_wc && p.wc_per_channel % pr != 0) {
            p.sample_stride = pr;
            break;
        }
    }
    p.n_sample = cdiv(p.total_wc, p.sample_stride);
    const double ks = (double)k * (double)p.n_sample / (double)(p.total_wc > 0 ? p.total_wc : 1);
    double margin = 8.0 / __builtin_sqrt(ks > 1.0 ? ks : 1.0);
    if (margin < 0.10) margin = 0.10;
    p.sample_rank = (uint64_t)(ks * (1.0 + margin)) + 8;
    return p;
}

// Eight consecutive entries of a channel as loaded: weights and codes still packed.
template <typename TW>
struct Raw8;
template <>
struct Raw8<__half> {
    uint4 w;
    uint2 c;
};
template <>
struct Raw8<float> {
    float4 w0, w1;
    uint2 c;
};

// (o0, a lane's first output of the wave-chunk, is a 32-bit offset from the channel's row, whose
// address is the same in every lane: loads take that address from scalar registers)
__device__ __forceinline__ uint2 fetch_codes8(const WselArgs &a, int64_t i, int o0, bool vec) {
    uint2 c = make_uint2(0, 0);
    if (!a.codes) return c;
    const uint8_t *crow = a.codes + i * a.d_out;
    const int d_out = (int)a.d_out;
    if (vec) {  // streamed: every pass over the layer reads it once
        typedef uint32_t U2 __attribute__((ext_vector_type(2)));
        const U2 nt = __builtin_nontemporal_load(reinterpret_cast<const U2 *>(crow + o0));
        return make_uint2(nt.x, nt.y);
    }
    if (o0 + 8 <= d_out) {  // at any alignment
        __builtin_memcpy(&c, crow + o0, 8);
        return c;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (o0 + j < d_out) {
            const uint32_t b = crow[o0 + j];
            if (j < 4) c.x |= b << (8 * j); else c.y |= b << (8 * (j - 4));
        }
    }
    return c;
}

__device__ __forceinline__ void fetch8(const WselArgs &a, int64_t i, int o0, Raw8<__half> &r) {
    const uint16_t *wrow = static_cast<const uint16_t *>(a.W) + i * a.ldw;
    const int d_out = (int)a.d_out;
    const bool vec = a.vec_ok && o0 + 8 <= d_out;
    if (vec) {
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        const U4 nt = __builtin_nontemporal_load(reinterpret_cast<const U4 *>(wrow + o0));
        r.w = make_uint4(nt.x, nt.y, nt.z, nt.w);
    } else if (o0 + 8 <= d_out) {  // at any alignment
        __builtin_memcpy(&r.w, wrow + o0, 16);
    } else {
        uint32_t h[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = o0 + j < d_out ? wrow[o0 + j] : 0u;
        r.w = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    }
    r.c = fetch_codes8(a, i, o0, vec);
}

__device__ __forceinline__ void fetch8(const WselArgs &a, int64_t i, int o0, Raw8<float> &r) {
    const float *wrow = static_cast<const float *>(a.W) + i * a.ldw;
    const int d_out = (int)a.d_out;
    const bool vec = a.vec_ok && o0 + 8 <= d_out;
    if (vec) {
        r.w0 = *reinterpret_cast<const float4 *>(wrow + o0);
        r.w1 = *reinterpret_cast<const float4 *>(wrow + o0 + 4);
    } else if (o0 + 8 <= d_out) {  // at any alignment
        __builtin_memcpy(&r.w0, wrow + o0, 16);
        __builtin_memcpy(&r.w1, wrow + o0 + 4, 16);
    } else {
        float f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = o0 + j < d_out ? wrow[o0 + j] : 0.f;
        r.w0 = make_float4(f[0], f[1], f[2], f[3]);
        r.w1 = make_float4(f[4], f[5], f[6], f[7]);
    }
    r.c = fetch_codes8(a, i, o0, vec);
}

__device__ __forceinline__ void unpack8(const Raw8<__half> &r, float (&wv)[8]) {
    const uint32_t w4[4] = {r.w.x, r.w.y, r.w.z, r.w.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        wv[2 * j] = __half2float(__ushort_as_half((uint16_t)w4[j]));
        // the upper half converted in place (the compiler would shift it down first)
        asm("v_cvt_f32_f16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1"
            : "=v"(wv[2 * j + 1])
            : "v"(w4[j]));
    }
}
__device__ __forceinline__ void unpack8(const Raw8<float> &r, float (&wv)[8]) {
    wv[0] = r.w0.x, wv[1] = r.w0.y, wv[2] = r.w0.z, wv[3] = r.w0.w;
    wv[4] = r.w1.x, wv[5] = r.w1.y, wv[6] = r.w1.z, wv[7] = r.w1.w;
}

// Residual scores without codes (Sec. 3.2.2 with Q(x) of Sec. 3: the preliminary quantization
// puts every weight on its nearest level, so |w - Q(w)| is the smallest |w - level| over the
// channel's levels; rounding to fp32 keeps the order, so the smallest rounded difference is the
// rounded difference to the nearest level).  `cent` holds level (lane & 15), +inf past the
// channel's K levels: the number of finite lanes among the first 16 is K.
__device__ __forceinline__ int levels_in(float cent) {
    return (int)__popcll(__ballot(cent < INFINITY) & 0xffffull);
}
__device__ __forceinline__ float min3_abs(float x, float y, float m) {
    asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(x), "v"(y));
    return m;
}
__device__ __forceinline__ float level_of_lane(float cent, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cent), k));
}
template <int K>
__device__ __forceinline__ void nearest_abs8(const float (&wv)[8], float cent, float (&m)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) m[j] = INFINITY;
#pragma unroll
    for (int k = 0; k < K; k += 2) {
        const float s0 = level_of_lane(cent, k), s1 = level_of_lane(cent, k + 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) m[j] = min3_abs(wv[j] - s0, wv[j] - s1, m[j]);
    }
}
__device__ __forceinline__ void nearest_abs8(const float (&wv)[8], float cent, float (&m)[8]) {
    switch (levels_in(cent)) {  // uniform over the wavefront
        case 2: nearest_abs8<2>(wv, cent, m); break;
        case 4: nearest_abs8<4>(wv, cent, m); break;
        case 8: nearest_abs8<8>(wv, cent, m); break;
        default: nearest_abs8<16>(wv, cent, m); break;  // lanes past K hold +inf and never win
    }
}

// Score keys of the 8 entries.  `cent` holds level (lane & 15) of the channel: the level
// of a code comes from the lane of that number (all lanes of the wavefront take part).
template <typename TW>
__device__ __forceinline__ void score_keys8(const WselArgs &a, const Raw8<TW> &r, float cent,
                                            uint32_t (&key)[8], float (&wv)[8]) {
    unpack8(r, wv);
    if (a.score != CMPQ_SCORE_RESIDUAL) {
#pragma unroll
        for (int j = 0; j < 8; ++j) key[j] = __float_as_uint(fabsf(wv[j]));
        return;
    }
    if (!a.codes) {
        float m[8];
        nearest_abs8(wv, cent, m);
#pragma unroll
        for (int j = 0; j < 8; ++j) key[j] = __float_as_uint(m[j]);
        return;
    }
    // One branch for the whole piece, so that the eight lane exchanges below are issued back to
    // back.  Four codes per word, one per byte: the byte address of lane `code` (code * 4) is a
    // bit-field extract of the word shifted up by two.
    float level[8];
    const uint32_t c4[2] = {(r.c.x & 0x0f0f0f0fu) << 2, (r.c.y & 0x0f0f0f0fu) << 2};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t at;  // written out: the compiler turns the extract back into a shift and a mask
        asm("v_bfe_u32 %0, %1, %2, 6" : "=v"(at) : "v"(c4[j >> 2]), "n"(8 * (j & 3)));
        level[j] = __int_as_float(__builtin_amdgcn_ds_bpermute((int)at, __float_as_int(cent)));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) key[j] = __float_as_uint(fabsf(wv[j] - level[j]));
}

__device__ __forceinline__ uint32_t valid8(int o0, int64_t d_out64) {
    const int d_out = (int)d_out64;
    if (o0 + 8 <= d_out) return 0xffu;
    return o0 < d_out ? (1u << (d_out - o0)) - 1u : 0u;
}

__device__ __forceinline__ bool channel_live(const WselArgs &a, int64_t i) {
    const uint8_t b = a.bits[i];
    return b >= 1 && b <= 4;
}

__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Calls body(i, o0, raw, cent) for every wave-chunk in [q0, q1) of a live channel, in order;
// o0 is this lane's first output, raw its 8 entries as loaded, cent level (lane & 15) of the
// channel.  The loads of the next wave-chunk are issued before the current one is worked on
// (two ahead was measured and is slower).
template <typename TW, typename F>
__device__ __forceinline__ void for_each_raw_chunk(const WselArgs &a, int64_t q0, int64_t q1, F &&body) {
    if (q0 >= q1) return;
    const int lane = threadIdx.x & (CMPQ_WAVE - 1);
    // (the same in every lane, but out of a division the compiler does per lane: taken back into
    // scalar registers, so that the walk over channels and wave-chunks below is scalar work)
    int64_t i = uniform_i64(q0 / a.wc_per_channel);
    int c = __builtin_amdgcn_readfirstlane((int)(q0 % a.wc_per_channel));  // a channel has at most 2^31 / 512 wave-chunks
    const int wc_per_channel = (int)a.wc_per_channel, lane0 = lane * kWPerLane;
    // (all loads at once: a channel of O_act is fetched and then dropped)
    const uint32_t bits = a.bits[i];
    float cent = a.centroids ? a.centroids[i * CMPQ_KMAX + (lane & 15)] : 0.f;
    Raw8<TW> cur, nxt = {};
    fetch8(a, i, c * kWaveChunk + lane0, cur);
    bool live = bits >= 1 && bits <= 4;
    for (int64_t q = q0; q < q1; ++q) {
        int64_t ni = i;
        int nc = c + 1;
        bool live_n = live;
        float cent_n = cent;
        if (nc == wc_per_channel) {
            nc = 0;
            ++ni;
        }
        if (q + 1 < q1) {
            if (ni != i) {
                live_n = channel_live(a, ni);
                cent_n = live_n && a.centroids ? a.centroids[ni * CMPQ_KMAX + (lane & 15)] : 0.f;
            }
            if (live_n) fetch8(a, ni, nc * kWaveChunk + lane0, nxt);
        }
        if (live) body(i, c * kWaveChunk + lane0, cur, cent);
        cur = nxt;
        i = ni;
        c = nc;
        live = live_n;
        cent = cent_n;
    }
}

// The same with the score keys formed: body(i, o0, key, wv, valid).
template <typename TW, typename F>
__device__ __forceinline__ void for_each_wave_chunk(const WselArgs &a, int64_t q0, int64_t q1, F &&body) {
    for_each_raw_chunk<TW>(a, q0, q1, [&](int64_t i, int o0, const Raw8<TW> &raw, float cent) {
        uint32_t key[8];
        float wv[8];
        score_keys8<TW>(a, raw, cent, key, wv);
        body(i, o0, key, wv, valid8(o0, a.d_out));
    });
}

// w - level in fp32 straight from a packed FP16 weight (the conversion is part of the
// instruction: a fused multiply-add w * 1 - level with an FP16 first operand, rounded once,
// which is the subtraction's own rounding).  HI picks the upper half of the word.
template <int HI>
__device__ __forceinline__ float half_minus(uint32_t packed, float level) {
    float d;
    if (HI)
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(packed), "v"(level));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(packed), "v"(level));
    return d;
}

// Signed scores of the 8 FP16 entries: w - level (residual score) or w (magnitude score); the
// ranking key of an entry is the bit pattern of the magnitude of its score.
__device__ __forceinline__ void signed_scores8(const WselArgs &a, const Raw8<__half> &r, float cent, float (&d)[8]) {
    const uint32_t w4[4] = {r.w.x, r.w.y, r.w.z, r.w.w};
    float level[8];
    if (a.score == CMPQ_SCORE_RESIDUAL && !a.codes) {  // no codes: the magnitude itself, from the nearest level
        float wv[8];
        unpack8(r, wv);
        nearest_abs8(wv, cent, d);
        return;
    }
    if (a.score == CMPQ_SCORE_RESIDUAL) {
        // one branch for the whole piece, so that the eight lane exchanges are issued back to back
        const uint32_t c4[2] = {(r.c.x & 0x0f0f0f0fu) << 2, (r.c.y & 0x0f0f0f0fu) << 2};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            uint32_t at;
            asm("v_bfe_u32 %0, %1, %2, 6" : "=v"(at) : "v"(c4[j >> 2]), "n"(8 * (j & 3)));
            level[j] = __int_as_float(__builtin_amdgcn_ds_bpermute((int)at, __float_as_int(cent)));
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) level[j] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        d[2 * j] = half_minus<0>(w4[j], level[2 * j]);
        d[2 * j + 1] = half_minus<1>(w4[j], level[2 * j + 1]);
    }
}

// Appends the entries of this wave-chunk flagged in `cand` (bit j: entry j of the lane) to
// the unit's staging list, in index order: a lane's entries follow those of the lanes
// below it.  Few lanes hold any and hardly one holds two: every lane with entries left
// stores its next one, until none is left.  Called by all lanes of the wavefront.
__device__ __forceinline__ void stage_chunk(uint32_t cand, int64_t i, int o0, int64_t d_out,
                                            const uint32_t (&key)[8], const float (&wv)[8],
                                            unsigned long long *__restrict__ stage_ik,
                                            uint16_t *__restrict__ stage_val, uint32_t cap,
                                            uint32_t &n_staged, bool &over) {
    const unsigned long long has = __ballot(cand != 0);
    if (has == 0ull) return;
    // usual case: no lane holds two - places come from the lane mask alone
    uint32_t excl, tot;
    if (__ballot((cand & (cand - 1)) != 0) == 0ull) {
        excl = __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
        tot = (uint32_t)__popcll(has);
    } else {
        const uint32_t n_cand = __popc(cand);
        const uint32_t incl = wave_scan_incl_u32(n_cand);
        tot = __shfl(incl, CMPQ_WAVE - 1, CMPQ_WAVE);
        excl = incl - n_cand;
    }
    if (n_staged + tot <= cap) {
        uint32_t pos = n_staged + excl;
        while (__ballot(cand != 0) != 0ull) {
            if (cand) {
                const int j = __ffs(cand) - 1;
                cand &= cand - 1;
                uint32_t kj = key[0];
                float wj = wv[0];
#pragma unroll
                for (int t = 1; t < 8; ++t) {
                    if (j == t) {
                        kj = key[t];
                        wj = wv[t];
                    }
                }
                stage_ik[pos] = ((unsigned long long)((uint32_t)(i * d_out) + (uint32_t)(o0 + j)) << 32) | kj;
                stage_val[pos] = __half_as_ushort(__float2half_rn(wj));
                ++pos;
            }
        }
    } else {
        over = true;
    }
    n_staged += tot;
}

// stage_chunk for FP16 input: the key of a candidate is the magnitude of its signed score d,
// its value the packed FP16 weight itself.
__device__ __forceinline__ void stage_chunk_half(uint32_t cand, int64_t i, int o0, int64_t d_out,
                                                 const float (&d)[8], const uint4 &w,
                                                 unsigned long long *__restrict__ stage_ik,
                                                 uint16_t *__restrict__ stage_val, uint32_t cap,
                                                 uint32_t &n_staged, bool &over) {
    const unsigned long long has = __ballot(cand != 0);
    if (has == 0ull) return;
    uint32_t excl, tot;
    if (__ballot((cand & (cand - 1)) != 0) == 0ull) {  // usual case: no lane holds two
        excl = __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
        tot = (uint32_t)__popcll(has);
    } else {
        const uint32_t n_cand = __popc(cand);
        const uint32_t incl = wave_scan_incl_u32(n_cand);
        tot = __shfl(incl, CMPQ_WAVE - 1, CMPQ_WAVE);
        excl = incl - n_cand;
    }
    if (n_staged + tot <= cap) {
        uint32_t pos = n_staged + excl;
        const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
        while (__ballot(cand != 0) != 0ull) {
            if (cand) {
                const int j = __ffs(cand) - 1;
                cand &= cand - 1;
                float dj = d[0];
                uint32_t wj = w4[0];
#pragma unroll
                for (int t = 1; t < 8; ++t) {
                    if (j == t) dj = d[t];
                    if ((t & 1) == 0 && (j >> 1) == (t >> 1)) wj = w4[t >> 1];
                }
                stage_ik[pos] = ((unsigned long long)((uint32_t)(i * d_out) + (uint32_t)(o0 + j)) << 32) | __float_as_uint(fabsf(dj));
                stage_val[pos] = (uint16_t)(wj >> (16 * (j & 1)));
                ++pos;
            }
        }
    } else {
        over = true;
    }
    n_staged += tot;
}

// ---- staging without codes, FP16 weights: which weights can reach the threshold at all
//
// A weight stays below the threshold t iff it is closer than t to SOME level: the weights that do
// are, level by level, a run of consecutive FP16 values around the level (the rounded difference
// grows with the distance), and the runs of a channel's levels merge into a few intervals - one,
// where the levels lie closer together than 2t.  The intervals are found once per channel, by
// bisection on the very comparison the ranking makes (|fp32(w - level)| < t), so a weight is
// inside one exactly when its score is below t; a wave-chunk is then tested with three packed
// FP16 instructions per pair of weights and interval, and only the few weights outside every
// interval get a score.

// FP16 bit pattern <-> position in the order of the values (-0 just below +0).
__device__ __forceinline__ uint32_t ord_of_half(uint32_t h) { return (h & 0x8000u) ? (~h & 0xffffu) : (h | 0x8000u); }
__device__ __forceinline__ uint32_t half_of_ord(uint32_t o) { return (o & 0x8000u) ? (o & 0x7fffu) : (~o & 0xffffu); }
constexpr uint32_t kOrdLo = 0x0400u, kOrdHi = 0xfbffu;  // -65504 and +65504: the finite values

// What safe_intervals leaves for a channel: in lanes g < n the bounds of interval g (an FP16
// pattern in both halves of a word) and the smallest and largest level whose run it holds.
struct SafeIntervals {
    int n;       // intervals; 0: none (then every weight is a candidate)
    bool whole;  // every level has a run: a weight outside the intervals has one of the levels
                 // lo_level / hi_level as its nearest
    uint32_t lo_pk, hi_pk;
    float lo_level, hi_level;
};

// The intervals of channel levels `cent` (level lane & 15 in every lane; K of them) for threshold
// t (none when t is not positive: then every weight reaches it).  Called by all lanes of the
// wavefront.
__device__ __forceinline__ SafeIntervals safe_intervals(float cent, int K, float t) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), k = lane & 15;
    // lanes 0-15: the lower end of level k's run; lanes 16-31: its upper end, searched in
    // mirrored positions (0xffff - position) so that both searches look for a first position
    const bool upper = (lane & 16) != 0, mine = lane < 32 && k < K;
    auto reached = [&](uint32_t pos) -> bool {  // at or past the end searched for
        const float v = __half2float(__ushort_as_half((uint16_t)half_of_ord(upper ? 0xffffu - pos : pos)));
        return fabsf(v - cent) < t || (upper ? v <= cent : v >= cent);
    };
    // reached(a) false or a before the finite values; reached(b) true or b past them
    uint32_t a = kOrdLo - 1, b = kOrdHi + 1;
    uint32_t guess = ord_of_half(__half_as_ushort(__float2half_rn(upper ? cent + t : cent - t)));
    if (upper) guess = 0xffffu - guess;
    guess = min(max(guess, kOrdLo + 2), kOrdHi - 2);
    if (mine) {  // two positions either side of the rounded end bracket it, but for rare roundings
        if (!reached(guess - 2)) a = guess - 2;
        if (reached(guess + 2)) b = guess + 2;
    }
    while (__ballot(mine && b - a > 1) != 0ull) {
        if (mine && b - a > 1) {
            const uint32_t mid = (a + b) >> 1;
            if (reached(mid)) b = mid; else a = mid;
        }
    }
    const uint32_t end = upper ? 0xffffu - b : b;  // first position of the run / its last
    const uint32_t first = end, last = (uint32_t)__shfl((int)end, k + 16, CMPQ_WAVE);
    // (a level that is itself an FP16 value would be "inside" at t <= 0 by the second clause above)
    const bool valid = lane < 16 && k < K && first <= last && t > 0.f;
    SafeIntervals r;
    r.whole = (int)__popcll(__ballot(valid)) == K;
    // runs in ascending order of their levels (first and last positions ascend with the level):
    // rank by counting, send to the lane of the rank
    const uint32_t cb = __float_as_uint(cent);
    const uint32_t key = valid ? cb ^ ((cb >> 31) ? 0xffffffffu : 0x80000000u) : 0xffffffffu;
    uint32_t sf = valid ? first : 0x10000u, sl = valid ? last : 0u;
    float sc = cent;
    const uint32_t key_up = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x101, 0xF, 0xF, true);  // row_shl:1
    if (__ballot(lane < 16 && k < K - 1 && key > key_up) != 0ull) {  // (levels that ascend are in place: the usual case)
        uint32_t rank = 0;
        for (int j = 0; j < K; ++j) {  // (lanes past K hold the largest key and keep their places)
            const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
            rank += (kj < key || (kj == key && j < k)) ? 1u : 0u;
        }
        if (k >= K) rank = (uint32_t)k;
        const int to = (lane < 16 ? (int)rank : lane) << 2;  // a permutation of the lanes
        sf = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)sf);
        sl = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)sl);
        sc = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(cent)));
    }
    const bool svalid = lane < 16 && sf <= 0xffffu;
    // running largest last position; a run starts a new interval when an FP16 value lies between
    uint32_t run_max = svalid ? sl : 0u;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)run_max, d, 16);
        if (k >= d) run_max = max(run_max, up);
    }
    const uint32_t before = (uint32_t)__shfl_up((int)run_max, 1, 16);
    const bool start = svalid && (lane == 0 || sf > before + 1u);
    const uint32_t smask = (uint32_t)__ballot(start) & 0xffffu, vmask = (uint32_t)__ballot(svalid) & 0xffffu;
    r.n = (int)__popc(smask);
    const int gid = (int)__popc(smask & ((2u << k) - 1u)) - 1;
    const bool stop = svalid && (((smask >> (k + 1)) & 1u) || !((vmask >> (k + 1)) & 1u));
    const int to_lo = (start ? gid : 63) << 2, to_hi = (stop ? gid : 63) << 2;
    r.lo_pk = half_of_ord((uint32_t)__builtin_amdgcn_ds_permute(to_lo, (int)sf)) * 0x10001u;
    r.hi_pk = half_of_ord((uint32_t)__builtin_amdgcn_ds_permute(to_hi, (int)run_max)) * 0x10001u;
    r.lo_level = __int_as_float(__builtin_amdgcn_ds_permute(to_lo, __float_as_int(sc)));
    r.hi_level = __int_as_float(__builtin_amdgcn_ds_permute(to_hi, __float_as_int(sc)));
    return r;
}

// The entries of the lane outside every interval: bit q for entry 2q, bit 16 + q for entry
// 2q + 1 (the two halves of word q).  0 in every lane of the wavefront in many wave-chunks.
__device__ __forceinline__ uint32_t outside_intervals8(const uint4 &w, const SafeIntervals &iv) {
    const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
    uint32_t acc[4] = {~0u, ~0u, ~0u, ~0u};  // a half stays non-zero while no interval holds it
    for (int g = 0; g < iv.n; ++g) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)iv.lo_pk, g);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)iv.hi_pk, g);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t c;  // the pair clamped into the interval: unchanged halves are inside
            asm("v_pk_max_f16 %0, %1, %2" : "=v"(c) : "v"(w4[q]), "s"(lo));
            asm("v_pk_min_f16 %0, %1, %2" : "=v"(c) : "v"(c), "s"(hi));
            const uint32_t moved = c ^ w4[q];
            if (g == 0) acc[q] = moved;
            else asm("v_pk_min_u16 %0, %1, %2" : "=v"(acc[q]) : "v"(acc[q]), "v"(moved));
        }
    }
    if (__ballot((acc[0] | acc[1] | acc[2] | acc[3]) != 0u) == 0ull) return 0u;
    uint32_t out = 0;
#pragma unroll
    for (int q = 3; q >= 0; --q) {
        uint32_t one;  // 1 in each half that is not zero
        asm("v_pk_min_u16 %0, %1, %2" : "=v"(one) : "v"(acc[q]), "v"(0x00010001u));
        out = out + out + one;
    }
    return out;
}

// The same layout for "entry j exists" (bit j of valid8).
__device__ __forceinline__ uint32_t pairs_layout(uint32_t valid) {
    uint32_t out = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) out |= (((valid >> (2 * q)) & 1u) << q) | (((valid >> (2 * q + 1)) & 1u) << (16 + q));
    return out;
}

// The smallest |w - level| over the K levels in the first lanes of `cent` (K uniform).
__device__ __forceinline__ float nearest_abs1(float w, float cent, int K) {
    float m = INFINITY;
    for (int k = 0; k < K; k += 2) m = min3_abs(w - level_of_lane(cent, k), w - level_of_lane(cent, k + 1), m);
    return m;
}

// The score of a weight outside every interval, formed by all lanes of the wavefront (the levels
// cross lanes): such a weight lies below all levels of the interval above it and above all
// levels of the one below, so its nearest level is among the intervals' end levels.
__device__ __forceinline__ float outside_score(float wf, float cent, int K, const SafeIntervals &iv) {
    if (iv.whole && iv.n > 0) {
        float key = INFINITY;
        for (int g = 0; g < iv.n; ++g)
            key = min3_abs(wf - level_of_lane(iv.lo_level, g), wf - level_of_lane(iv.hi_level, g), key);
        return key;
    }
    return nearest_abs1(wf, cent, K);
}

// stage_chunk_half for staging without codes: `cand` in the layout of outside_intervals8; the
// key of a candidate is formed here.
__device__ __forceinline__ void stage_chunk_nearest(uint32_t cand, int64_t i, int o0, int64_t d_out, const uint4 &w,
                                                    float cent, int K, const SafeIntervals &iv,
                                                    unsigned long long *__restrict__ stage_ik,
                                                    uint16_t *__restrict__ stage_val, uint32_t cap,
                                                    uint32_t &n_staged, bool &over) {
    const unsigned long long has = __ballot(cand != 0);
    if (has == 0ull) return;
    const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
    auto half_at = [&](int q, int hi) -> uint16_t {  // half `hi` of word q
        uint32_t wq = w4[0];
#pragma unroll
        for (int t = 1; t < 4; ++t)
            if (q == t) wq = w4[t];
        return (uint16_t)(wq >> (16 * hi));
    };
    const uint32_t base = (uint32_t)(i * d_out) + (uint32_t)o0;
    if (__ballot((cand & (cand - 1)) != 0) == 0ull) {  // usual case: no lane holds two
        const uint32_t tot = (uint32_t)__popcll(has);
        if (n_staged + tot <= cap) {
            const uint32_t pos = n_staged + __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
            const int bit = cand ? __ffs(cand) - 1 : 0, q = bit & 15, hi = bit >> 4;
            const uint16_t hj = half_at(q, hi);
            const float key = outside_score(__half2float(__ushort_as_half(hj)), cent, K, iv);
            if (cand) {
                stage_ik[pos] = ((unsigned long long)(base + (uint32_t)(2 * q + hi)) << 32) | __float_as_uint(key);
                stage_val[pos] = hj;
            }
        } else {
            over = true;
        }
        n_staged += tot;
        return;
    }
    const uint32_t n_cand = __popc(cand);
    const uint32_t incl = wave_scan_incl_u32(n_cand);
    const uint32_t tot = __shfl(incl, CMPQ_WAVE - 1, CMPQ_WAVE);
    if (n_staged + tot <= cap) {
        // index order inside the lane: entry 2q before 2q + 1 before 2q + 2
        uint32_t order = 0;  // bit j: entry j
#pragma unroll
        for (int q = 0; q < 4; ++q) order |= (((cand >> q) & 1u) << (2 * q)) | (((cand >> (16 + q)) & 1u) << (2 * q + 1));
        uint32_t pos = n_staged + incl - n_cand;
        while (__ballot(order != 0) != 0ull) {
            const int j = order ? __ffs(order) - 1 : 0;
            const uint16_t hj = half_at(j >> 1, j & 1);
            const float key = outside_score(__half2float(__ushort_as_half(hj)), cent, K, iv);
            if (order) {
                order &= order - 1;
                stage_ik[pos] = ((unsigned long long)(base + (uint32_t)j) << 32) | __float_as_uint(key);
                stage_val[pos] = hj;
                ++pos;
            }
        }
    } else {
        over = true;
    }
    n_staged += tot;
}

struct PickShared {
    uint32_t scan[17];
    uint32_t bin, total;
    uint64_t rem_in;
    int ok;
};

// The bin of the histogram h (2048 bins, or NBINS) that holds rank `rem`, counted from the largest
// bin down (1-based), and the rank inside that bin.  Called by all 256 threads of a workgroup
// (contains barriers); false when rem is 0 or exceeds the total.
// SETS histograms that lie `stride` words apart count together.
template <int NBINS = kBins, int SETS = 1>
__device__ __forceinline__ bool block_pick(const uint32_t *__restrict__ h, uint64_t rem, PickShared &ps,
                                           uint32_t &bin, uint64_t &rem_in, uint32_t &total, int stride = 0) {
    constexpr int kPer = NBINS / kWThreads;
    const int r0 = threadIdx.x * kPer;  // position r <-> bin NBINS - 1 - r
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        v[r] = h[NBINS - 1 - (r0 + r)];
#pragma unroll
        for (int c = 1; c < SETS; ++c) v[r] += h[c * stride + NBINS - 1 - (r0 + r)];
        sum += v[r];
    }
    uint32_t tot;
    const uint32_t before = block_scan_excl_u32(sum, ps.scan, &tot);
    if (threadIdx.x == 0) {
        ps.ok = 0;
        ps.total = tot;
        ps.bin = 0;
        ps.rem_in = 0;
    }
    __syncthreads();
    if (rem != 0 && rem <= tot) {
        uint64_t run = before;
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            if (v[r] && run < rem && rem <= run + v[r]) {
                ps.bin = (uint32_t)(NBINS - 1 - (r0 + r));
                ps.rem_in = rem - run;
                ps.ok = 1;
            }
            run += v[r];
        }
    }
    __syncthreads();
    bin = ps.bin;
    rem_in = ps.rem_in;
    total = ps.total;
    return ps.ok != 0;
}

// Exact chain: the digits fixed by the first `passes` histograms (11, 11, 10 bits from
// the top) for rank k, and the rank left inside them.  `all` when k exceeds the number of
// candidates: every candidate is taken (prefix 0).  Called by all threads of a workgroup.
__device__ __forceinline__ void exact_prefix(const uint32_t *__restrict__ hist, uint64_t k, int passes,
                                             PickShared &ps, uint32_t &prefix, uint64_t &rem, bool &all) {
    prefix = 0;
    rem = k;
    all = false;
    for (int pass = 0; pass < passes; ++pass) {
        uint32_t bin, tot;
        uint64_t rem_in;
        if (!block_pick(hist + pass * kBins, rem, ps, bin, rem_in, tot)) {
            all = true;
            prefix = 0;
            return;
        }
        prefix |= bin << (pass == 0 ? 21 : (pass == 1 ? 10 : 0));
        rem = rem_in;
    }
}

// The one of 8 neighbouring fine bins that holds rank `rem` of their sum (from the largest down) and
// the rank inside it.  Every lane for itself, so in 32 bits (a sum of the bins fits).
__device__ __forceinline__ int pick_of_8(const uint32_t *__restrict__ fine, uint32_t rem, uint64_t &rem_in) {
    uint32_t v[8], run = 0, before = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = fine[r];
    int bin = -1;
#pragma unroll
    for (int r = 7; r >= 0; --r) {
        run += v[r];
        if (bin < 0 && rem <= run) {
            bin = r;
            before = run - v[r];
        }
    }
    rem_in = rem - before;
    return bin < 0 ? 0 : bin;
}

// Fast chain, the list's digits.  First: the bin that holds the k-th key; false when the list is too
// short.
__device__ __forceinline__ uint32_t list_bin_of(uint32_t key, uint32_t reach) {  // key >= reach
    const uint32_t d = (key >> kListShift) - (reach >> kListShift);
    return d < kListNear ? d : kListNear + ((d - kListNear) >> kListFarShift);
}
static_assert(kListNear + ((0x7fffffffu >> kListShift) >> kListFarShift) < (uint32_t)kBins, "the bins reach every key");
__device__ __forceinline__ bool list_bin(const uint32_t *__restrict__ hist, uint64_t k, uint32_t reach, PickShared &ps,
                                         uint32_t &first_key, uint32_t &shift, uint64_t &rem) {
    uint32_t bin, tot;
    const bool ok = block_pick<kBins, kSets>(hist + kHistList, k, ps, bin, rem, tot, kBins);
    shift = bin < kListNear ? 0 : kListFarShift;
    first_key = ((reach >> kListShift) + (shift ? kListNear + ((bin - kListNear) << kListFarShift) : bin)) << kListShift;
    return ok;
}
// Then the key (the first of 2^shift) and how many keys equal to it (in them) are to be taken.
__device__ __forceinline__ void list_key(const uint32_t *__restrict__ hist, uint32_t first_key, uint32_t shift, uint64_t rem,
                                         PickShared &ps, uint32_t &T, uint64_t &need) {
    uint32_t bin, tot;
    uint64_t rem8;
    block_pick<kListFine / 8>(hist + kHistList2, rem, ps, bin, rem8, tot);
    T = first_key + ((8 * bin + (uint32_t)pick_of_8(hist + kHistList2Fine + 8 * bin, (uint32_t)rem8, need)) << shift);
}

// Calls body(key) for the listed entries of this workgroup's share of the units, one of `blocks`.
template <typename F>
__device__ __forceinline__ void for_each_listed(const WselArgs &a, int nunits, int blocks, F &&body) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    // 8 lanes per unit: units hold a few entries to a few hundred
    constexpr int kShare = 8;
    const int sub = lane & (kShare - 1);
    for (int64_t unit = ((int64_t)blockIdx.x * kWaves + wave) * (CMPQ_WAVE / kShare) + lane / kShare; unit < nunits;
         unit += (int64_t)blocks * (kWThreads / kShare)) {
        const unsigned long long *ik = a.stage_ik + unit * a.cap;
        const uint32_t n = a.stage_cnt[unit];
#pragma unroll 4
        for (uint32_t e = sub; e < n; e += kShare) body((uint32_t)ik[e]);
    }
}

// Adds a workgroup's fine histogram, 16 bits a counter, two to a word, to the global one, and the
// sums of 8 to the coarse one.
__device__ __forceinline__ void flush_fine(const uint32_t *lh, int n_fine, uint32_t *__restrict__ coarse,
                                           uint32_t *__restrict__ fine) {
    for (int b = threadIdx.x; b < n_fine / 8; b += (int)blockDim.x) {
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t two = lh[4 * b + r], lo = two & 0xffffu, hi = two >> 16;
            if (lo) atomicAdd(&fine[8 * b + 2 * r], lo);
            if (hi) atomicAdd(&fine[8 * b + 2 * r + 1], hi);
            sum += lo + hi;
        }
        if (sum) atomicAdd(&coarse[b], sum);
    }
}

// Fast chain, the sample: histogram of the keys' top 12 bits over every sample_stride-th wave-chunk.
// A workgroup takes at most kSampleChunks of them, so that 16 bits a counter do.
// Workgroups of 16 wavefronts: a wavefront's wave-chunks wait for memory one after the other, and a
// workgroup more is a flush more into the same counters.
constexpr int kSampleChunks = 96, kSampleThreads = 1024;
static_assert(kSampleChunks * kWaveChunk < 65536, "");
template <typename TW>
__global__ __launch_bounds__(kSampleThreads) void wsel_sample_kernel(WselArgs a, uint32_t *__restrict__ hist) {
    __shared__ uint32_t lh[kSampleFine / 2], largest;
    for (int b = threadIdx.x; b < kSampleFine / 2; b += kSampleThreads) lh[b] = 0;
    if (threadIdx.x == 0) largest = 0;
    __syncthreads();
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    constexpr int kSampleWaves = kSampleThreads / CMPQ_WAVE;
    const int64_t n_waves = (int64_t)gridDim.x * kSampleWaves;
    // few workgroups (every one ends with a flush into the same global counters), several
    // wave-chunks per wavefront, the next one's loads issued before the current one is used
    struct Item {
        int64_t i, o0;
        bool live;
        float cent;
        Raw8<TW> raw;
    };
    auto load = [&](int64_t j, Item &it) {
        const uint32_t q = (uint32_t)(j * a.sample_stride);  // total_wc is below 2^31
        it.i = q / (uint32_t)a.wc_per_channel;
        it.o0 = (int64_t)(q % (uint32_t)a.wc_per_channel) * kWaveChunk + lane * kWPerLane;
        // all loads at once: the few channels of O_act are fetched and then dropped
        it.live = channel_live(a, it.i);  // uniform over the wavefront
        fetch8(a, it.i, it.o0, it.raw);
        it.cent = a.centroids ? a.centroids[it.i * CMPQ_KMAX + (lane & 15)] : 0.f;
    };
    int64_t j = (int64_t)blockIdx.x * kSampleWaves + wave;
    uint32_t top = 0;
    Item cur = {}, nxt = {};
    if (j < a.n_sample) load(j, cur);
    for (; j < a.n_sample; j += n_waves) {
        if (j + n_waves < a.n_sample) load(j + n_waves, nxt);
        if (cur.live) {
            uint32_t key[8];
            float wv[8];
            score_keys8<TW>(a, cur.raw, cur.cent, key, wv);
            const uint32_t valid = valid8(cur.o0, a.d_out);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (!((valid >> e) & 1u)) continue;
                top = max(top, key[e]);
                const uint32_t bin = key[e] >> kSampleShift;
                atomicAdd(&lh[bin >> 1], bin & 1u ? 0x10000u : 1u);
            }
        }
        cur = nxt;
    }
    // the largest of the wavefront ends up in its last lane (steps of wave_scan_incl_u32)
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x111, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x112, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x114, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x118, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x142, 0xA, 0xF, false));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x143, 0xC, 0xF, false));
    if (lane == CMPQ_WAVE - 1) atomicMax(&largest, top);
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&hist[kHistTop + (blockIdx.x & (kSets - 1))], largest);
    uint32_t *set = hist + kHistSample + (blockIdx.x & (kSets - 1)) * kSampleSet;
    flush_fine(lh, kSampleFine, set, set + kSampleFine / 8);
}

// The guess: the key that `rank` entries of the sample reach, placed inside its fine bin.  0 where
// there is no usable sample: then everything reaches it, the list overflows and the exact chain runs.
// Called by all threads of a workgroup, every lane for itself.
//   * The topmost bin ends at the sample's largest key, not at its edge: scores with a bound, weights
//     drawn uniformly or clipped.  (4096x4096 such weights, 1 % by magnitude: 58 us, 165
//     by the edge.)
//   * Between empty bins a bin most likely holds one value, weights on a coarse grid: the whole bin.
//     (On a grid of a quarter of their deviation 58 us, 149 with a guess inside.)
//   * Elsewhere the density of the scores is taken to change evenly across the bin, as the bins beside
//     it say; with an even density the list came out short where the scores thin out quickly.
// At most infinity: as the pattern of a NaN the guess would not stand in the floats' order by which
// FP16 weights are staged, and the list would hold keys beneath it, which its histogram has no place
// for.
__device__ __forceinline__ uint32_t sample_guess(const uint32_t *__restrict__ hist, uint64_t rank, PickShared &ps) {
    uint32_t coarse, tot;
    uint64_t rem64;
    if (!block_pick<kSampleFine / 8, kSets>(hist + kHistSample, rank, ps, coarse, rem64, tot, kSampleSet)) return 0;
    const int first = 8 * (int)coarse;
    const uint32_t rem = (uint32_t)rem64;
    const uint32_t *fine = hist + kHistSample + kSampleFine / 8;
    uint32_t v[10];  // the 8 bins and one on either side (none past the ends)
    const int before = first > 0 ? first - 1 : 0, after = first + 8 < kSampleFine ? first + 8 : first + 7;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const int b = r == 0 ? before : (r == 9 ? after : first + r - 1);
        v[r] = 0;
#pragma unroll
        for (int c = 0; c < kSets; ++c) v[r] += fine[c * kSampleSet + b];
    }
    if (before == first) v[0] = 0;
    if (after < first + 8) v[9] = 0;
    uint32_t run = 0, in = 1, count = 1, below = 0, above = 0;
    int at = 0;
#pragma unroll
    for (int r = 8; r >= 1; --r) {
        run += v[r];
        if (at == 0 && rem <= run) {
            at = r;
            in = rem - (run - v[r]);
            count = v[r], below = v[r - 1], above = v[r + 1];
        }
    }
    const uint32_t lower = (uint32_t)(first - 1 + at) << kSampleShift;
    float from_top, width = (float)((1 << kSampleShift) - 1);
    if (in == rank) {
        uint32_t top = hist[kHistTop];
#pragma unroll
        for (int c = 1; c < kSets; ++c) top = max(top, hist[kHistTop + c]);
        width = (float)(top - lower);
        from_top = (float)in * __builtin_amdgcn_rcpf((float)count);
    } else if ((below | above) == 0) {
        return min(lower, 0x7f800000u);
    } else {
        // densities l at the lower edge and h at the upper one, (l + h) / 2 = count; the guess lies t
        // below the upper edge, h t + (l - h) t^2 / 2 = in
        const float n = (float)count, l0 = (float)below + n, h0 = (float)above + n;
        const float scale = 2.f * n * __builtin_amdgcn_rcpf(l0 + h0), l = l0 * scale, h = h0 * scale, i = (float)in;
        from_top = 2.f * i * __builtin_amdgcn_rcpf(h + __builtin_amdgcn_sqrtf(fmaxf(h * h + 2.f * (l - h) * i, 0.f)));
    }
    const float share = fminf(fmaxf(1.f - from_top, 0.f), 1.f);
    return min(lower + (uint32_t)(share * width), 0x7f800000u);
}

// Fast chain, the one pass over the data: stages every entry whose key reaches the guess read off
// the sample's histograms (inside a bin, by the share of its entries that lie above).
// NEAR (FP16 weights, residual score, no codes): candidates by the channel's intervals.
// At most 80 scalar registers: with more a SIMD holds a wavefront less, whatever the vector registers
// allow, and this pass lives on wavefronts in flight (8192x28672 weights, k = 1 %, whole selection:
// 236 -> 208 us, by magnitude 217 with 87 registers, 193 with 80).
template <typename TW, bool NEAR>
__global__ __launch_bounds__(kWThreads) __attribute__((amdgpu_num_sgpr(80))) void wsel_stage_kernel(WselArgs a, WselState *st,
                                                                const uint32_t *__restrict__ hist) {
    __shared__ PickShared ps;
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const int64_t unit = (int64_t)blockIdx.x * kWaves + wave;
    const int64_t q0 = unit * a.wc_per_unit;
    const int64_t q1 = min(a.total_wc, q0 + a.wc_per_unit);
    const uint32_t reach = sample_guess(hist, a.sample_rank, ps);
    if (blockIdx.x == 0 && threadIdx.x == 0) st->reach = reach;
    uint32_t n_staged = 0;
    bool over = false;
    unsigned long long *stage_ik = a.stage_ik + unit * a.cap;
    uint16_t *stage_val = a.stage_val + unit * a.cap;
    if constexpr (std::is_same<TW, __half>::value) {
        // FP16 weights: the scores stay signed floats and are compared by magnitude (the order of
        // non-negative floats is that of their bit patterns, and "not below" keeps a NaN score a
        // candidate, as its bit pattern would be), the conversion of a weight is folded into the
        // subtraction, and only a candidate's key and value are formed
        const float reach_f = __uint_as_float(reach);
        if constexpr (NEAR) {
            // no codes: per channel the intervals of weights that stay below the guess, per
            // wave-chunk the weights outside them
            int64_t have = -1;
            int K = 0;
            SafeIntervals iv = {};
            for_each_raw_chunk<TW>(a, q0, q1, [&](int64_t i, int o0, const Raw8<TW> &raw, float cent) {
                if (i != have) {
                    have = i;
                    K = levels_in(cent);
                    iv = safe_intervals(cent, K, reach_f);
                }
                uint32_t cand = outside_intervals8(raw.w, iv);
                if (o0 - lane * kWPerLane + kWaveChunk > (int)a.d_out)  // the ragged end of a channel (uniform)
                    cand &= pairs_layout(valid8(o0, a.d_out));
                stage_chunk_nearest(cand, i, o0, a.d_out, raw.w, cent, K, iv, stage_ik, stage_val, a.cap, n_staged, over);
            });
        } else
        for_each_raw_chunk<TW>(a, q0, q1, [&](int64_t i, int o0, const Raw8<TW> &raw, float cent) {
            float d[8];
            signed_scores8(a, raw, cent, d);
            uint32_t cand = 0;  // bit j: entry j reaches the guess
#pragma unroll
            for (int j = 7; j >= 0; --j) cand = cand + cand + (!(fabsf(d[j]) < reach_f) ? 1u : 0u);
            cand &= valid8(o0, a.d_out);
            stage_chunk_half(cand, i, o0, a.d_out, d, raw.w, stage_ik, stage_val, a.cap, n_staged, over);
        });
    } else {
        for_each_wave_chunk<TW>(a, q0, q1, [&](int64_t i, int o0, const uint32_t (&key)[8], const float (&wv)[8], uint32_t valid) {
            // bit j of cand: entry j exists and reaches the guess
            uint32_t cand = 0;
#pragma unroll
            for (int j = 7; j >= 0; --j) cand = cand + cand + (key[j] >= reach ? 1u : 0u);
            cand &= valid;
            stage_chunk(cand, i, o0, a.d_out, key, wv, stage_ik, stage_val, a.cap, n_staged, over);
        });
    }
    if (lane == 0) {
        a.stage_cnt[unit] = over ? 0u : n_staged;
        if (over) st->fast_overflow = 1u;
    }
}

// Exact chain, a pass over the data.  PASS 0: digit = key >> 21 (11 bits), PASS 1: (key >> 10) & 2047, PASS 2:
// key & 1023.  The last pass also stages the entries whose top 22 bits reach the prefix and leaves,
// per workgroup, how many of its keys lie above the 22-bit prefix and its own histogram
// of the last digit (what the full path needs to place its output without counting again).
// Usually there is none, so it is launched with few workgroups, each of which takes the shares
// blk = blockIdx.x, + gridDim.x, ... of the nblocks in turn.  `lh` holds kCopies * kBins counters.
template <int PASS>
constexpr int kCopies = PASS == 0 ? 4 : 1;  // the first digit is the same for most keys: copies, chosen by lane
template <typename TW, int PASS>
__device__ __forceinline__ void exact_pass(const WselArgs &a, WselState *st, uint64_t k, int nblocks, uint32_t *__restrict__ hist,
                                           uint32_t *__restrict__ above, uint32_t *__restrict__ local_last, uint32_t *lh,
                                           uint32_t *red, PickShared &ps) {
    uint32_t prefix = 0;
    {
        uint64_t rem;
        bool all;
        exact_prefix(hist, k, PASS, ps, prefix, rem, all);  // the digits the passes before this one fixed
    }
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    for (int blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        __syncthreads();  // the counters of the share before are no longer read
        for (int b = threadIdx.x; b < kCopies<PASS> * kBins; b += kWThreads) lh[b] = 0;
        __syncthreads();
        uint32_t *lh0 = lh + (lane & (kCopies<PASS> - 1)) * kBins;
        const int64_t unit = (int64_t)blk * kWaves + wave;
        const int64_t q0 = unit * a.wc_per_unit;
        const int64_t q1 = min(a.total_wc, q0 + a.wc_per_unit);
        uint32_t n_above = 0, n_staged = 0;
        bool over = false;
        unsigned long long *stage_ik = a.stage_ik + unit * a.cap;
        uint16_t *stage_val = a.stage_val + unit * a.cap;
        for_each_wave_chunk<TW>(a, q0, q1, [&](int64_t i, int o0, const uint32_t (&key)[8], const float (&wv)[8], uint32_t valid) {
            uint32_t cand = 0;  // bit j: entry j reaches the 22-bit prefix
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (!((valid >> j) & 1u)) continue;
                if (PASS == 0) {
                    atomicAdd(&lh0[key[j] >> 21], 1u);
                } else if (PASS == 1) {
                    if ((key[j] >> 21) == (prefix >> 21)) atomicAdd(&lh[(key[j] >> 10) & 2047u], 1u);
                } else {
                    if ((key[j] >> 10) == (prefix >> 10)) atomicAdd(&lh[key[j] & 1023u], 1u);
                    n_above += (key[j] >> 10) > (prefix >> 10);
                    cand |= (uint32_t)((key[j] >> 10) >= (prefix >> 10)) << j;
                }
            }
            if (PASS == 2) stage_chunk(cand, i, o0, a.d_out, key, wv, stage_ik, stage_val, a.cap, n_staged, over);
        });
        __syncthreads();
        for (int b = threadIdx.x; b < kBins; b += kWThreads) {
            uint32_t n = lh[b];
#pragma unroll
            for (int r = 1; r < kCopies<PASS>; ++r) n += lh[r * kBins + b];
            if (n) atomicAdd(&hist[PASS * kBins + b], n);
        }
        if (PASS == 2) {
            if (lane == 0) {
                a.stage_cnt[unit] = over ? 0u : n_staged;
                if (over) st->overflow = 1u;
            }
            for (int b = threadIdx.x; b < 1024; b += kWThreads) local_last[(int64_t)blk * 1024 + b] = lh[b];
            n_above = wave_sum_u32(n_above);
            if (lane == 0) red[wave] = n_above;
            __syncthreads();
            if (threadIdx.x == 0) {
                uint32_t t = 0;
                for (int w = 0; w < kWaves; ++w) t += red[w];
                above[blk] = t;
            }
        }
    }
}

// Fast chain, passes over the list: its first two histograms.  The second pass also settles whether
// the list holds the answer at all: it does unless it overflowed or is shorter than k.
// Where it does not, the second pass is the exact chain's first instead if `exact_here`: in a kernel of its own
// that one was a launch of 4 us that nearly always returned at once.  The first list_blocks workgroups go over the
// list.
template <typename TW, int PASS>
__global__ __launch_bounds__(kWThreads) void wsel_list_kernel(WselArgs a, WselState *st, int nunits, int list_blocks,
                                                               int exact_here, uint32_t *__restrict__ hist, uint64_t k) {
    constexpr int kWords = PASS == 0 ? kBins : kListFine;
    static_assert(PASS == 0 || kCopies<0> * kBins == kListFine, "both passes' counters fit");
    __shared__ uint32_t lh[kWords];
    __shared__ PickShared ps;
    for (int b = threadIdx.x; b < kWords; b += kWThreads) lh[b] = 0;
    const bool overflowed = st->fast_overflow != 0;
    const uint32_t reach = st->reach;
    uint32_t first_key = 0, shift = 0;
    if (PASS == 1) {
        uint64_t rem;
        const bool failed = !list_bin(hist, k, reach, ps, first_key, shift, rem) || overflowed;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->fast_failed = failed ? 1u : 0u;
            st->first_key = first_key;
            st->list_shift = shift;
            st->rem = rem;
        }
        if (failed) {
            if (exact_here) exact_pass<TW, 0>(a, st, k, nunits / kWaves, hist, nullptr, nullptr, lh, nullptr, ps);
            return;
        }
        if ((int)blockIdx.x >= list_blocks) return;
    } else if (overflowed) {
        return;
    }
    __syncthreads();
    for_each_listed(a, nunits, list_blocks, [&](uint32_t key) {
        if (PASS == 0) {
            atomicAdd(&lh[list_bin_of(key, reach)], 1u);
        } else {
            const uint32_t at = (key - first_key) >> shift;  // keys below the bin wrap around past it
            if (at < (uint32_t)kListFine) atomicAdd(&lh[at], 1u);
        }
    });
    __syncthreads();
    if (PASS == 0) {
        for (int b = threadIdx.x; b < kBins; b += kWThreads)
            if (lh[b]) atomicAdd(&hist[kHistList + (blockIdx.x & (kSets - 1)) * kBins + b], lh[b]);
    } else {
        for (int b = threadIdx.x; b < kListFine / 8; b += kWThreads) {
            uint32_t sum = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t v = lh[8 * b + r];
                if (v) atomicAdd(&hist[kHistList2Fine + 8 * b + r], v);
                sum += v;
            }
            if (sum) atomicAdd(&hist[kHistList2 + b], sum);
        }
    }
}

__global__ void wsel_init_kernel(WselState *st, uint32_t *hist) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < kHistWords / 4) reinterpret_cast<uint4 *>(hist)[t] = make_uint4(0, 0, 0, 0);
    if (t == 0) {
        st->T = 0;
        st->need = 0;
        st->overflow = 0;
        st->fast_overflow = 0;
        st->fast_failed = 0;
        st->reach = 0;
        st->first_key = 0;
        st->list_shift = 0;
        st->rem = 0;
    }
}

// The exact chain's passes, where the fast chain does not hold the answer.  Where that one found the
// k-th key in a coarse bin, PASS 1 counts the list's last 8 bits instead.
template <typename TW, int PASS>
__global__ __launch_bounds__(kWThreads) void wsel_hist_kernel(WselArgs a, WselState *st, uint64_t k, int nblocks,
                                                               uint32_t *__restrict__ hist,
                                                               uint32_t *__restrict__ above,
                                                               uint32_t *__restrict__ local_last) {
    __shared__ uint32_t lh[kCopies<PASS> * kBins];
    __shared__ uint32_t red[kWaves];
    __shared__ PickShared ps;
    if (!st->fast_failed) {  // the fast chain settles the answer
        const uint32_t shift = st->list_shift;
        if (PASS != 1 || shift == 0) return;
        uint32_t first;
        uint64_t rem;
        list_key(hist, st->first_key, shift, st->rem, ps, first, rem);
        static_assert(1 << kListFarShift == kWThreads, "a bin per thread");
        lh[threadIdx.x] = 0;
        __syncthreads();
        for_each_listed(a, nblocks * kWaves, (int)gridDim.x, [&](uint32_t key) {
            if (key - first < 1u << kListFarShift) atomicAdd(&lh[key - first], 1u);
        });
        __syncthreads();
        if (lh[threadIdx.x]) atomicAdd(&hist[kHistList3 + threadIdx.x], lh[threadIdx.x]);
        return;
    }
    exact_pass<TW, PASS>(a, st, k, nblocks, hist, above, local_last, lh, red, ps);
}

// Keys above the threshold and keys equal to it, per workgroup (4 units) and, from the staging list,
// per unit; on the full path per workgroup only, from the tables the last histogram pass left.
// First settles the threshold: read off the list's histograms when the fast chain holds the answer,
// else off the three histograms of the exact chain.
__global__ __launch_bounds__(kWThreads) void wsel_count_kernel(WselState *st, WselArgs a, uint64_t k,
                                                                const uint32_t *__restrict__ hist,
                                                                const uint32_t *__restrict__ above,
                                                                const uint32_t *__restrict__ local_last,
                                                                uint2 *__restrict__ cnt_unit,
                                                                uint2 *__restrict__ cnt_block) {
    __shared__ uint2 red[kWaves];
    __shared__ PickShared ps;
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    // the unit's first entries, on their way while the threshold is worked out (`cap` is 256 or more)
    const int64_t unit = (int64_t)blockIdx.x * kWaves + wave;
    const unsigned long long *ik = a.stage_ik + unit * a.cap;
    const uint32_t n = a.stage_cnt[unit], first = (uint32_t)ik[lane];
    const bool exact = st->fast_failed != 0;
    uint32_t T;
    uint64_t need;
    if (exact) {
        bool all;
        exact_prefix(hist, k, 3, ps, T, need, all);
        if (all) need = ~0ull;  // T = 0: every candidate counts
    } else {
        const uint32_t shift = st->list_shift;
        list_key(hist, st->first_key, shift, st->rem, ps, T, need);
        if (shift) {  // uniform over the launch
            uint32_t bin, tot;
            uint64_t rem = need;
            block_pick<1 << kListFarShift>(hist + kHistList3, rem, ps, bin, need, tot);
            T += bin;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->T = T;
        st->need = need;
    }
    uint32_t gt = 0, eq = 0;
    if (!exact || !st->overflow) {
        for (uint32_t e = lane; e < n; e += CMPQ_WAVE) {
            const uint32_t key = e < CMPQ_WAVE ? first : (uint32_t)ik[e];
            gt += key > T;
            eq += key == T;
        }
        gt = wave_sum_u32(gt);
        eq = wave_sum_u32(eq);
        if (lane == 0) cnt_unit[unit] = make_uint2(gt, eq);
    } else {
        const uint32_t digit = T & 1023u;
        const bool everything = need == ~0ull;  // more asked than there is: every candidate counts
        const uint32_t *h = local_last + (int64_t)blockIdx.x * 1024;
        for (int b = threadIdx.x; b < 1024; b += kWThreads)
            if (everything ? b > 0 : (uint32_t)b > digit) gt += h[b];
        gt = wave_sum_u32(gt);
        if (threadIdx.x == 0) {
            gt += above[blockIdx.x];
            eq = h[everything ? 0 : digit];
        }
    }
    if (lane == 0) red[wave] = make_uint2(gt, eq);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint2 t = red[0];
        for (int w = 1; w < kWaves; ++w) {
            t.x += red[w].x;
            t.y += red[w].y;
        }
        cnt_block[blockIdx.x] = t;
    }
}

// Keys above the threshold and equal to it before this workgroup's share, and in all of the layer
// (every workgroup adds up the at most 2048 counts for itself; contains barriers).
struct Before {
    uint32_t gt, eq, all_gt, all_eq;
};
__device__ __forceinline__ Before counts_before(const uint2 *__restrict__ cnt_block, uint32_t (*red)[4]) {
    uint32_t s[4] = {0, 0, 0, 0};
    constexpr int kPer = kMaxBlocks / kWThreads;
    uint2 c[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int b = r * kWThreads + (int)threadIdx.x;
        c[r] = b < (int)gridDim.x ? cnt_block[b] : make_uint2(0, 0);
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const bool before = r * kWThreads + (int)threadIdx.x < (int)blockIdx.x;
        s[0] += before ? c[r].x : 0u;
        s[1] += before ? c[r].y : 0u;
        s[2] += c[r].x;
        s[3] += c[r].y;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s[q] = wave_sum_u32(s[q]);
        if ((threadIdx.x & (CMPQ_WAVE - 1)) == 0) red[wave_index()][q] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s[q] = red[0][q];
        for (int w = 1; w < kWaves; ++w) s[q] += red[w][q];
    }
    return Before{s[0], s[1], s[2], s[3]};
}

__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Writes the answer from the staging list: a wavefront per unit, 64 staged entries a step.  `ties`
// and `outp`: the equal keys and the taken entries before the workgroup's units.
struct UnitList {  // what is on its way while the counts before the unit are added up
    const unsigned long long *ik;
    const uint16_t *sv;
    uint32_t n;
    unsigned long long ik0;
    uint16_t sv0;
    uint2 cnt[kWaves - 1];  // of the workgroup's units
    __device__ __forceinline__ void fetch(const WselArgs &a, const uint2 *__restrict__ cnt_unit) {
        const int lane = threadIdx.x & (CMPQ_WAVE - 1);
        const int64_t unit0 = (int64_t)blockIdx.x * kWaves, unit = unit0 + wave_index();
        ik = a.stage_ik + unit * a.cap;
        sv = a.stage_val + unit * a.cap;
        n = a.stage_cnt[unit];
        ik0 = ik[lane], sv0 = sv[lane];  // (`cap` is 256 or more)
#pragma unroll
        for (int w = 0; w < kWaves - 1; ++w) cnt[w] = cnt_unit[unit0 + w];
    }
};
__device__ __forceinline__ void emit_from_list(const UnitList &l, uint32_t T, uint64_t need, uint32_t gt_before,
                                               uint32_t eq_before, int64_t k,
                                               int32_t *__restrict__ idx_out, uint16_t *__restrict__ val_out) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w) {
        if (w < wave) {
            gt_before += l.cnt[w].x;
            eq_before += l.cnt[w].y;
        }
    }
    const uint32_t n = l.n;
    // equal keys are taken in index order until `need` are in
    uint64_t ties = eq_before, outp = gt_before + (ties < need ? ties : need);
    for (uint32_t e0 = 0; e0 < n; e0 += CMPQ_WAVE) {
        const uint32_t e = e0 + lane;
        const unsigned long long v = e0 == 0 ? l.ik0 : (e < n ? l.ik[e] : 0ull);
        const uint32_t key = (uint32_t)v;
        const bool is_eq = e < n && key == T, is_gt = e < n && key > T;
        const unsigned long long eq_mask = __ballot(is_eq);
        const bool sel = is_gt || (is_eq && ties + lanes_below(eq_mask) < need);
        const unsigned long long sel_mask = __ballot(sel);
        const uint64_t pos = outp + lanes_below(sel_mask);
        if (sel && (int64_t)pos < k) {
            idx_out[pos] = (int32_t)(v >> 32);
            if (val_out) val_out[pos] = e0 == 0 ? l.sv0 : l.sv[e];
        }
        ties += __popcll(eq_mask);
        outp += __popcll(sel_mask);
    }
}

// Writes, in index order, the selected entries of the wave-chunks [q0, q1): keys above T, and
// of the keys equal to T those whose running tie count is still below `need`.  The whole
// workgroup takes 4 wave-chunks (2048 consecutive entries) a step; `ties` and `outp` are the
// tie count and the output position before q0, positions at or beyond out_end are dropped.
template <typename TW>
__device__ __forceinline__ void write_chunks(const WselArgs &a, uint32_t T, uint64_t need, uint64_t ties,
                                             uint64_t outp, int64_t q0, int64_t q1, int64_t out_end,
                                             int32_t *__restrict__ idx_out, uint16_t *__restrict__ val_out,
                                             uint32_t *scan) {
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    for (int64_t qb = q0; qb < q1; qb += kWaves) {
        const int64_t q = qb + wave;
        const int64_t i = q / a.wc_per_channel, c = q % a.wc_per_channel;
        const int64_t o0 = c * kWaveChunk + lane * kWPerLane;
        uint32_t key[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        float wv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        uint32_t valid = 0;
        if (q < q1 && channel_live(a, i)) {  // uniform over the wavefront
            Raw8<TW> raw;
            fetch8(a, i, o0, raw);
            const float cent = a.centroids ? a.centroids[i * CMPQ_KMAX + (lane & 15)] : 0.f;
            score_keys8<TW>(a, raw, cent, key, wv);
            valid = valid8(o0, a.d_out);
        }
        uint32_t n_eq = 0, n_gt = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool v = (valid >> j) & 1u;
            n_eq += v && key[j] == T;
            n_gt += v && key[j] > T;
        }
        // ties are taken in index order until `need` are in: the number of taken ties before
        // a position is min(ties before it, need), so one scan places everything
        uint32_t eq_excl, gt_excl, eq_total, gt_total;
        block_scan_excl_2xu32(n_eq, n_gt, scan, eq_excl, gt_excl, eq_total, gt_total);
        uint64_t my_tie = ties + eq_excl;
        const uint64_t taken_before = (my_tie < need ? my_tie : need) - (ties < need ? ties : need);
        uint64_t pos = outp + gt_excl + taken_before;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (!((valid >> j) & 1u)) continue;
            bool sel = key[j] > T;
            if (key[j] == T) {
                sel = my_tie < need;
                ++my_tie;
            }
            if (sel) {
                if ((int64_t)pos < out_end) {
                    idx_out[pos] = (int32_t)(i * a.d_out + o0 + j);
                    if (val_out) val_out[pos] = __half_as_ushort(__float2half_rn(wv[j]));
                }
                ++pos;
            }
        }
        const uint64_t ties_after = ties + eq_total;
        const uint32_t sel_total =
            gt_total + (uint32_t)((ties_after < need ? ties_after : need) - (ties < need ? ties : need));
        ties += eq_total;
        outp += sel_total;
    }
}

// The last kernel of a call: from the list, unless the exact chain ran and its list overflowed: then
// with one more pass over the data, a workgroup per run of 4 units.  Where there are fewer
// candidates than asked for, the rest of idx_out is filled with -1.
// (Held to 8 wavefronts a SIMD: what is on its way for the list takes more than 96 scalar registers, which leaves 7, and
// the pass over the data then takes 331 us instead of 316 for 8192x28672 weights.)
template <typename TW>
__global__ __launch_bounds__(kWThreads, 8) void wsel_emit_kernel(WselArgs a, const WselState *st,
                                                               const uint2 *__restrict__ cnt_unit,
                                                               const uint2 *__restrict__ cnt_block,
                                                               int64_t k, int32_t *__restrict__ idx_out,
                                                               uint16_t *__restrict__ val_out) {
    __shared__ uint32_t scan[34];
    __shared__ uint32_t red[kWaves][4];
    const uint32_t T = st->T;
    const uint64_t need = st->need;
    UnitList list;
    list.fetch(a, cnt_unit);
    const Before c = counts_before(cnt_block, red);
    if (st->fast_failed && st->overflow) {
        const int64_t q0 = (int64_t)blockIdx.x * kWaves * a.wc_per_unit;
        const int64_t q1 = min(a.total_wc, q0 + kWaves * a.wc_per_unit);
        write_chunks<TW>(a, T, need, c.eq, c.gt + (c.eq < need ? (uint64_t)c.eq : need), q0, q1, k, idx_out, val_out, scan);
    } else {
        emit_from_list(list, T, need, c.gt, c.eq, k, idx_out, val_out);
    }
    const uint64_t found = c.all_gt + (c.all_eq < need ? (uint64_t)c.all_eq : need);
    for (int64_t j = (int64_t)found + (int64_t)blockIdx.x * kWThreads + threadIdx.x; j < k; j += (int64_t)gridDim.x * kWThreads)
        idx_out[j] = -1;
}

// ------------------------------------------------------------------ one channel at a time
//
// The variant of O_q with the same count in every channel: a workgroup per channel finds the
// channel's k-th largest key by the same three digits (11 + 11 + 10 bits, the keys formed
// again from the weights in every pass: a channel's row stays in cache) and writes the
// channel's k entries in index order at the place its rank among the quantized channels gives.

// rank[i] = number of channels before i with bits in 1..4.
__global__ __launch_bounds__(1024) void wsel_live_rank_kernel(const uint8_t *__restrict__ bits, int64_t d_in,
                                                              int32_t *__restrict__ rank) {
    __shared__ uint32_t scan[17];
    uint32_t run = 0;
    for (int64_t base = 0; base < d_in; base += blockDim.x) {
        const int64_t i = base + threadIdx.x;
        const uint32_t f = i < d_in && bits[i] >= 1 && bits[i] <= 4;
        uint32_t total;
        const uint32_t before = run + block_scan_excl_u32(f, scan, &total);
        if (i < d_in) rank[i] = (int32_t)before;
        run += total;
    }
}

template <typename TW>
__global__ __launch_bounds__(kWThreads) void wsel_channel_kernel(WselArgs a, const int32_t *__restrict__ live_rank,
                                                                  int64_t k, int32_t *__restrict__ idx_out,
                                                                  uint16_t *__restrict__ val_out) {
    __shared__ uint32_t lh[kBins];
    __shared__ PickShared ps;
    __shared__ uint32_t scan[34];
    const int64_t i = blockIdx.x;
    if (!channel_live(a, i)) return;  // uniform over the workgroup
    const int lane = threadIdx.x & (CMPQ_WAVE - 1), wave = wave_index();
    const float cent = a.centroids ? a.centroids[i * CMPQ_KMAX + (lane & 15)] : 0.f;
    uint32_t prefix = 0;
    uint64_t rem = (uint64_t)k;  // 1 <= k <= d_out: every pass finds its digit
    for (int pass = 0; pass < 3; ++pass) {
        for (int b = threadIdx.x; b < kBins; b += kWThreads) lh[b] = 0;
        __syncthreads();
        for (int64_t c = wave; c < a.wc_per_channel; c += kWaves) {
            const int64_t o0 = c * kWaveChunk + lane * kWPerLane;
            Raw8<TW> raw;
            fetch8(a, i, o0, raw);
            uint32_t key[8];
            float wv[8];
            score_keys8<TW>(a, raw, cent, key, wv);
            const uint32_t valid = valid8(o0, a.d_out);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (!((valid >> j) & 1u)) continue;
                if (pass == 0) {
                    atomicAdd(&lh[key[j] >> 21], 1u);
                } else if (pass == 1) {
                    if ((key[j] >> 21) == (prefix >> 21)) atomicAdd(&lh[(key[j] >> 10) & 2047u], 1u);
                } else {
                    if ((key[j] >> 10) == (prefix >> 10)) atomicAdd(&lh[key[j] & 1023u], 1u);
                }
            }
        }
        __syncthreads();
        uint32_t bin, tot;
        uint64_t rem_in;
        block_pick(lh, rem, ps, bin, rem_in, tot);
        prefix |= bin << (pass == 0 ? 21 : (pass == 1 ? 10 : 0));
        rem = rem_in;
        __syncthreads();
    }
    const int64_t out0 = (int64_t)live_rank[i] * k;
    write_chunks<TW>(a, prefix, rem, 0, (uint64_t)out0, i * a.wc_per_channel, (i + 1) * a.wc_per_channel, out0 + k,
                     idx_out, val_out, scan);
}

struct WselWs {
    WselState *st;
    uint32_t *hist, *above, *local_last, *stage_cnt;
    uint2 *cnt_unit, *cnt_block;
    unsigned long long *stage_ik;
    uint16_t *stage_val;
    size_t bytes;
};

WselWs wsel_carve(void *ws, const WselPlan &p) {
    WsCarver carve(ws);
    WselWs w;
    w.st = carve.take<WselState>(1);
    w.hist = carve.take<uint32_t>(kHistWords);
    w.cnt_unit = carve.take<uint2>(kMaxUnits);
    w.cnt_block = carve.take<uint2>(kMaxBlocks);
    w.above = carve.take<uint32_t>(kMaxBlocks);
    w.local_last = carve.take<uint32_t>((size_t)kMaxBlocks * 1024);
    w.stage_cnt = carve.take<uint32_t>(kMaxUnits);
    w.stage_ik = carve.take<unsigned long long>((size_t)p.nunits * p.cap);
    w.stage_val = carve.take<uint16_t>((size_t)p.nunits * p.cap);
    w.bytes = carve.need();
    return w;
}

template <typename TW>
int launch_weight_select(WselArgs a, const WselPlan &p, int64_t k, int32_t *idx_out,
                         uint16_t *val_out, void *ws, hipStream_t s) {
    const WselWs w = wsel_carve(ws, p);
    a.stage_ik = w.stage_ik;
    a.stage_val = w.stage_val;
    a.stage_cnt = w.stage_cnt;
    a.cap = p.cap;
    a.sample_stride = p.sample_stride;
    a.n_sample = p.n_sample;
    a.sample_rank = p.sample_rank;
    int64_t sample_blocks = cdiv(p.n_sample, 16);
    if (sample_blocks > 128) sample_blocks = 128;  // every one ends with a flush into the same counters
    if (sample_blocks < cdiv(p.n_sample, kSampleChunks)) sample_blocks = cdiv(p.n_sample, kSampleChunks);
    if (sample_blocks < 1) sample_blocks = 1;
    static_assert(kHistWords % 4 == 0, "");
    wsel_init_kernel<<<(unsigned)cdiv(kHistWords / 4, 256), 256, 0, s>>>(w.st, w.hist);
    // fast chain
    wsel_sample_kernel<TW><<<(unsigned)sample_blocks, kSampleThreads, 0, s>>>(a, w.hist);
    cmpq_timing_before(CMPQ_KERNEL_OUTLIER_STAGE, s);
    constexpr bool kHalf = std::is_same<TW, __half>::value;
    if (kHalf && a.score == CMPQ_SCORE_RESIDUAL && !a.codes)
        wsel_stage_kernel<TW, kHalf><<<p.nblocks, kWThreads, 0, s>>>(a, w.st, w.hist);
    else
        wsel_stage_kernel<TW, false><<<p.nblocks, kWThreads, 0, s>>>(a, w.st, w.hist);
    cmpq_timing_after(CMPQ_KERNEL_OUTLIER_STAGE, s);
    const int list_blocks = (int)cdiv(p.nunits, 32) < 256 ? (int)cdiv(p.nunits, 32) : 256;  // a unit per 8 lanes
    // exact chain: its passes return at once, or are not there, unless the fast chain raised its flag
    // (Workgroups that return at once still cost: three launches of 1024 0.1 us, of 1536 0.5 us more than
    // of 512.  Where they do work they hide its latency: channels of different scale, 8192x28672
    // weights, 512 workgroups 1300 us for the call, 1024 1067, 1536 988, 2048 999; 4096x4096 186, 168,
    // 163, 167.)
    const int most_blocks = p.wc_per_unit >= 16 ? 1536 : 1024;
    const int hist_blocks = p.nblocks < most_blocks ? p.nblocks : most_blocks;
    // The first of them is part of the list's second pass in layers of up to 67 million weights.  Larger ones keep it
    // apart: it wants more workgroups than the list, whose second pass takes 9.7 us instead of 7.6 with that many,
    // beside other streams' kernels more.
    const bool apart = p.wc_per_unit >= 16;
    const int second_blocks = apart || hist_blocks < list_blocks ? list_blocks : hist_blocks;
    wsel_list_kernel<TW, 0><<<list_blocks, kWThreads, 0, s>>>(a, w.st, p.nunits, list_blocks, 0, w.hist, (uint64_t)k);
    wsel_list_kernel<TW, 1><<<second_blocks, kWThreads, 0, s>>>(a, w.st, p.nunits, list_blocks, !apart, w.hist, (uint64_t)k);
    if (apart)
        wsel_hist_kernel<TW, 0><<<hist_blocks, kWThreads, 0, s>>>(a, w.st, (uint64_t)k, p.nblocks, w.hist, w.above, w.local_last);
    wsel_hist_kernel<TW, 1><<<hist_blocks, kWThreads, 0, s>>>(a, w.st, (uint64_t)k, p.nblocks, w.hist, w.above, w.local_last);
    wsel_hist_kernel<TW, 2><<<hist_blocks, kWThreads, 0, s>>>(a, w.st, (uint64_t)k, p.nblocks, w.hist, w.above, w.local_last);
    // threshold, placement and output, from whichever chain holds the answer
    wsel_count_kernel<<<p.nblocks, kWThreads, 0, s>>>(w.st, a, (uint64_t)k, w.hist, w.above, w.local_last, w.cnt_unit, w.cnt_block);
    wsel_emit_kernel<TW><<<p.nblocks, kWThreads, 0, s>>>(a, w.st, w.cnt_unit, w.cnt_block, k, idx_out, val_out);
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

}  // namespace

size_t cmpq_ws_allocate_bits(int64_t) { return 256; }
size_t cmpq_ws_outlier_channels(int64_t) { return 256; }
size_t cmpq_ws_outlier_weights(int64_t d_in, int64_t d_out, int64_t k) {
    if (k < 0) k = 0;
    // the layer-wide selection's tables and lists; the per-channel one needs d_in ranks
    const size_t layer = wsel_carve(nullptr, wsel_plan(d_in, d_out, k)).bytes;
    const size_t channel = align_up((size_t)(d_in > 0 ? d_in : 1) * sizeof(int32_t), 256);
    return layer > channel ? layer : channel;
}

namespace {

// Algorithm 1's integer budget: the k_hi channels with the largest statistic get w_hi, the next up to k_mid
// w_mid, the rest w_lo (all_mid: every other one w_mid).
struct Budget {
    int64_t k_hi, k_mid;
    int w_hi, w_mid, w_lo, all_mid;
};
int channel_budget(int64_t d_in, int64_t n_protected, const int32_t *bit_set, int n_set, double avg_bits,
                   int64_t *counts_host, Budget &p) {
    if (n_set < 1 || n_set > 4) return CMPQ_EBUDGET;
    for (int j = 0; j < n_set; ++j) {
        if (bit_set[j] < 1 || bit_set[j] > 4) return CMPQ_EBUDGET;
        if (j && bit_set[j] != bit_set[j - 1] + 1) return CMPQ_EBUDGET;
    }
    const int lo = bit_set[0], hi = bit_set[n_set - 1];
    if (!(avg_bits >= lo - 1e-9 && avg_bits <= hi + 1e-9)) return CMPQ_EBUDGET;
    const int64_t d_eff = d_in - n_protected;
    const double nearest = (double)(int64_t)(avg_bits + 0.5);
    const double gap = avg_bits - nearest;
    if ((gap < 0 ? -gap : gap) < 1e-9) {
        const int s = (int)nearest;
        int64_t m = 0;
        if (s - 1 >= lo && s + 1 <= hi && d_eff > 0) {
            const double x = 0.01 * (double)(d_eff - 1) - 1e-12;
            m = (int64_t)x;
            if ((double)m < x) ++m;  // ceil
            if (m < 0) m = 0;
            if (2 * m > d_eff) m = d_eff / 2;
        }
        p = Budget{m, d_eff - m, s + 1, s, s - 1, m == 0};
    } else {
        const int s = (int)avg_bits;  // floor, avg_bits > 0
        const int64_t T = (int64_t)(avg_bits * (double)d_eff + 1e-9);
        p = Budget{T - (int64_t)s * d_eff, d_eff, s + 1, s, s, 1};
    }
    if (counts_host) {
        for (int j = 0; j < n_set; ++j) counts_host[j] = 0;
        if (p.k_hi > 0) counts_host[p.w_hi - lo] += p.k_hi;
        if (p.k_mid - p.k_hi > 0) counts_host[p.w_mid - lo] += p.k_mid - p.k_hi;
        if (d_eff - p.k_mid > 0) counts_host[p.w_lo - lo] += d_eff - p.k_mid;
    }
    return CMPQ_OK;
}

void launch_top_channels(const float *sumsq, int64_t d_in, int64_t k, int32_t *idx_out, uint8_t *mask_out, hipStream_t s) {
    if (d_in <= kRankPer * kRankThreads)
        top_channels_reg_kernel<kRankPer><<<1, kRankThreads, 0, s>>>(sumsq, (int)d_in, (uint32_t)k, idx_out, mask_out);
    else
        top_channels_kernel<<<1, kSelThreads, 0, s>>>(sumsq, d_in, (uint32_t)k, idx_out, mask_out);
}

void launch_allocate_bits(const float *sumsq, int64_t d_in, const uint8_t *chan_mask, const Budget &p, uint8_t *bits, hipStream_t s) {
    if (d_in <= kRankPer * kRankThreads)
        allocate_bits_reg_kernel<kRankPer><<<1, kRankThreads, 0, s>>>(sumsq, (int)d_in, chan_mask, (uint32_t)p.k_hi,
                                                                       (uint32_t)p.k_mid, p.all_mid, p.w_hi, p.w_mid, p.w_lo, bits);
    else
        allocate_bits_kernel<<<1, kSelThreads, 0, s>>>(sumsq, d_in, chan_mask, (uint32_t)p.k_hi, (uint32_t)p.k_mid, p.all_mid,
                                                       p.w_hi, p.w_mid, p.w_lo, bits);
}

}  // namespace

extern "C" int cmpq_allocate_bits(const float *sumsq, int64_t d_in, const uint8_t *chan_mask,
                                  int64_t n_protected, const int32_t *bit_set, int n_set,
                                  double avg_bits, uint8_t *bits, int64_t *counts_host, void *ws,
                                  size_t ws_bytes, void *stream) {
    (void)ws;
    (void)ws_bytes;
    if (!sumsq || !bits || !bit_set || d_in < 0 || n_protected < 0 || n_protected > d_in)
        return CMPQ_EINVAL;
    if (!chan_mask && n_protected != 0) return CMPQ_EINVAL;
    if (d_in >= (int64_t)1 << 31) return CMPQ_ESHAPE;
    Budget p;
    const int rc = channel_budget(d_in, n_protected, bit_set, n_set, avg_bits, counts_host, p);
    if (rc != CMPQ_OK) return rc;
    if (d_in == 0) return CMPQ_OK;
    launch_allocate_bits(sumsq, d_in, chan_mask, p, bits, static_cast<hipStream_t>(stream));
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

extern "C" int cmpq_rank_channels(const float *sumsq, int64_t d_in, int64_t k_act, const int32_t *bit_set, int n_set,
                                  double avg_bits, int32_t *act_idx, uint8_t *chan_mask, uint8_t *bits,
                                  int64_t *counts_host, void *stream) {
    if (!sumsq || !bits || !bit_set || !chan_mask || d_in < 0 || k_act < 0 || (k_act > 0 && !act_idx)) return CMPQ_EINVAL;
    if (d_in >= (int64_t)1 << 31) return CMPQ_ESHAPE;
    if (k_act > d_in) return CMPQ_ECOUNT;
    Budget p;
    const int rc = channel_budget(d_in, k_act, bit_set, n_set, avg_bits, counts_host, p);
    if (rc != CMPQ_OK) return rc;
    if (d_in == 0) return CMPQ_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d_in <= kRankPer * kRankThreads) {
        const uint3 k = make_uint3((uint32_t)k_act, (uint32_t)(k_act + p.k_hi), (uint32_t)(k_act + p.k_mid));
        auto kern = p.all_mid ? rank_channels_kernel<kRankPer, 2> : rank_channels_kernel<kRankPer, 3>;
        kern<<<1, kRankThreads, 0, s>>>(sumsq, (int)d_in, k, p.w_hi, p.w_mid, p.w_lo, act_idx, chan_mask, bits);
    } else {
        launch_top_channels(sumsq, d_in, k_act, act_idx, chan_mask, s);
        launch_allocate_bits(sumsq, d_in, chan_mask, p, bits, s);
    }
    CMPQ_LAUNCH_CHECK();
    return CMPQ_OK;
}

extern "C" int cmpq_extract_outliers(int mode, int score, int scope, const float *sumsq, const void *W,
                                     int dtype, int64_t d_in, int64_t d_out, int64_t ldw,
                                     const float *centroids, const uint8_t *codes,
                                     const uint8_t *bits, int64_t k, int32_t *idx_out,
                                     uint16_t *val_out, uint8_t *chan_mask_out, void *ws,
                                     size_t ws_bytes, void *stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d_in < 0 || k < 0) return CMPQ_EINVAL;
    if (mode == CMPQ_OUTLIER_CHANNELS) {
        if (!sumsq || (k > 0 && !idx_out)) return CMPQ_EINVAL;
        if (d_in >= (int64_t)1 << 31) return CMPQ_ESHAPE;
        if (k > d_in) return CMPQ_ECOUNT;
        if (d_in == 0) return CMPQ_OK;
        launch_top_channels(sumsq, d_in, k, idx_out, chan_mask_out, s);
        CMPQ_LAUNCH_CHECK();
        return CMPQ_OK;
    }
    if (mode != CMPQ_OUTLIER_WEIGHTS) return CMPQ_EINVAL;
    if (score != CMPQ_SCORE_RESIDUAL && score != CMPQ_SCORE_MAGNITUDE) return CMPQ_EINVAL;
    if (scope != CMPQ_SCOPE_LAYER && scope != CMPQ_SCOPE_CHANNEL) return CMPQ_EINVAL;
    if (dtype != CMPQ_F16 && dtype != CMPQ_F32) return CMPQ_EINVAL;
    if (d_out < 0 || !bits || (k > 0 && !idx_out)) return CMPQ_EINVAL;
    if (d_in > 0 && d_out > 0 && !W) return CMPQ_EINVAL;
    if (score == CMPQ_SCORE_RESIDUAL && d_in > 0 && d_out > 0 && !centroids) return CMPQ_EINVAL;
    if (ldw < d_out) return CMPQ_ESHAPE;
    if (d_in > 0 && d_out > ((int64_t)1 << 31) / d_in) return CMPQ_ESHAPE;  // linear index in int32
    if (scope == CMPQ_SCOPE_CHANNEL ? k > d_out : k > d_in * d_out) return CMPQ_ECOUNT;
    if (scope == CMPQ_SCOPE_CHANNEL && d_in > 0 && k > ((int64_t)1 << 31) / d_in) return CMPQ_ESHAPE;
    if (k == 0 || d_in == 0 || d_out == 0) return CMPQ_OK;
    if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 != 0 || ws_bytes < cmpq_ws_outlier_weights(d_in, d_out, k))
        return CMPQ_EWORKSPACE;
    const WselPlan p = wsel_plan(d_in, d_out, k);
    WselArgs a;
    a.W = W;
    a.centroids = centroids;
    a.codes = score == CMPQ_SCORE_RESIDUAL ? codes : nullptr;
    a.bits = bits;
    a.d_in = d_in;
    a.d_out = d_out;
    a.ldw = ldw;
    a.wc_per_channel = p.wc_per_channel;
    a.total_wc = p.total_wc;
    a.wc_per_unit = p.wc_per_unit;
    a.score = score;
    const int esz = dtype == CMPQ_F16 ? 2 : 4;
    a.vec_ok = reinterpret_cast<uintptr_t>(W) % 16 == 0 && (ldw * esz) % 16 == 0 &&
               (a.codes == nullptr || (reinterpret_cast<uintptr_t>(codes) % 8 == 0 && d_out % 8 == 0));
    if (scope == CMPQ_SCOPE_CHANNEL) {
        int32_t *live_rank = static_cast<int32_t *>(ws);
        wsel_live_rank_kernel<<<1, 1024, 0, s>>>(bits, d_in, live_rank);
        if (dtype == CMPQ_F16)
            wsel_channel_kernel<__half><<<(unsigned)d_in, kWThreads, 0, s>>>(a, live_rank, k, idx_out, val_out);
        else
            wsel_channel_kernel<float><<<(unsigned)d_in, kWThreads, 0, s>>>(a, live_rank, k, idx_out, val_out);
        CMPQ_LAUNCH_CHECK();
        return CMPQ_OK;
    }
    return dtype == CMPQ_F16 ? launch_weight_select<__half>(a, p, k, idx_out, val_out, ws, s)
                             : launch_weight_select<float>(a, p, k, idx_out, val_out, ws, s);
}
