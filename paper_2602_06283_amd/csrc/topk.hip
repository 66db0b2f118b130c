// Alg. 3, TopK step: exact selection of the k largest scores per (sequence, KV head), spread over
// many workgroups: a histogram, a sweep with the threshold bin it gives, and an ordered emit.
//
//   topk_row_kernel     short rows: the whole select of a row in one workgroup, one launch.
// Longer rows:
//   topk_hist_kernel    histogram of every valid score, in bins from a sample of the row and the
//                       scores' exponents (sampled_bin); the fused decode step gets an adaptive
//                       one from the scoring pass instead, with bins sized from the
//                       bucket-probability tables (score_bin).
//   topk_filter_kernel<true, .>  finds the threshold bin, then sweeps: scores above it are selected,
//                       scores in it are candidates: a few dozen where the bins fit the row, any
//                       number where many scores lie close together or tie.  More than kSplitMin
//                       of sampled bins are counted by sub-bin.
//   topk_emit_kernel    a workgroup per region of the sweep ranks the candidates on the score and
//                       then on the token position (smaller position wins a tie; emit_long: long
//                       lists, by sub-bin) and writes its part of the index row in ascending
//                       order.  Leaves histograms and counters at zero.
// Where the scoring pass could not size bins it leaves a histogram of leading 11-bit digits:
//   topk_hist2_kernel   finds the threshold digit, then histograms the next 11 bits over the
//                       scores in that digit.
//   topk_filter_kernel<false, .>  the sweep with the two-digit threshold.
// Stages talk through global memory across kernel boundaries only: no workgroup waits on
// another and no fence is needed.  LDS arrays that a thread walks in runs of PER consecutive
// words carry one pad word per run, which makes those walks free of bank conflicts.
#include "topk_device.h"

namespace sk {

// Bin of a score in a row nobody has binned yet: the sum of an adaptive bin (512 equal ones per
// octave of 1 + (v - lo) * inv over the first two octaves, 256 over the next two) and of the
// score's sign and exponent.  Both are non-decreasing in v, so the sum is too, and two scores share
// a bin only if they share both parts: fine steps where (lo, inv) fit the row, never more than an
// octave where they do not.
static_assert(kHistBins == 2048, "1536 adaptive bins and 511 for sign and exponent");
__device__ __forceinline__ uint32_t sampled_bin(float v, float lo, float inv) {
    const float y = fmaf(fmaxf(v - lo, 0.0f), inv, 1.0f);
    const uint32_t fine = (__float_as_uint(y) - 0x3f800000u) >> 14;
    return min(min(fine, 512 + (fine >> 1)), 1535u) + (order_key(v) >> 23);   // (the halved steps are the smaller from 1024 on)
}

// (lo, inv) from a sample: every workgroup takes a mean and a deviation from the same 512 scores of
// the row, spread evenly, so all of them (and, through the threshold record, the sweep) bin alike.
// Scores further than four deviations from the mean are left out and both taken again, so that a
// few spikes do not widen the bins.  By the one-sided Chebyshev inequality the largest share f of
// any numbers lies above their mean - sqrt(f / (1 - f)) deviations: 0.34 for f = 0.1, 0.58 for 0.25.
// The bins start half a deviation or one below the mean there, a 512th of a deviation wide at their
// start.  That is a rule of thumb, for a (trimmed) sample only stands for the row; where the cut
// lies below, or a cluster of close scores or a spread over decades puts many scores into one bin,
// the sweep counts them by sub-bin and emit_long goes on from there.  The select is exact for any
// bins.
// 131072 scores x 8 heads, k = 2048, us, with adaptive bins alone / now (sign and exponent in the bin,
// sub-bins): a bell 14.3 / 14.8, 6 % in a tight cluster far up 130 / 24, clusters in a cluster 84 / 24,
// counts with a small soft part 59 / 24, a long tail below 257 / 21, seventy decades 685 / 17; 32768
// scores, k = 1024: 13.3 / 13.6, 51 / 20, 54 / 21, 41 / 19, 66 / 19, 155 / 14.  (Laying the bins between
// two order statistics of 256 sampled scores cost every row 3.7.)
__global__ __launch_bounds__(kTopkThreads) void topk_hist_kernel(TopkArgs a) {
    constexpr int NW = kTopkThreads / 64;
    __shared__ uint32_t h[kHistBins];
    __shared__ float part[2][3][NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.z, bh = b * a.Hkv + blockIdx.y;
    const int key0 = blockIdx.x * kSlice;
    const int i = key0 + tid * kPer;
    const float *row = a.scores + (int64_t)bh * a.max_n;
    float e[kPer];
    load_scores(row, i, a.max_n, e);
    const int seq = clamp_len(scalar_load(&a.seq_len[b]), a.max_n);
    const int kreq = clamp_len(scalar_load(&a.k[b]), a.max_k);
    const int key1 = min(key0 + kSlice, seq);
    if (key0 >= key1 && blockIdx.x != 0) return;       // workgroup 0 always publishes the bins
    const float v = seq > 0 ? row[(int)(((int64_t)tid * seq) / kTopkThreads)] : 0.0f;
    for (int j = tid; j < kHistBins; j += kTopkThreads) h[j] = 0;
    bool use = seq > 0 && fabsf(v) < 3.0e38f;          // (false for NaN and both infinities)
    float cnt = 0.0f, mu = 0.0f, sigma = 0.0f, finite = 0.0f;
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const float n0 = row_sum<64>(use ? 1.0f : 0.0f), n1 = row_sum<64>(use ? v : 0.0f);
        if (lane == 0) {
            part[round][0][wave] = n0;
            part[round][1][wave] = n1;
        }
        __syncthreads();
        cnt = mu = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            cnt += part[round][0][w];
            mu += part[round][1][w];
        }
        if (round == 0) finite = cnt;
        mu = cnt > 0.0f ? mu / cnt : 0.0f;
        const float d = use ? v - mu : 0.0f;
        const float n2 = row_sum<64>(d * d);
        if (lane == 0) part[round][2][wave] = n2;
        __syncthreads();
        float var = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) var += part[round][2][w];
        sigma = sqrtf(cnt > 0.0f ? var / cnt : 0.0f);
        use = use && fabsf(v - mu) <= 4.0f * sigma;
    }
    sigma = fminf(fmaxf(sigma, fmaxf(fabsf(mu) * 1e-6f, 1e-30f)), 1.0e37f);
    const float share = (float)kreq * (float)kTopkThreads / fmaxf((float)seq * finite, 1.0f);   // of the finite scores
    const float lo = mu - (share <= 0.1f ? 0.5f : share <= 0.25f ? 1.0f : 4.0f) * sigma;
    const float inv = 1.0f / (share <= 0.25f ? sigma : 4.0f * sigma);
    if (blockIdx.x == 0 && tid == 0) {
        uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
        thr[kThrBinLo] = __float_as_uint(lo);
        thr[kThrBinInv] = __float_as_uint(inv);
    }
    if (key0 >= key1) return;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (i + j < key1 && selectable(e[j])) atomicAdd(&h[sampled_bin(e[j], lo, inv)], 1u);
    __syncthreads();
    uint32_t *gh = a.hist + (int64_t)bh * kHistBins;
    for (int j = tid; j < kHistBins; j += kTopkThreads)
        if (h[j]) atomicAdd(&gh[j], h[j]);
}

// First score key of a bin and of the bin after it (the bin function is non-decreasing in the
// score).  Whole wavefronts: the lower half searches for the one, the upper half for the other.
template <typename F> __device__ __forceinline__ uint2 bin_keys(uint32_t bin, F bin_of) {
    const int lane = threadIdx.x & 63;
    const uint32_t want = bin + (lane >> 5);
    uint32_t below = 0;                                          // a key below the one sought, or 0
#pragma unroll 1
    for (int sh = 27; sh >= 0; sh -= sh > 2 ? 5 : 2) {           // 32 probes a step
        const uint32_t probe = below + ((uint32_t)(lane & 31) << sh);
        const uint32_t key = min(max(probe, 0x007fffffu), 0xff800000u);   // -inf .. +inf
        const float v = __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
        const uint64_t hit = __ballot(probe <= 0xff800000u && bin_of(v) < want);
        const int n = __popc(lane < 32 ? (uint32_t)hit : (uint32_t)(hit >> 32));
        below += (uint32_t)max(n - 1, 0) << sh;
    }
    return make_uint2((uint32_t)__builtin_amdgcn_readlane((int)below, 0) + 1, (uint32_t)__builtin_amdgcn_readlane((int)below, 32) + 1);
}

// Sub-bins of a threshold bin of sampled_bin: equal steps of the score key between the bin's two
// ends.  Non-decreasing in the score, and the same for all workgroups of a row.
struct SubBins {
    uint32_t lo;
    int shift;
    __device__ __forceinline__ uint32_t of(uint32_t key) const {
        return key <= lo ? 0u : min((key - lo) >> shift, (uint32_t)(kHistBins - 1));
    }
};
__device__ __forceinline__ SubBins sub_bins(uint32_t bin, float bin_lo, float bin_inv) {
    const uint2 k = bin_keys(bin, [&](float v) { return sampled_bin(v, bin_lo, bin_inv); });
    const uint32_t last = k.y > k.x + 1 ? k.y - k.x - 1 : 1u;    // the largest offset
    const int bits = 32 - __clz((int)last);
    return SubBins{k.x, bits > kHistBits ? bits - kHistBits : 0};
}

// First threshold digit, then the histogram of the second digit over the scores in it.
__global__ __launch_bounds__(kTopkThreads) void topk_hist2_kernel(TopkArgs a) {
    constexpr int PER = kHistBins / kTopkThreads;
    __shared__ uint32_t h[padded_size<kHistBins, PER>()];
    __shared__ uint32_t tmp[16];
    __shared__ uint32_t res[4];
    const int tid = threadIdx.x;
    const int b = blockIdx.z, bh = b * a.Hkv + blockIdx.y;
    const int key0 = blockIdx.x * kSlice;
    const int i = key0 + tid * kPer;
    float e[kPer];
    load_scores(a.scores + (int64_t)bh * a.max_n, i, a.max_n, e);   // first: overlaps what follows
    const uint32_t *gh1 = a.hist + (int64_t)bh * kHistBins;
    uint32_t c1[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) c1[j] = gh1[tid + j * kTopkThreads];
    const int key1 = min(key0 + kSlice, clamp_len(a.seq_len[b], a.max_n));
    const uint32_t kreq = (uint32_t)clamp_len(a.k[b], a.max_k);
    if (key0 >= key1 && blockIdx.x != 0) return;       // workgroup 0 always publishes the record
#pragma unroll
    for (int j = 0; j < PER; ++j) h[padded<PER>(tid + j * kTopkThreads)] = c1[j];
    if (tid < 4) res[tid] = 0;
    __syncthreads();
    // a target beyond the number of valid scores finds nothing; res[3] then gives that number
    find_threshold<kHistBins>(h, kreq, res, tmp);
    uint32_t k_eff = kreq, tb1 = res[0], above1 = res[1], cnt1 = res[2];
    const uint32_t valid = res[3];
    if (valid < kreq) {                                 // fewer valid scores than asked for: take all
        k_eff = valid;
        if (valid > 0) {
            __syncthreads();
            find_threshold<kHistBins>(h, valid, res, tmp);
            tb1 = res[0]; above1 = res[1]; cnt1 = res[2];
        }
    }
    uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
    if (blockIdx.x == 0 && tid == 0) {
        thr[0] = k_eff; thr[1] = tb1; thr[2] = above1; thr[3] = cnt1;
    }
    if (k_eff == 0 || key0 >= key1) return;
    __syncthreads();
    uint32_t *h2 = h;                                   // plain (unpadded) use from here on
    for (int j = tid; j < kHistBins; j += kTopkThreads) h2[j] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t key = order_key(e[j]);
        if (i + j < key1 && selectable(e[j]) && (key >> kLowBits) == tb1) atomicAdd(&h2[digit2(key)], 1u);
    }
    __syncthreads();
    uint32_t *gh2 = a.hist2 + (int64_t)bh * kHistBins;
    for (int j = tid; j < kHistBins; j += kTopkThreads)
        if (h2[j]) atomicAdd(&gh2[j], h2[j]);
}

// Threshold, then the sweep.  ADAPT = false: the second threshold digit from the histogram of
// topk_hist2_kernel, lead = the two leading digits of the score key.  ADAPT = true: the
// threshold bin of the adaptive histogram, lead = that bin.
// REFINE: the bins are sampled_bin's, and a long list is counted by sub-bin.
template <bool ADAPT, bool REFINE>
__global__ __launch_bounds__(kTopkThreads) void topk_filter_kernel(TopkArgs a) {
    constexpr int PER = kHistBins / kTopkThreads;
    __shared__ uint32_t h[padded_size<kHistBins, PER>()];
    __shared__ uint32_t tmp[16];
    __shared__ uint32_t res[4];
    __shared__ uint32_t s_base[2];
    asm volatile("" ::"s"(a.scores), "s"(a.hist), "s"(a.thr), "s"(a.sel_cnt), "s"(a.seq_len), "s"(a.k), "s"(a.max_k), "s"(a.n_regions),
                 "s"(a.counters), "s"(a.cand_key), "s"(a.sel_regions));          // (arguments in one trip)
    const int tid = threadIdx.x;
    const int b = blockIdx.z, bh = b * a.Hkv + blockIdx.y;
    const int key0 = blockIdx.x * kSlice;
    const int i = key0 + tid * kPer;
    float e[kPer];
    load_scores(a.scores + (int64_t)bh * a.max_n, i, a.max_n, e);
    const uint32_t *gh = (ADAPT ? a.hist : a.hist2) + (int64_t)bh * kHistBins;
    uint32_t c2[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) c2[j] = gh[tid + j * kTopkThreads];
    uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
    // (the length, the request and the record in one trip, not one behind the other; of the record only
    // what an earlier launch has written, the rest is for workgroup 0 to write)
    const int len = scalar_load(&a.seq_len[b]);
    uint32_t kreq = 0, rec0 = 0, rec1 = 0, rec2 = 0;
    float bin_lo = 0.0f, bin_inv = 0.0f;
    if constexpr (ADAPT) {
        kreq = (uint32_t)clamp_len(scalar_load(&a.k[b]), a.max_k);
        bin_lo = __uint_as_float(scalar_load(&thr[kThrBinLo]));
        bin_inv = __uint_as_float(scalar_load(&thr[kThrBinInv]));
        asm volatile("" ::"s"(len), "s"(kreq), "s"(bin_lo), "s"(bin_inv));
    } else {
        rec0 = scalar_load(&thr[0]);
        rec1 = scalar_load(&thr[1]);
        rec2 = scalar_load(&thr[2]);
        asm volatile("" ::"s"(len), "s"(rec0), "s"(rec1), "s"(rec2));
    }
    const int key1 = min(key0 + kSlice, clamp_len(len, a.max_n));
    // this workgroup's region of the selected list: empty unless the sweep below says otherwise
    uint32_t *selcnt = a.sel_cnt + (int64_t)bh * a.n_regions + blockIdx.x;
    if (tid == 0) *selcnt = 0u;
    uint32_t k_eff, pair, above, n_cand;
    if (ADAPT) {
        if (key0 >= key1 && blockIdx.x != 0) return;   // workgroup 0 always publishes the record
#pragma unroll
        for (int j = 0; j < PER; ++j) h[padded<PER>(tid + j * kTopkThreads)] = c2[j];
        if (tid < 4) res[tid] = 0;
        __syncthreads();
        // a target beyond the number of valid scores finds nothing; res[3] then gives that number
        find_threshold<kHistBins>(h, kreq, res, tmp);
        k_eff = kreq;
        const uint32_t valid = res[3];
        if (valid < kreq) {                             // fewer valid scores than asked for: take all
            k_eff = valid;
            if (valid > 0) {
                __syncthreads();
                find_threshold<kHistBins>(h, valid, res, tmp);
            }
        }
        pair = res[0]; above = res[1]; n_cand = res[2];
        if (blockIdx.x == 0 && tid == 0) {
            thr[0] = k_eff; thr[5] = k_eff ? above : 0u; thr[6] = k_eff ? n_cand : 0u;
        }
        if (k_eff == 0) return;
    } else {
        k_eff = rec0;
        const uint32_t tb1 = rec1, above1 = rec2;
        if (k_eff == 0) return;
        if (key0 >= key1 && blockIdx.x != 0) return;
#pragma unroll
        for (int j = 0; j < PER; ++j) h[padded<PER>(tid + j * kTopkThreads)] = c2[j];
        if (tid < 4) res[tid] = 0;
        __syncthreads();
        find_threshold<kHistBins>(h, k_eff - above1, res, tmp);    // 1 <= k_eff - above1 <= scores in tb1
        const uint32_t tb2 = res[0];
        above = above1 + res[1]; n_cand = res[2];
        if (blockIdx.x == 0 && tid == 0) {
            thr[4] = tb2; thr[5] = above; thr[6] = n_cand;
        }
        pair = (tb1 << kHistBits) | tb2;                           // the 2*kHistBits leading bits
    }
    if (key0 >= key1) return;
    uint32_t *cnt = a.counters + (int64_t)bh * kCounterStride;
    uint32_t *ckey = a.cand_key + (int64_t)bh * a.max_n;
    int32_t *cidx = a.cand_idx + (int64_t)bh * a.max_n;
    int32_t *region = a.sel_regions + ((int64_t)bh * a.n_regions + blockIdx.x) * kSlice;

    // Scores above the threshold bin go to this workgroup's own region of the selected list, in
    // position order (no reservation across workgroups: what a region holds depends on the
    // scores alone); candidates of the threshold bin, a handful, are appended to one list with
    // an atomic per workgroup - they are ranked as a set, so their order does not matter.
    uint32_t keys[kPer];
    uint32_t flags = 0;                           // bit j: selected, bit 16+j: candidate
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const bool ok = i + j < key1 && selectable(e[j]);
        keys[j] = order_key(e[j]);
        const uint32_t lead = !ADAPT ? keys[j] >> kDigit2Shift : REFINE ? sampled_bin(e[j], bin_lo, bin_inv) : score_bin(e[j], bin_lo, bin_inv);
        if (ok && lead > pair) flags |= 1u << j;
        if (ok && lead == pair) flags |= 1u << (16 + j);
    }
    const uint32_t mine = (uint32_t)__popc(flags & 0xffffu) | ((uint32_t)__popc(flags >> 16) << 16);
    uint32_t total;
    const uint32_t before = block_excl_scan(mine, &total, tmp);   // both counts in one word
    if (tid == 0) {
        const uint32_t ncand = total >> 16;
        *selcnt = total & 0xffffu;
        s_base[1] = ncand ? atomicAdd(&cnt[1], ncand) : 0u;
    }
    __syncthreads();
    uint32_t at_sel = before & 0xffffu, at_cand = s_base[1] + (before >> 16);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (flags & (1u << j)) region[at_sel++] = i + j;
        if (flags & (1u << (16 + j))) {
            ckey[at_cand] = keys[j];
            cidx[at_cand] = i + j;
            ++at_cand;
        }
    }
    // a long list: the candidates' sub-bins, for the emit kernel
    if (REFINE && n_cand > (uint32_t)kSplitMin && (total >> 16 || blockIdx.x == 0)) {
        const SubBins sub = sub_bins(pair, bin_lo, bin_inv);
        if (blockIdx.x == 0 && tid == 0) {
            thr[kThrSubLo] = sub.lo;
            thr[kThrSubShift] = (uint32_t)sub.shift;
        }
        for (int j = tid; j < kHistBins; j += kTopkThreads) h[j] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (flags & (1u << (16 + j))) atomicAdd(&h[sub.of(keys[j])], 1u);
        __syncthreads();
        uint32_t *gh2 = a.hist2 + (int64_t)bh * kHistBins;
        for (int j = tid; j < kHistBins; j += kTopkThreads)
            if (h[j]) atomicAdd(&gh2[j], h[j]);
    }
}

// the rest of the index row, the count, and the scratch for the next call
__device__ __forceinline__ void finish_row(const TopkArgs &a, int bh, uint32_t k_eff, bool clear2) {
    const int tid = threadIdx.x;
    for (int i = (int)k_eff + tid; i < a.max_k; i += kTopkThreads) a.idx[(int64_t)bh * a.max_k + i] = -1;
    uint32_t *gh1 = a.hist + (int64_t)bh * kHistBins, *gh2 = a.hist2 + (int64_t)bh * kHistBins;
    for (int i = tid; i < kHistBins; i += kTopkThreads) {
        gh1[i] = 0;
        if (clear2) gh2[i] = 0;
    }
    if (tid < 2) a.counters[(int64_t)bh * kCounterStride + tid] = 0;
    if (tid == 0) a.n_selected[bh] = (int32_t)k_eff;
}

// A region's part of the index row where the threshold bin holds more scores than are ranked in
// pairs (a.refine: the sweep has counted them by sub-bin).  Every workgroup of the row finds the
// threshold sub-bin and goes through the whole list: candidates above that sub-bin are kept, those
// in it counted by what is left of their keys (a bin spans an octave at most, so a sub-bin 4096
// keys), and of those that tie on the last key the smallest positions are kept.  The region is
// written through a bitmap; nobody waits for another workgroup.
//   (Bound by the list, which each of the row's workgroups reads from L2: once, three times where
//   the sub-bin holds more than LDS does.  131072 x 8 equal scores, k = 2048: 192 us; 1387 refined
//   digit by digit by one workgroup.)
__device__ __forceinline__ void emit_long(const TopkArgs &a, int bh, int reg, uint32_t k_eff, uint32_t above, uint32_t n_cand,
                                          uint32_t *lds) {
    constexpr int NT = kTopkThreads, PER = kHistBins / NT, RPER = kRefineBins / NT;
    static_assert(kSlice == 8 * NT, "a thread emits the eight positions of a bitmap byte");
    static_assert(kRefineBins >= 1 << (23 - kHistBits), "a refinement bin for every key of a sub-bin");
    __shared__ uint32_t tmp[16], res[4], s_n;
    const int tid = threadIdx.x;
    unsigned long long *ck = (unsigned long long *)lds;          // [kRankMax + 4] candidates of the threshold sub-bin
    uint32_t *h = (uint32_t *)(ck + kRankMax + 4);               // [padded kRefineBins]
    uint32_t *bitmap = h + padded_size<kRefineBins, RPER>();     // [kSlice / 32] kept positions of the region
    uint32_t *ties = bitmap + kSlice / 32;                       // [kSlice / 32] its candidates that tie on the last key kept
    uint32_t *gh2 = a.hist2 + (int64_t)bh * kHistBins;
    for (int j = tid; j < kHistBins; j += NT) h[padded<PER>(j)] = gh2[j];
    for (int j = tid; j < kSlice / 32; j += NT) bitmap[j] = ties[j] = 0;
    if (tid < 4) res[tid] = 0;
    if (tid == 0) s_n = 0;
    const uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
    const SubBins sub{thr[kThrSubLo], (int)thr[kThrSubShift]};
    __syncthreads();
    const uint32_t need = k_eff - above;
    find_threshold<kHistBins>(h, need, res, tmp);                // 1 <= need <= n_cand
    const uint32_t t2 = res[0], need2 = need - res[1], n2 = res[2];
    // the row's last workgroup to have read hist2 clears it for the next call
    uint32_t *ticket = a.counters + (int64_t)bh * kCounterStride + kTicket;
    uint32_t turn = 0;
    if (tid == 0) turn = atomicAdd(ticket, 1u);
    if (reg == 0) finish_row(a, bh, k_eff, false);
    // ---- the candidates, and what earlier regions hold
    const uint32_t *selcnt = a.sel_cnt + (int64_t)bh * a.n_regions;
    const uint32_t *ckey = a.cand_key + (int64_t)bh * a.max_n;
    const int32_t *cidx = a.cand_idx + (int64_t)bh * a.max_n;
    const int32_t *entries = a.sel_regions + ((int64_t)bh * a.n_regions + reg) * kSlice;
    __syncthreads();                                             // (every thread has its t2, need2, n2)
    for (int j = tid; j < padded_size<kRefineBins, RPER>(); j += NT) h[j] = 0;
    if (tid < 4) res[tid] = 0;
    auto mark = [&](uint32_t *map, int32_t pos) { atomicOr(&map[(pos % kSlice) >> 5], 1u << (pos & 31)); };
    uint32_t earlier = 0;
    for (int r = tid; r < reg; r += NT) earlier += selcnt[r];
    const uint32_t cnt = selcnt[reg];
    for (uint32_t i = tid; i < cnt; i += NT) mark(bitmap, entries[i]);
    __syncthreads();
    auto keep = [&](int32_t pos) {
        const int r = pos / kSlice;
        if (r < reg) ++earlier;
        if (r == reg) mark(bitmap, pos);
    };
    auto for_list = [&](auto f) {
        constexpr int U = 4;                                     // loads in flight
        for (uint32_t i0 = tid; i0 < n_cand; i0 += U * NT) {
            uint32_t key[U];
            int32_t pos[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = min(i0 + u * NT, n_cand - 1);
                key[u] = ckey[i];
                pos[u] = cidx[i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < n_cand) f(sub.of(key[u]), key[u], pos[u]);
        }
    };
    const bool fits = n2 <= (uint32_t)kRankMax;
    for_list([&](uint32_t d, uint32_t key, int32_t pos) {
        if (d > t2) keep(pos);
        if (d == t2 && fits) {
            const uint32_t at = atomicAdd(&s_n, 1u);             // (n2 of them)
            if (at < (uint32_t)kRankMax) ck[at] = ((unsigned long long)key << 32) | (uint32_t)pos;
        }
    });
    __syncthreads();
    // ---- the threshold sub-bin, key by key
    auto for_sub = [&](auto f) {
        if (fits)
            for (uint32_t i = tid; i < n2; i += NT) f((uint32_t)(ck[i] >> 32), (int32_t)(uint32_t)ck[i]);
        else
            for_list([&](uint32_t d, uint32_t key, int32_t pos) {
                if (d == t2) f(key, pos);
            });
    };
    const uint32_t k0 = sub.lo + (t2 << sub.shift);
    auto digit = [&](uint32_t key) { return key <= k0 ? 0u : min(key - k0, (uint32_t)(kRefineBins - 1)); };
    for_sub([&](uint32_t key, int32_t) {
        // (lanes with the first one's digit add together: equal scores come by the thousand)
        const uint32_t d = digit(key), first = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const uint64_t same = __ballot(d == first);
        if (d != first) atomicAdd(&h[padded<RPER>((int)d)], 1u);
        else if ((tid & 63) == __ffsll((unsigned long long)same) - 1) atomicAdd(&h[padded<RPER>((int)d)], (uint32_t)__popcll(same));
    });
    __syncthreads();
    find_threshold<kRefineBins>(h, need2, res, tmp);             // 1 <= need2 <= n2
    const uint32_t t3 = res[0];
    uint32_t ties_earlier = 0;
    for_sub([&](uint32_t key, int32_t pos) {
        const uint32_t d = digit(key);
        if (d > t3) keep(pos);
        if (d == t3) {
            if (pos / kSlice < reg) ++ties_earlier;
            if (pos / kSlice == reg) mark(ties, pos);
        }
    });
    uint32_t base, before, total;
    block_excl_scan(earlier, &base, tmp);                        // (barriers: the bitmaps are complete)
    block_excl_scan(ties_earlier, &before, tmp);
    const uint32_t need3 = need2 - res[1];                       // ties to keep: the smallest positions
    base += min(before, need3);
    const uint32_t left = need3 - min(before, need3);            // of them in this region and later ones
    uint32_t mine = (ties[tid >> 2] >> (8 * (tid & 3))) & 0xffu;
    uint32_t rank = block_excl_scan(__popc(mine), &total, tmp);
    uint32_t byte = (bitmap[tid >> 2] >> (8 * (tid & 3))) & 0xffu;
    for (; mine != 0 && rank < left; mine &= mine - 1, ++rank) byte |= mine & (0u - mine);
    uint32_t at = base + block_excl_scan(__popc(byte), &total, tmp);
    int32_t *out = a.idx + (int64_t)bh * a.max_k;
    for (int j = 0; j < 8; ++j)
        if ((byte & (1u << j)) && at < k_eff) out[at++] = reg * kSlice + 8 * tid + j;
    // (late: the ticket is a round trip to memory)
    if (tid == 0) s_n = turn == gridDim.x - 1;
    __syncthreads();
    if (s_n) {
        for (int j = tid; j < kHistBins; j += NT) gh2[j] = 0;
        if (tid == 0) *ticket = 0;
    }
}
constexpr size_t kLongLds = (size_t)(kRankMax + 4) * 8 + (size_t)(padded_size<kRefineBins, kRefineBins / kTopkThreads>() + 2 * (kSlice / 32)) * 4;

// The index row, from the sweep's regions and candidates: one workgroup per region, each ranking
// the few candidates itself.  The regions one after the other are the positions selected outright
// in ascending order, so an entry's slot is the number of entries in earlier regions, its index
// in its own, and the kept candidates before it; a kept candidate's slot is the same counts for
// its position.  (One workgroup per row, walking all regions, took 8.4-9.5 us at 32768 scores, 8
// heads.  A whole select, launches back to back: 13.6 us, 19.6 with that kernel and two digit
// histograms; 131072 scores 14.8 / 22.9; 16 x 20000 scores 24.4 / 28.7; 4 M scores 39 us / 7.6 ms.)
// A list too long for pairs goes to emit_long (sampled bins) or, beyond two candidates per thread,
// to the row's first workgroup (topk_resolve_body: bins of the scoring pass).
template <bool REFINE>
__global__ __launch_bounds__(kTopkThreads, 4) void topk_emit_kernel(TopkArgs a) {
    extern __shared__ __align__(16) uint32_t emit_lds[];
    constexpr int NT = kTopkThreads, NW = NT / 64;
    __shared__ uint32_t s_sum[2][NW];            // entries of earlier regions; kept candidates of earlier regions
    __shared__ uint32_t s_nown;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int reg = blockIdx.x, bh = blockIdx.z * a.Hkv + blockIdx.y;
    // ---- every load that needs no other one (inside the buffers whatever the counts are)
    const uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
    const uint32_t t0 = thr[0], t5 = thr[5], t6 = thr[6];
    const uint32_t *selcnt = a.sel_cnt + (int64_t)bh * a.n_regions;
    const int32_t *entries = a.sel_regions + ((int64_t)bh * a.n_regions + reg) * kSlice;
    const uint32_t cnt = selcnt[reg];
    uint32_t pk[2], earlier[2];
    int32_t pp[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int i = tid + j * NT, c = min(i, a.max_n - 1);
        pk[j] = a.cand_key[(int64_t)bh * a.max_n + c];
        pp[j] = a.cand_idx[(int64_t)bh * a.max_n + c];
        earlier[j] = selcnt[min(i, a.n_regions - 1)];
    }
    static_assert(kMaxRegions <= 2 * NT && kRankMax == 2 * NT, "two words per thread");
    int32_t e0 = entries[tid];
    asm volatile("" ::: "memory");               // (keeps the loads together, ahead of what uses them)
    const uint32_t k_eff = t0, above = k_eff ? t5 : 0u, n_cand = k_eff ? t6 : 0u;
    const uint32_t need = k_eff - above;
    if (n_cand > (uint32_t)(REFINE ? kSplitMin : kRankMax)) {
        if constexpr (REFINE) emit_long(a, bh, reg, k_eff, above, n_cand, emit_lds);
        else if (reg == 0) topk_resolve_body(a, bh, emit_lds);
        return;
    }
    int32_t *out = a.idx + (int64_t)bh * a.max_k;
    if (reg == 0) finish_row(a, bh, k_eff, !REFINE);   // (nobody wrote hist2 where the list is short)
    if (k_eff == 0) return;
    // ---- rank the candidates on (score, smaller position first); kept ones in earlier regions
    //      are counted, those of this region listed
    unsigned long long *ck = (unsigned long long *)emit_lds;     // [kRankMax + 4]
    int32_t *s_own = (int32_t *)(ck + kRankMax + 4);             // [kRankMax] kept candidates of this region, any order
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t i = tid + j * NT;
        if (i < n_cand) ck[i] = ((unsigned long long)pk[j] << 32) | (0x7fffffffu - (uint32_t)pp[j]);
    }
    if (tid < 4) ck[n_cand + tid] = 0;           // (whole quads; beats nobody)
    if (tid == 0) s_nown = 0;
    __syncthreads();
    uint32_t kept_earlier = 0;
    const int lg = n_cand <= NT / 8 ? 3 : n_cand <= NT / 4 ? 2 : n_cand <= NT / 2 ? 1 : 0;   // lanes that share a candidate
    for (uint32_t i = (uint32_t)tid >> lg; i < n_cand; i += NT >> lg) {
        const unsigned long long me = ck[i];
        const int32_t pos = (int32_t)(0x7fffffffu - (uint32_t)me);
        if (pos / kSlice > reg) continue;        // (the same for the lanes that share a candidate)
        uint32_t rank = 0;
#pragma unroll 2
        for (uint32_t o = 4 * (tid & ((1 << lg) - 1)); o < n_cand; o += 4 << lg) {
            const ulonglong2 c0 = *(const ulonglong2 *)&ck[o], c1 = *(const ulonglong2 *)&ck[o + 2];
            rank += (c0.x > me) + (c0.y > me) + (c1.x > me) + (c1.y > me);
        }
        if (lg >= 1) rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0xB1, 0xF, 0xF, true);    // lane ^ 1
        if (lg >= 2) rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0x4E, 0xF, 0xF, true);    // lane ^ 2
        if (lg >= 3) rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0x141, 0xF, 0xF, true);   // the other four of eight
        if (rank < need && (tid & ((1 << lg) - 1)) == 0) {
            if (pos / kSlice < reg) ++kept_earlier;
            else s_own[atomicAdd(&s_nown, 1u)] = pos;
        }
    }
    const uint32_t before = (tid < reg ? earlier[0] : 0u) + (tid + NT < reg ? earlier[1] : 0u);
    const uint32_t w0 = wave_incl_scan(before), w1 = wave_incl_scan(kept_earlier);
    if (lane == 63) {
        s_sum[0][wave] = w0;
        s_sum[1][wave] = w1;
    }
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) base += s_sum[0][w] + s_sum[1][w];
    const uint32_t n_own = s_nown;
    // ---- the region's entries, slipped past the kept candidates below them
    for (uint32_t i = tid; i < cnt; i += NT) {
        const int32_t p = i == (uint32_t)tid ? e0 : entries[i];
        uint32_t at = base + i;
        for (uint32_t q = 0; q < n_own; ++q) at += s_own[q] < p;
        out[at] = p;
    }
    for (uint32_t i = tid; i < n_own; i += NT) {
        const int32_t p = s_own[i];
        uint32_t lo = 0, hi = cnt;               // entries of the region below it
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (entries[mid] < p) lo = mid + 1; else hi = mid;
        }
        uint32_t at = base + lo;
        for (uint32_t q = 0; q < n_own; ++q) at += s_own[q] < p;
        out[at] = p;
    }
}
constexpr size_t kEmitLds = (size_t)(kRankMax + 4) * 8 + (size_t)kRankMax * 4;

// ---------------------------------------------------------------------------------------
// Short rows in one launch: one workgroup of 16 wavefronts per (sequence, KV head) holds the row in
// registers (NC chunks of 4096 scores), so the select is a chain of phases in LDS:
//   window   two keys between which the cut should lie: of a sample of 1024 scores, as many ranks above and
//            below the wanted share as three of its deviations (to a bin of the sample's own histogram;
//            where both lie in one bin, equal or close scores, the scores themselves)
//   bins     2048 equal steps of the score key between the two, five instructions a score; the scores
//            above are only counted.  Where the cut lies outside the window after all, the scores on
//            that side are refined
//   refine   while the threshold bin holds more than kRowPairs scores that are not all kept: 2048
//            equal steps of the key over it, and again, down to a single key (three rounds of bins at
//            most: exact for any), which a look at the least and the largest key there finds at once
//   cut      up to kRowPairs scores are ranked in pairs on (score, smaller position first); more
//            only where they tie on one key: the smallest positions, by a scan.  The selection is
//            what is not below one (key, position)
//   emit     slots in position order, from a scan over the kept scores
// Nothing is kept between calls; no scratch.
// Bound by the instructions of one compute unit behind 6 us of launch, loads and phases.
// us a select of a 32nd of 8 rows, this kernel / three launches: like a bell 20496 scores 9.0 / 14.3, 24576 9.3 /
// 13.5, 28672 10.2 / 13.7, 32768 10.7 / 13.8, 36864 11.4 / 14.2; counts 32768 14.7 / 19.2; a heavy tail 32768 10.8 /
// 13.1; a cluster in a cluster 36864 16.7 / 21.0.  An eighth of 36864: a bell 12.1 / 14.1, counts 17.7 / 20.3, counts
// with a soft part 19.7 / 20.9; a third 25.4 / 25.8.  64 rows like a bell 36864 11.8 / 16.4, 49152 13.7 / 19.3.  So
// up to kRowRegions regions of 4096 scores always, where none of 12 shapes of rows with a 32nd, an eighth and a
// third selected was slower; up to kRowRegionsMany from kRowRowsMany rows on, where three launches fill the card.
// (A window by the mean and the deviation of the sample: a bell 0.4 us slower, and rows whose cut lay below it were
// binned twice, those with a window across zero in steps of an octave: a 32nd of 36864 with infinities 30.1 / 11.9
// now, an eighth of counts with a soft part 35.5 / 19.7, a third of 20480 rising scores 27.3 / 10.0.)
// ---------------------------------------------------------------------------------------
constexpr int kRowThreads = 1024, kRowWaves = kRowThreads / 64;
constexpr int kRowPairs = 256;
constexpr int kRowRegions = 9, kRowRegionsMany = 12, kRowRowsMany = 64;
static_assert(kSlice == 4 * kRowThreads, "a chunk is four scores a thread");

// exclusive prefix sum over the workgroup; *total gets the sum
__device__ __forceinline__ uint32_t row_excl_scan(uint32_t v, uint32_t *total, uint32_t *tmp) {
    const int lane = threadIdx.x & 63;
    const uint32_t x = wave_incl_scan(v);
    if (lane == 63) tmp[threadIdx.x >> 6] = x;
    __syncthreads();
    const uint32_t t = wave_incl_scan(lane < kRowWaves ? tmp[lane] : 0u);
    __syncthreads();
    *total = (uint32_t)__builtin_amdgcn_readlane((int)t, kRowWaves - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    return (w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)t, w > 0 ? w - 1 : 0) : 0u) + x - v;
}

// largest over the 64 lanes; every lane ends with it
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
    auto with = [&](uint32_t o) { v = max(v, o); };
    with((uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true));
    with((uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, true));
    with((uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));
    with((uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max(r[0], r[1]);
    r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return max(r[0], r[1]);
}

template <int NC>
__global__ __launch_bounds__(kRowThreads) void topk_row_kernel(TopkArgs a) {
    __shared__ __align__(16) uint32_t h[kHistBins];
    __shared__ __align__(16) unsigned long long ck[kRowPairs + 4];
    __shared__ __align__(16) uint32_t tot[256];                  // [chunk][wavefront]
    __shared__ uint32_t tmp[kRowWaves], s_valid[kRowWaves], res[3], s_n;
    __shared__ unsigned long long s_cut, s_next;
    __shared__ uint2 s_ends[2][kRowWaves], s_count[2][kRowWaves];
    static_assert(NC * kRowWaves <= 256, "four totals a lane");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bh = blockIdx.x, b = bh / a.Hkv;
    const float ninf = -__builtin_inff();
    const float *row = a.scores + (int64_t)bh * a.max_n;
    u32x4_t w[NC];                                               // the scores' bits, or their keys if the cut is negative
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int i = c * kSlice + 4 * tid;
        w[c] = __float_as_uint(ninf);
        if (i < a.max_n) w[c] = *(const u32x4_t *)(row + i);
    }
    const int seq = clamp_len(a.seq_len[b], a.max_n);
    const uint32_t kreq = (uint32_t)clamp_len(a.k[b], a.max_k);
    for (int j = tid; j < kHistBins; j += kRowThreads) h[j] = 0;
    if (tid == 0) s_n = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if ((c + 1) * kSlice > seq) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c * kSlice + 4 * tid + j >= seq) w[c][j] = __float_as_uint(ninf);
        }

    // ---- keys klo .. khi - 1, between which the cut should lie, from a sample: a score a thread, the chunks
    //      in turn
    uint32_t klo, khi;
    {
        const int live = max(1, (seq + kSlice - 1) / kSlice);
        const int mine = tid - live * ((tid * (65536 / live + 1)) >> 16);      // tid % live
        uint32_t v = w[0][0];
#pragma unroll
        for (int c = 1; c < NC; ++c)
            if (c == mine) v = w[c][0];
        const uint32_t key = selectable(__uint_as_float(v)) ? order_key(__uint_as_float(v)) : 0u;   // (-inf behind the end)
        auto lanes16 = [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_umax(x)); };
        const uint32_t sampled = (uint32_t)__popcll(__ballot(mine * kSlice + 4 * tid < seq));
        const uint32_t wmax = wave_umax(key), wmin = wave_umax(key ? ~key : 0u);
        if (lane == 0) {
            s_ends[0][wave] = make_uint2(wmin, wmax);
            s_count[0][wave] = make_uint2(sampled, 0);
        }
        __syncthreads();
        const uint2 ends = s_ends[0][lane & 15];
        const uint32_t least = ~lanes16(ends.x), most = lanes16(ends.y);
        const int bits = most > least ? 32 - __clz((int)(most - least)) : 0, shift = bits > kHistBits ? bits - kHistBits : 0;
        const uint32_t bin = (key - least) >> shift;
        if (key) atomicAdd(&h[bin], 1u);
        const float r = (float)kreq * row_sum<16>((float)s_count[0][lane & 15].x) / fmaxf((float)seq, 1.0f), dev = 3.0f * sqrtf(r) + 3.0f;
        __syncthreads();
        const uint2 c = *(const uint2 *)&h[kHistBins - 2 - 2 * tid];
        uint32_t all;
        const uint32_t above = row_excl_scan(c.x + c.y, &all, tmp);
        const uint32_t rank_lo = min((uint32_t)(r + dev) + 1, all), rank_hi = min((uint32_t)fmaxf(r - dev, 1.0f), all);
        auto here = [&](uint32_t rank, uint32_t *at) {
            if (above < rank && rank <= above + c.x + c.y) *at = (uint32_t)(kHistBins - 2 - 2 * tid + (rank <= above + c.y ? 1 : 0));
        };
        here(rank_lo, &res[0]);
        here(rank_hi, &res[1]);
        *(uint2 *)&h[kHistBins - 2 - 2 * tid] = make_uint2(0, 0);
        __syncthreads();
        const uint32_t bin_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[0]), bin_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[1]);
        klo = least + (bin_lo << shift);
        khi = least + min(((bin_hi + 1) << shift) - 1, most - least) + 1;
        if (bin_lo == bin_hi || khi > 0xff800000u) {             // equal or close scores, or infinities: the keys themselves
            const uint32_t lo = wave_umax(key && bin >= bin_lo ? ~key : 0u);
            const uint32_t hi = wave_umax(key < 0xff800000u && bin <= bin_hi ? key : 0u);   // (+inf would stretch the bins)
            if (lane == 0) s_ends[1][wave] = make_uint2(lo, hi);
            __syncthreads();
            const uint2 cut = s_ends[1][lane & 15];
            klo = ~lanes16(cut.x);
            khi = max(lanes16(cut.y), klo) + 1;
        }
        if (most == 0) klo = 1, khi = 2;                         // (nothing but NaN and -inf)
    }
    // Scores from +0 on compare by their bits, counted from +0; where the bins start below, w takes keys (0
    // for what is never selected, NaN and -inf)
    auto to_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float v = __uint_as_float(w[c][j]);
                w[c][j] = selectable(v) ? order_key(v) : 0u;
            }
    };
    uint32_t zero = 0x80000000u;                                 // the key that w counts from

    // the bin of h with the rank(number of scores in h)-th score from the top in it: the bin, the scores above
    // it, those in it (in res, complete after the barrier); returns the number of scores in h
    auto find = [&](auto rank) {
        const uint2 c = *(const uint2 *)&h[kHistBins - 2 - 2 * tid];
        uint32_t total;
        const uint32_t above = row_excl_scan(c.x + c.y, &total, tmp), target = rank(total);
        if (above < target && target <= above + c.x + c.y) {
            const bool upper = target <= above + c.y;
            res[0] = (uint32_t)(kHistBins - 2 - 2 * tid + (upper ? 1 : 0));
            res[1] = upper ? above : above + c.y;
            res[2] = upper ? c.y : c.x;
        }
        __syncthreads();
        return total;
    };
    if (klo < zero) {
        zero = 0;
        to_keys();
    }
    // ---- how many there are from klo on, and those before khi in bins (one key: only counted, equal scores
    //      come by the thousand)
    const uint32_t range = khi - klo, top0 = 0xff800000u - klo;  // +inf is top0 above klo
    const int bits0 = 32 - __clz((int)(range - 1)), shift0 = bits0 > kHistBits ? bits0 - kHistBits : 0;
    uint32_t from_lo = 0, between = 0;
    if (range > 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t off = w[c][j] - (klo - zero);
                from_lo += off <= top0 ? 1u : 0u;
                if (off < range) atomicAdd(&h[off >> shift0], 1u);
            }
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t off = w[c][j] - (klo - zero);
                from_lo += off <= top0 ? 1u : 0u;
                between += off == 0 ? 1u : 0u;
            }
    }
    from_lo = (uint32_t)row_sum<64>((float)from_lo);
    between = (uint32_t)row_sum<64>((float)between);
    if (lane == 0) s_count[1][wave] = make_uint2(from_lo, between);
    __syncthreads();
    {
        const uint2 n = s_count[1][lane & 15];
        from_lo = (uint32_t)row_sum<16>((float)n.x);
        between = (uint32_t)row_sum<16>((float)n.y);
    }
    if (range > 1) between = find([&](uint32_t total) { return kreq + total - from_lo; });   // (wraps where the cut lies elsewhere)
    // ---- the scores in question: keys k0 .. k0 + span - 1, n_in of them, `need` to keep
    uint32_t k_eff = kreq, k0, span, need, n_in;
    if (from_lo < kreq) {                                        // the cut lies below, or there are fewer scores
        if (zero != 0) {
            zero = 0;
            to_keys();
        }
        uint32_t valid = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) valid += (uint32_t)__popcll(__ballot(w[c][j] != 0u));
        if (lane == 0) s_valid[wave] = valid;
        __syncthreads();
        const uint32_t n_valid = (uint32_t)row_sum<16>((float)s_valid[lane & 15]);
        k_eff = min(kreq, n_valid);
        k0 = 1; span = klo - 1; need = k_eff - from_lo; n_in = n_valid - from_lo;
    } else if (from_lo - between >= kreq) {                      // above
        k0 = khi; span = 0xff800000u - khi + 1; need = kreq; n_in = from_lo - between;
    } else if (range == 1) {
        k0 = klo; span = 1; need = kreq - (from_lo - between); n_in = between;
    } else {
        const uint32_t step = res[0] << shift0;
        k0 = klo + step; span = min(range - step, 1u << shift0); need = kreq - (from_lo - between) - res[1]; n_in = res[2];
    }
    int32_t *out = a.idx + (int64_t)bh * a.max_k;
    if (tid == 0) a.n_selected[bh] = (int32_t)k_eff;
    for (int i = (int)k_eff + tid; i < a.max_k; i += kRowThreads) out[i] = -1;
    if (k_eff == 0) return;
    __syncthreads();
    for (bool ends_only = n_in > (uint32_t)seq / 8; n_in != need && n_in > (uint32_t)kRowPairs && span > 1; ends_only = false) {
        // (where an eighth of the row is in the bin they are likely equal scores, which would add up one behind
        // the other: only their ends first.  A sixteenth: counts the same, counts with a soft part 22.7, not 19.7)
        const int bits = 32 - __clz((int)(span - 1)), shift = bits > kHistBits ? bits - kHistBits : 0;
        for (int j = tid; j < kHistBins; j += kRowThreads) h[j] = 0;
        __syncthreads();
        uint32_t inv = 0, most = 0;                              // largest ~offset, largest offset
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t off = w[c][j] - (k0 - zero);
                if (off < span) {
                    if (!ends_only) atomicAdd(&h[off >> shift], 1u);
                    inv = max(inv, ~off);
                    most = max(most, off);
                }
            }
        inv = wave_umax(inv);
        most = wave_umax(most);
        if (lane == 0) s_ends[0][wave] = make_uint2(inv, most);
        __syncthreads();
        const uint2 ends = s_ends[0][lane & 15];
        const uint32_t least = ~wave_umax(ends.x), last = wave_umax(ends.y);
        if (last == least || ends_only) {                        // (equal scores are one key at once)
            k0 += least;
            span = last - least + 1;
            __syncthreads();
            continue;
        }
        find([&](uint32_t) { return need; });
        const uint32_t step = res[0] << shift;
        k0 += step;
        span = min(span - step, 1u << shift);
        need -= res[1];
        n_in = res[2];
        __syncthreads();
    }
    // slots in position order of the scores that flags(c) picks: at[c] = those before this thread's four of chunk c
    uint32_t at[NC];
    auto place = [&](auto flags) {
        constexpr int NP = (NC + 1) / 2;
        uint32_t excl[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {                           // two chunks to a word: a wavefront has 256 scores of each
            const uint32_t n = (uint32_t)__popc(flags(2 * p)) | (2 * p + 1 < NC ? (uint32_t)__popc(flags(2 * p + 1)) << 16 : 0u);
            const uint32_t x = wave_incl_scan(n);
            excl[p] = x - n;
            if (lane == 63) {
                tot[(2 * p) * kRowWaves + wave] = x & 0xffffu;
                if (2 * p + 1 < NC) tot[(2 * p + 1) * kRowWaves + wave] = x >> 16;
            }
        }
        __syncthreads();
        if (wave == 0) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (4 * lane < NC * kRowWaves) v = *(const uint4 *)&tot[4 * lane];
            const uint32_t sum = v.x + v.y + v.z + v.w, e = wave_incl_scan(sum) - sum;
            *(uint4 *)&tot[4 * lane] = make_uint4(e, e + v.x, e + v.x + v.y, e + v.x + v.y + v.z);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NC; ++c) at[c] = tot[c * kRowWaves + wave] + ((excl[c >> 1] >> (16 * (c & 1))) & 0xffffu);
    };
    // ---- selected: keys from cut on; with ties across the cut, those equal to it only up to position cut_pos
    uint32_t cut = k0;
    int32_t cut_pos = 0x7fffffff;
    if (n_in != need && n_in <= (uint32_t)kRowPairs) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t off = w[c][j] - (k0 - zero);
                if (off < span) {
                    const uint32_t n = atomicAdd(&s_n, 1u);      // (n_in of them)
                    if (n < (uint32_t)kRowPairs) ck[n] = ((unsigned long long)(k0 + off) << 32) | (0x7fffffffu - (uint32_t)(c * kSlice + 4 * tid + j));
                }
            }
        if (tid < 4) ck[n_in + tid] = 0;                         // (whole quads; beats nobody)
        __syncthreads();
        const uint32_t i = (uint32_t)tid >> 2;                   // four lanes share a candidate
        if (i < n_in) {
            const unsigned long long me = ck[i];
            uint32_t rank = 0;
            for (uint32_t o = 4 * (tid & 3); o < n_in; o += 16) {
                const ulonglong2 c0 = *(const ulonglong2 *)&ck[o], c1 = *(const ulonglong2 *)&ck[o + 2];
                rank += (c0.x > me) + (c0.y > me) + (c1.x > me) + (c1.y > me);
            }
            rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0xB1, 0xF, 0xF, true);    // lane ^ 1
            rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0x4E, 0xF, 0xF, true);    // lane ^ 2
            if (rank == need - 1) s_cut = me;                    // the last one kept (its four lanes)
            if (rank == need) s_next = me;                       // the first one left
        }
        __syncthreads();
        cut = (uint32_t)(s_cut >> 32);
        if ((uint32_t)(s_next >> 32) == cut) cut_pos = (int32_t)(0x7fffffffu - (uint32_t)s_cut);
    } else if (n_in != need) {                                   // ties on one key: the position of the need-th of them
        auto ties = [&](int c) {
            uint32_t f = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) f |= (uint32_t)(w[c][j] == k0 - zero) << j;
            return f;
        };
        place(ties);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint32_t f = ties(c);
            if (at[c] < need && need <= at[c] + (uint32_t)__popc(f)) {
                for (uint32_t m = need - at[c]; m > 1; --m) f &= f - 1;
                s_cut = (unsigned long long)(c * kSlice + 4 * tid + __ffs((int)f) - 1);
            }
        }
        __syncthreads();
        cut_pos = (int32_t)s_cut;
    }
    // ---- the row of positions, in ascending order
    const uint32_t from = cut - zero, top = 0xff800000u - cut;   // kept: from .. +inf, with ties less those behind cut_pos
    uint32_t flags[(NC + 7) / 8] = {};                           // four bits a chunk
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) flags[c / 8] |= (uint32_t)(w[c][j] - from <= top) << (4 * (c % 8) + j);
    if (cut_pos != 0x7fffffff)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (w[c][j] == from && c * kSlice + 4 * tid + j > cut_pos) flags[c / 8] &= ~(1u << (4 * (c % 8) + j));
    auto kept = [&](int c) { return (flags[c / 8] >> (4 * (c % 8))) & 15u; };
    place(kept);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        for (uint32_t f = kept(c), i = at[c]; f != 0; f &= f - 1, ++i) out[i] = c * kSlice + 4 * tid + __ffs((int)f) - 1;
}

typedef void (*row_fn_t)(TopkArgs);
template <int NC> static row_fn_t row_kernel(int n_regions) {
    if constexpr (NC > kRowRegionsMany) return nullptr;
    else return n_regions == NC ? topk_row_kernel<NC> : row_kernel<NC + 1>(n_regions);
}
// (by the context's capacity: the lengths are on the device)
static row_fn_t pick_row(int n_regions, int rows) {
    return n_regions <= (rows >= kRowRowsMany ? kRowRegionsMany : kRowRegions) ? row_kernel<1>(n_regions) : nullptr;
}

// Everything up to the sweep: the threshold and the two unordered lists (selected outright,
// candidates in the threshold bin).  The fused decode step continues from those lists.
static void launch_sweep(const TopkArgs &a, dim3 grid, hipStream_t st) {
    if (a.adaptive) {
        hipLaunchKernelGGL((a.refine ? topk_filter_kernel<true, true> : topk_filter_kernel<true, false>), grid, dim3(kTopkThreads), 0, st, a);
    } else {
        hipLaunchKernelGGL(topk_hist2_kernel, grid, dim3(kTopkThreads), 0, st, a);
        hipLaunchKernelGGL((topk_filter_kernel<false, false>), grid, dim3(kTopkThreads), 0, st, a);
    }
}
int launch_topk_sweep(socket_ctx *ctx, const float *scores, const int32_t *seq_len, const int32_t *k,
                      int batch, int32_t *idx, int32_t *n_selected, int hist_mode, hipStream_t st) {
    launch_sweep(topk_args(ctx, scores, seq_len, k, idx, n_selected, hist_mode), dim3(ctx->g.n_regions, ctx->g.Hkv, batch), st);
    return record_hip(ctx, hipGetLastError());
}

int launch_topk(socket_ctx *ctx, const float *scores, const int32_t *seq_len, const int32_t *k,
                int batch, int32_t *idx, int32_t *n_selected, int hist_mode, hipStream_t st) {
    const dim3 grid(ctx->g.n_regions, ctx->g.Hkv, batch);
    TopkArgs a = topk_args(ctx, scores, seq_len, k, idx, n_selected, hist_mode);
    const int rows = batch * ctx->g.Hkv;
    const row_fn_t row_fn = hist_mode == kHistNone ? pick_row(ctx->g.n_regions, rows) : nullptr;
    if (row_fn) {
        hipLaunchKernelGGL(row_fn, dim3(rows), dim3(kRowThreads), 0, st, a);
        return record_hip(ctx, hipGetLastError());
    }
    if (hist_mode == kHistNone) {                // bins from the scores themselves
        a.adaptive = a.refine = 1;
        hipLaunchKernelGGL(topk_hist_kernel, grid, dim3(kTopkThreads), 0, st, a);
    }
    launch_sweep(a, grid, st);
    constexpr size_t long_lds = kLongLds > kEmitLds ? kLongLds : kEmitLds, resolve_lds = kResolveLds > kEmitLds ? kResolveLds : kEmitLds;
    static_assert(long_lds <= 64 * 1024 && resolve_lds <= 64 * 1024, "within the default dynamic LDS limit");
    if (a.refine) hipLaunchKernelGGL(topk_emit_kernel<true>, grid, dim3(kTopkThreads), long_lds, st, a);
    else hipLaunchKernelGGL(topk_emit_kernel<false>, grid, dim3(kTopkThreads), resolve_lds, st, a);
    return record_hip(ctx, hipGetLastError());
}

}  // namespace sk
