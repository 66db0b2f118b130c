// Alg. 3, TopK step: exact selection of the k largest scores per (sequence, KV head) by a
// most-significant-digit radix select on the fp32 bit patterns, spread over many workgroups.
//
//   topk_hist_kernel    adaptive histogram (bins from a sample of the row) of every valid score;
//                       the fused decode step gets it from the scoring pass instead, with bins
//                       sized from the bucket-probability tables.
//   topk_filter_kernel<true>  finds the threshold bin, then sweeps: scores above it are selected,
//                       scores in it are candidates (a few dozen unless many scores tie).
//   topk_emit_kernel    a workgroup per region of the sweep ranks the candidates on the score and
//                       then on the token position (smaller position wins a tie) and writes its
//                       part of the index row in ascending order.  Leaves histograms and counters
//                       at zero.
// Where the scoring pass could not size bins it leaves a histogram of leading 11-bit digits:
//   topk_hist2_kernel   finds the threshold digit, then histograms the next 11 bits over the
//                       scores in that digit.
//   topk_filter_kernel<false>  the sweep with the two-digit threshold.
// Stages talk through global memory across kernel boundaries only: no workgroup waits on
// another and no fence is needed.  LDS arrays that a thread walks in runs of PER consecutive
// words carry one pad word per run, which makes those walks free of bank conflicts.
#include "topk_device.h"

namespace sk {

// Adaptive histogram of a row nobody has binned yet.  The bins need a mean and a spread: every
// workgroup takes them from the same 512 scores of the row, spread evenly, so all of them (and,
// through the threshold record, the sweep) bin alike.  Scores further than four deviations from
// the mean are left out and both taken again, so that a few spikes do not widen the bins.
// At most a share f of any numbers lies sqrt(f / (1 - f)) deviations below their mean or higher
// (one-sided Chebyshev), so the k-th largest score is above mean - 0.34 deviations for f = 0.1 and
// mean - 0.58 for f = 0.25: the bins start half a deviation or one below the mean there, and are
// a 256th of a deviation wide where thresholds usually lie.  Which bins only decides how short
// the candidate list is; the select is exact for any.  (Laying the bins between two order
// statistics of 256 sampled scores instead bore any distribution, but cost 3.7 us more.)
__global__ __launch_bounds__(kTopkThreads) void topk_hist_kernel(TopkArgs a) {
    constexpr int NW = kTopkThreads / 64;
    __shared__ uint32_t h[kHistBins];
    __shared__ float part[2][3][NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bh = blockIdx.y, b = bh / a.Hkv;
    const int key0 = blockIdx.x * kSlice;
    const int i = key0 + tid * kPer;
    const float *row = a.scores + (int64_t)bh * a.max_n;
    float e[kPer];
    load_scores(row, i, a.max_n, e);
    const int seq = clamp_len(a.seq_len[b], a.max_n);
    const int kreq = clamp_len(a.k[b], a.max_k);
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
        if (i + j < key1 && selectable(e[j])) atomicAdd(&h[score_bin(e[j], lo, inv)], 1u);
    __syncthreads();
    uint32_t *gh = a.hist + (int64_t)bh * kHistBins;
    for (int j = tid; j < kHistBins; j += kTopkThreads)
        if (h[j]) atomicAdd(&gh[j], h[j]);
}

// First threshold digit, then the histogram of the second digit over the scores in it.
__global__ __launch_bounds__(kTopkThreads) void topk_hist2_kernel(TopkArgs a) {
    constexpr int PER = kHistBins / kTopkThreads;
    __shared__ uint32_t h[padded_size<kHistBins, PER>()];
    __shared__ uint32_t tmp[16];
    __shared__ uint32_t res[4];
    const int tid = threadIdx.x;
    const int bh = blockIdx.y, b = bh / a.Hkv;
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
template <bool ADAPT>
__global__ __launch_bounds__(kTopkThreads) void topk_filter_kernel(TopkArgs a) {
    constexpr int PER = kHistBins / kTopkThreads;
    __shared__ uint32_t h[padded_size<kHistBins, PER>()];
    __shared__ uint32_t tmp[16];
    __shared__ uint32_t res[4];
    __shared__ uint32_t s_base[2];
    const int tid = threadIdx.x;
    const int bh = blockIdx.y, b = bh / a.Hkv;
    const int key0 = blockIdx.x * kSlice;
    const int i = key0 + tid * kPer;
    float e[kPer];
    load_scores(a.scores + (int64_t)bh * a.max_n, i, a.max_n, e);
    const uint32_t *gh = (ADAPT ? a.hist : a.hist2) + (int64_t)bh * kHistBins;
    uint32_t c2[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) c2[j] = gh[tid + j * kTopkThreads];
    uint32_t *thr = a.thr + (int64_t)bh * kThrStride;
    const int key1 = min(key0 + kSlice, clamp_len(a.seq_len[b], a.max_n));
    // this workgroup's region of the selected list: empty unless the sweep below says otherwise
    uint32_t *selcnt = a.sel_cnt + (int64_t)bh * a.n_regions + blockIdx.x;
    if (tid == 0) *selcnt = 0u;
    uint32_t k_eff, pair, above, n_cand;
    float bin_lo = 0.0f, bin_inv = 0.0f;
    if (ADAPT) {
        bin_lo = __uint_as_float(thr[kThrBinLo]);
        bin_inv = __uint_as_float(thr[kThrBinInv]);
        const uint32_t kreq = (uint32_t)clamp_len(a.k[b], a.max_k);
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
        k_eff = thr[0];
        const uint32_t tb1 = thr[1], above1 = thr[2];
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
        const uint32_t lead = ADAPT ? score_bin(e[j], bin_lo, bin_inv) : keys[j] >> kDigit2Shift;
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
}

// The index row, from the sweep's regions and candidates: one workgroup per region, each ranking
// the few candidates itself.  The regions one after the other are the positions selected outright
// in ascending order, so an entry's slot is the number of entries in earlier regions, its index
// in its own, and the kept candidates before it; a kept candidate's slot is the same counts for
// its position.  (One workgroup per row, walking all regions, took 8.4-9.5 us at 32768 scores, 8
// heads.  A whole select, launches back to back: 13.3 us, 19.6 with that kernel and two digit
// histograms; 131072 scores 15.2 / 22.9; 16 x 20000 scores 24.4 / 28.7; 4 M scores 39 us / 7.6 ms.)
// A list of more candidates than two per thread (mass ties) is left to the row's first workgroup
// (topk_resolve_body).
__global__ __launch_bounds__(kTopkThreads, 4) void topk_emit_kernel(TopkArgs a) {
    extern __shared__ __align__(16) uint32_t emit_lds[];
    constexpr int NT = kTopkThreads, NW = NT / 64;
    __shared__ uint32_t s_sum[2][NW];            // entries of earlier regions; kept candidates of earlier regions
    __shared__ uint32_t s_nown;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int reg = blockIdx.x, bh = blockIdx.y;
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
    if (n_cand > (uint32_t)kRankMax) {
        if (reg == 0) topk_resolve_body(a, bh, emit_lds);
        return;
    }
    int32_t *out = a.idx + (int64_t)bh * a.max_k;
    if (reg == 0) {                              // the rest of the row, the count, and the scratch for the next call
        for (int i = (int)k_eff + tid; i < a.max_k; i += NT) out[i] = -1;
        uint32_t *gh1 = a.hist + (int64_t)bh * kHistBins, *gh2 = a.hist2 + (int64_t)bh * kHistBins;
        for (int i = tid; i < kHistBins; i += NT) {
            gh1[i] = 0;
            gh2[i] = 0;
        }
        if (tid < 2) a.counters[(int64_t)bh * kCounterStride + tid] = 0;
        if (tid == 0) a.n_selected[bh] = (int32_t)k_eff;
    }
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

// Everything up to the sweep: the threshold and the two unordered lists (selected outright,
// candidates in the threshold bin).  The fused decode step continues from those lists.
int launch_topk_sweep(socket_ctx *ctx, const float *scores, const int32_t *seq_len, const int32_t *k,
                      int batch, int32_t *idx, int32_t *n_selected, int hist_mode, hipStream_t st) {
    const Geometry &g = ctx->g;
    const TopkArgs a = topk_args(ctx, scores, seq_len, k, idx, n_selected, hist_mode);
    dim3 grid((g.max_n + kSlice - 1) / kSlice, batch * g.Hkv);
    if (hist_mode == kHistAdaptive) {
        hipLaunchKernelGGL(topk_filter_kernel<true>, grid, dim3(kTopkThreads), 0, st, a);
    } else {
        hipLaunchKernelGGL(topk_hist2_kernel, grid, dim3(kTopkThreads), 0, st, a);
        hipLaunchKernelGGL(topk_filter_kernel<false>, grid, dim3(kTopkThreads), 0, st, a);
    }
    return record_hip(ctx, hipGetLastError());
}

int launch_topk(socket_ctx *ctx, const float *scores, const int32_t *seq_len, const int32_t *k,
                int batch, int32_t *idx, int32_t *n_selected, int hist_mode, hipStream_t st) {
    const Geometry &g = ctx->g;
    if (hist_mode == kHistNone) {                // bins from the scores themselves
        hist_mode = kHistAdaptive;
        hipLaunchKernelGGL(topk_hist_kernel, dim3(g.n_regions, batch * g.Hkv), dim3(kTopkThreads), 0, st,
                           topk_args(ctx, scores, seq_len, k, idx, n_selected, hist_mode));
    }
    int rc = launch_topk_sweep(ctx, scores, seq_len, k, batch, idx, n_selected, hist_mode, st);
    if (rc != SOCKET_OK) return rc;
    const TopkArgs a = topk_args(ctx, scores, seq_len, k, idx, n_selected, hist_mode);
    constexpr size_t lds = kResolveLds > kEmitLds ? kResolveLds : kEmitLds;
    static_assert(lds <= 64 * 1024, "within the default dynamic LDS limit");
    hipLaunchKernelGGL(topk_emit_kernel, dim3(g.n_regions, batch * g.Hkv), dim3(kTopkThreads), lds, st, a);
    return record_hip(ctx, hipGetLastError());
}

}  // namespace sk
