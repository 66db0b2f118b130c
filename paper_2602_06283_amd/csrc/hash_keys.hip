// Alg. 1 (PrecomputeKeyHashes): sign random projections of cached keys, packed into bucket ids.
//
// Kernels:
//   hash_mfma8_kernel  8- or 4-plane tables (one-byte ids), bf16 keys, and long runs of fp32 keys of up to
//                      128 channels in bf16 pieces: the W slab of a chunk of up to 64 tables (half a
//                      chunk at d = 256 and of fp32) sits in LDS as MFMA fragments, keys go from
//                      memory straight into registers, the ids are assembled in registers.
//   hash_mfma10_kernel the same structure for 10-plane tables with packed 10-bit ids.
//   hash_mfma_kernel   bf16 keys, any other shape: K[rows x d] * W[d x L*P] on bf16 MFMA
//                      (v_mfma_f32_32x32x16_bf16, fp32 accumulate), W held in registers,
//                      key tiles staged through LDS, sign bits taken from the accumulators'
//                      sign bit and packed into a per-key bit matrix in LDS.
//   hash_f32_kernel    other fp32 keys, or fewer than 64 rows of bf16 keys: fp32 MFMA
//                      (v_mfma_f32_32x32x2_f32), W held in registers.
//   hash_rows_kernel   up to four rows, or groups too wide for hash_f32_kernel (9 or 10 planes at
//                      d = 256, in groups of 32 tables): fp32 FMA, one
//                      thread per projection column, sign bits gathered with a wavefront ballot.
// The last three end in pack_codes(), which cuts the bit matrix into P-bit bucket ids and writes
// them in the rotated order the scoring kernel reads.
#include <algorithm>
#include <type_traits>

#include "socket_internal.h"

namespace sk {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

struct HashArgs {
    const void *K;
    const void *W;
    void *codes;
    const int32_t *row_begin;
    const int32_t *row_count;
    RowMap map;
    int d, L, P, LP, Lpad, S, cb;
    int GT;                // tables per group of the packed 10-bit layout, 0 = unpacked ids
    int rows_per_wg;
    int tables_per_chunk;  // tables one workgroup covers (mfma kernel)
    int n_chunks;
    int batch, max_rows;   // sequences, and a bound on every row_count
    int group;             // sequences whose runs a workgroup shares out as one (SeqUnits), at most 64
};

// The runs of keys of the `group` sequences of blockIdx.z as one row of units of 2^SHIFT keys,
// sequence after sequence: what a wavefront has to know to find the keys of a unit.  Lane i holds
// sequence i's run and the units up to its end.  Workgroups that share units out over this row do
// equal work whatever the lengths are; shared out sequence by sequence, one long run in a batch of
// short ones was left to the few workgroups of its own sequence (16384 keys among 15 x 100, 8 heads:
// bf16, d = 256, 64 tables of 8 planes 323 us, 47 now; fp32, d = 64, 60 tables of 10 682 / 175; in a
// batch of equal lengths the look-up costs 1 to 2 us).
template <int SHIFT> struct SeqUnits {
    int count, begin, group;
    uint32_t end;
    __device__ __forceinline__ explicit SeqUnits(const HashArgs &a) {
        const int i = threadIdx.x & 63, b = blockIdx.z * a.group + i;
        const bool mine = i < a.group && b < a.batch;
        count = mine ? min(a.row_count[b], a.max_rows) : 0;
        begin = mine ? a.row_begin[b] : 0;
        group = a.group;
        end = wave_incl_scan((uint32_t)(max(count, 0) + (1 << SHIFT) - 1) >> SHIFT);
    }
    __device__ __forceinline__ int total() const { return __builtin_amdgcn_readlane((int)end, 63); }
    // sequence, run and first row of `unit` < total()
    __device__ __forceinline__ void find(int unit, int *b, int *b_count, int *b_begin, int *r0) const {
        const int s = __popcll(__ballot(end <= (uint32_t)unit));
        const int before = s > 0 ? __builtin_amdgcn_readlane((int)end, s - 1) : 0;
        *b = blockIdx.z * group + s;
        *b_count = __builtin_amdgcn_readlane(count, s);
        *b_begin = __builtin_amdgcn_readlane(begin, s);
        *r0 = (unit - before) << SHIFT;
    }
};

// Cut `nrows` bit rows (LDS, stride `stride` words, bit j of a row = sign bit of the
// projection onto column first_table*P + j) into bucket ids and store them.
// tok[r] = logical token of row r, grow[r] = its row in the codes tensor (-1 = skip).
// Only tables in [first_table, first_table+ntab) are written; when the workgroup owns
// whole 4-byte words (whole == true) the ids go out as aligned dwords.
__device__ __forceinline__ void pack_codes(const uint32_t *bits, int stride, int nrows,
                                           const int *tok, const int64_t *grow, void *codes,
                                           int L, int P, int Lpad, int S, int cb,
                                           int first_table, int ntab, bool whole, int tid,
                                           int nthreads) {
    if (whole) {
        const int cpd = 4 / cb;             // ids per dword
        const int pos0 = (first_table >> 6) << 6;
        const int span = ((ntab + 63) >> 6) << 6;  // positions owned (whole 64-groups)
        const int dspan = (span < Lpad ? span : Lpad) / cpd;
        for (int i = tid; i < nrows * dspan; i += nthreads) {
            int r = i / dspan, dw = i - r * dspan;
            if (grow[r] < 0) continue;
            uint32_t word = 0;
            for (int e = 0; e < cpd; ++e) {
                int pos = pos0 + dw * cpd + e;
                int l = table_at(pos, tok[r], S);
                uint32_t code = 0;
                if (l < L && l >= first_table && l < first_table + ntab)
                    code = bit_field(bits + r * stride, (l - first_table) * P, P);
                word |= code << (8 * cb * e);
            }
            uint32_t *dst = (uint32_t *)((char *)codes + grow[r] * (int64_t)Lpad * cb) + pos0 / cpd + dw;
            *dst = word;
        }
    } else {
        for (int i = tid; i < nrows * Lpad; i += nthreads) {
            int r = i / Lpad, pos = i - r * Lpad;
            if (grow[r] < 0) continue;
            int l = table_at(pos, tok[r], S);
            uint32_t code = 0;
            if (l >= L) {
                if (first_table != 0) continue;   // padding positions belong to the first chunk
            } else if (l < first_table || l >= first_table + ntab) {
                continue;
            } else {
                code = bit_field(bits + r * stride, (l - first_table) * P, P);
            }
            int64_t at = grow[r] * (int64_t)Lpad + pos;
            if (cb == 1) ((uint8_t *)codes)[at] = (uint8_t)code;
            else ((uint16_t *)codes)[at] = (uint16_t)code;
        }
    }
}

// The same for the packed 10-bit layout: the workgroup owns groups g0 .. g0+ngrp-1 of GT
// tables whole, and every thread builds one aligned dword of a token's 160-bit id string
// (parts of the four or five ids that overlap it).
__device__ __forceinline__ void pack_codes_packed(const uint32_t *bits, int stride, int nrows,
                                                  const int *tok, const int64_t *grow, void *codes,
                                                  int L, int P, int Lpad, int GT, int first_table,
                                                  int ntab, int ngrp, int tid, int nthreads) {
    const int S = GT >> 4;
    const int g0 = first_table / GT;
    const int per_row = ngrp * S * 5;                // dwords per token
    for (int i = tid; i < nrows * per_row; i += nthreads) {
        const int r = i / per_row;
        int u = i - r * per_row;
        if (grow[r] < 0) continue;
        const int gl = u / (S * 5);
        u -= gl * (S * 5);
        const int sub = u / 5, wi = u - sub * 5;     // string, dword of the string
        const int grp = g0 + gl, t = tok[r];
        const uint32_t *row = bits + r * stride;
        uint32_t word = 0;
        const int s0 = (32 * wi) / 10;               // first id that reaches into this dword
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            const int sidx = s0 + e, at = 10 * sidx - 32 * wi;   // bit of the dword where the id starts
            if (sidx > 15 || at >= 32) break;
            const int l = grp * GT + packed_table_at(sub * 16 + sidx, t, S);
            uint32_t id = 0;
            if (l < L && l >= first_table && l < first_table + ntab) id = bit_field(row, (l - first_table) * P, P);
            word |= at >= 0 ? id << at : id >> -at;
        }
        *(uint32_t *)((char *)codes + packed_word(grow[r], grp, sub, wi, Lpad, GT)) = word;
    }
}

// ---------------------------------------------------------------------------------------
// fp32-FMA kernel: ROWS rows per workgroup, one thread per projection column.
// ---------------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ float load_elem(const T *p);
template <> __device__ __forceinline__ float load_elem<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float load_elem<uint16_t>(const uint16_t *p) { return bf16_to_f32(*p); }

template <typename T, int ROWS>
__global__ __launch_bounds__(256) void hash_rows_kernel(HashArgs a) {
    extern __shared__ uint32_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.y, b = blockIdx.z;
    const int count = a.row_count[b];
    const int r0 = blockIdx.x * ROWS;
    if (r0 >= count) return;
    const int nrows = min(ROWS, count - r0);
    const int bw = 2 * ((a.LP + 63) / 64);     // bit-row stride in words

    float *ks = (float *)smem;                         // [ROWS][d]
    uint32_t *bits = smem + ROWS * a.d;                // [ROWS][bw]
    int *tok = (int *)(bits + ROWS * bw);              // [ROWS]
    int64_t *grow = (int64_t *)(tok + ROWS + (ROWS & 1));  // [ROWS], 8-byte aligned

    if (tid < ROWS) {
        int t = a.row_begin[b] + r0 + tid;
        bool live = tid < nrows && t >= 0 && t < a.map.max_n;
        tok[tid] = t;
        grow[tid] = live ? a.map.row(b, h, t) : -1;
    }
    __syncthreads();
    const T *K = (const T *)a.K;
    for (int i = tid; i < ROWS * a.d; i += 256) {
        int r = i / a.d, c = i - r * a.d;
        ks[i] = grow[r] >= 0 ? load_elem<T>(K + grow[r] * a.d + c) : 0.0f;
    }
    for (int i = tid; i < ROWS * bw; i += 256) bits[i] = 0;
    __syncthreads();

    const T *W = (const T *)a.W + (int64_t)h * a.d * a.LP;
    for (int base = 0; base < a.LP; base += 256) {
        const int col = base + tid;
        float acc[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = 0.0f;
        if (col < a.LP) {
            for (int c = 0; c < a.d; ++c) {
                float w = load_elem<T>(W + (int64_t)c * a.LP + col);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) acc[r] = fmaf(ks[r * a.d + c], w, acc[r]);
            }
        }
        const int word = (base + wave * 64) >> 5;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            unsigned long long m = __ballot(col < a.LP && acc[r] >= 0.0f);
            if (lane == 0 && word < bw) {
                bits[r * bw + word] = (uint32_t)m;
                if (word + 1 < bw) bits[r * bw + word + 1] = (uint32_t)(m >> 32);
            }
        }
    }
    __syncthreads();
    if (a.GT)
        pack_codes_packed(bits, bw, ROWS, tok, grow, a.codes, a.L, a.P, a.Lpad, a.GT, 0, a.L, a.Lpad / a.GT, tid, 256);
    else
        pack_codes(bits, bw, ROWS, tok, grow, a.codes, a.L, a.P, a.Lpad, a.S, a.cb, 0, a.L, true, tid, 256);
}

// ---------------------------------------------------------------------------------------
// fp32 MFMA kernel: fp32 caches (not long runs of ids of 4 and 8 planes and up to 128 channels: see
// CloseList), and short runs of bf16 keys.  Long runs are bound by the fp32 matrix rate (147 TFLOP/s in a
// large product on this card): 8 heads x 8192 keys, 60 tables of 10 planes 123 us = 102 TFLOP/s; the FMA
// kernel above takes three times as long, for it re-reads W from L2 for every 16 rows.  Short runs are bound by the fetch of W:
// 17 rows of 64 tables 13 us (33 through the FMA kernel, whose W loads wait for each other).
// v_mfma_f32_32x32x2_f32 adds its two products to the accumulator one after the other, each
// as an FMA, channel 2 s before channel 2 s + 1: a projection here is bit for bit the sum that
// hash_rows_kernel forms, so the two give the same ids.
// A wavefront owns 32 columns and keeps their W in registers (A operand: d/2 words a lane) for
// the whole kernel; the workgroup walks its rows in tiles of 32 keys staged through LDS.  A
// staged row is [even channels][odd channels], so that a lane of half g (B operand: channel
// 2 s + g of key n) reads four k-steps with one ds_read_b128; the 16-byte row pad spreads the
// rows over all banks.  One barrier per tile, as in hash_mfma_kernel below.
// 32 columns a wavefront rather than 64: the registers then allow four wavefronts per SIMD at
// d = 128, and 10-plane groups (320 columns) fill ten wavefronts instead of leaving three of
// eight idle.
// ---------------------------------------------------------------------------------------
constexpr int kF32TileShift = 5, kF32Tile = 1 << kF32TileShift;   // keys per tile
constexpr int kF32BitWords = 17;           // words per bit row: 512 columns and a pad
template <int D> constexpr int f32_min_threads() { return D == 64 ? 256 : 512; }   // (fewer would stage more pieces a thread than registers allow)

// SHARE: a workgroup's tiles are an equal share of those of a group of sequences (SeqUnits), else a
// piece of one sequence
template <typename T, int D, bool SHARE>
__global__ __launch_bounds__(D <= 128 ? 1024 : 512) void hash_f32_kernel(HashArgs a) {
    typedef typename std::conditional<sizeof(T) == 2, uint2, uint4>::type Quad;   // four channels as stored
    constexpr int KS = D / 2;                  // MFMA k-steps
    constexpr int TILE = kF32Tile, BW = kF32BitWords;
    constexpr int ROWW = D + 4;                // words of a staged key row
    constexpr int NST = TILE * D / 4 / f32_min_threads<D>();   // 16-byte pieces of a tile per thread of the smallest workgroup
    extern __shared__ uint32_t smem[];
    float *kt = (float *)smem;                         // [2][TILE][ROWW]
    uint32_t *bits = smem + 2 * TILE * ROWW;           // [2][TILE][BW]
    int64_t *grow = (int64_t *)(bits + 2 * TILE * BW); // [3][TILE]
    int *tok = (int *)(grow + 3 * TILE);               // [3][TILE]

    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, g = lane >> 5;
    const int chunk = blockIdx.y % a.n_chunks, h = blockIdx.y / a.n_chunks;
    int b = blockIdx.z, count, begin;
    int wg_r0, wg_r1, left = 0;                // rows of a sequence to do, tiles of later sequences after them
    if constexpr (!SHARE) {
        count = a.row_count[b];
        wg_r0 = blockIdx.x * a.rows_per_wg;
        if (wg_r0 >= count) return;
        wg_r1 = min(count, wg_r0 + a.rows_per_wg);
        begin = a.row_begin[b];
    } else {
        const SeqUnits<kF32TileShift> units(a);
        const int total = units.total(), share = total / (int)gridDim.x, extra = total % (int)gridDim.x, x = blockIdx.x;
        left = share + (x < extra);
        if (left == 0) return;
        units.find(x * share + min(x, extra), &b, &count, &begin, &wg_r0);
    }
    auto take = [&]() {                        // as many of the tiles left as sequence b has from wg_r0 on
        const int tiles = min(left, (count - wg_r0 + TILE - 1) >> kF32TileShift);
        wg_r1 = min(count, wg_r0 + (tiles << kF32TileShift));
        left -= tiles;
    };
    if (SHARE) take();
    const int first_table = chunk * a.tables_per_chunk;
    const int ntab = max(0, min(a.tables_per_chunk, a.L - first_table));   // 0: a group of padding tables only
    const int ncols = ntab * a.P;

    Quad stage[NST];
    auto fetch = [&](int r0, int slot) {       // slot: which third of the row bookkeeping
#pragma unroll
        for (int v = 0; v < NST; ++v) {
            const int i = tid + v * nt, row = i / (D / 4), seg = i % (D / 4);
            if (i >= TILE * (D / 4)) break;
            const int t = begin + r0 + row;
            const bool live = r0 + row < wg_r1 && t >= 0 && t < a.map.max_n;
            const int64_t gr = live ? a.map.row(b, h, t) : -1;
            if (seg == 0) {
                tok[slot * TILE + row] = t;
                grow[slot * TILE + row] = gr;
            }
            stage[v] = gr >= 0 ? *((const Quad *)((const T *)a.K + gr * D) + seg) : Quad{};
        }
    };
    auto commit = [&](int buf) {
#pragma unroll
        for (int v = 0; v < NST; ++v) {
            const int i = tid + v * nt, row = i / (D / 4), seg = i % (D / 4);
            if (i >= TILE * (D / 4)) break;
            uint32_t *dst = (uint32_t *)(kt + (buf * TILE + row) * ROWW) + 2 * seg;
            if constexpr (sizeof(T) == 2) {
                *(uint2 *)dst = make_uint2(stage[v].x << 16, stage[v].y << 16);
                *(uint2 *)(dst + D / 2) = make_uint2(stage[v].x & 0xffff0000u, stage[v].y & 0xffff0000u);
            } else {
                *(uint2 *)dst = make_uint2(stage[v].x, stage[v].z);
                *(uint2 *)(dst + D / 2) = make_uint2(stage[v].y, stage[v].w);
            }
        }
    };
    fetch(wg_r0, 0);

    // ---- this wavefront's 32 columns of W: lane (column n, half g) holds channels 2 s + g
    const int col = wave * 32 + n;
    const T *Wg = (const T *)a.W + (int64_t)h * D * a.LP + first_table * a.P;
    // (a lane beyond the last column reads that column again: its bits are never packed)
    float wr[KS];
    if (wave * 32 < ncols) {
        const T *Wc = Wg + (int64_t)g * a.LP + min(col, ncols - 1);
        T raw[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) raw[s] = Wc[(int64_t)(2 * s) * a.LP];
#pragma unroll
        for (int s = 0; s < KS; ++s) wr[s] = load_elem<T>(raw + s);
    }

    const bool whole = a.n_chunks == 1 || (a.tables_per_chunk & 63) == 0;
    int buf = 0, slot = 0;                     // (turn on over sequences: the same waits cover their first tiles)
    for (;;) {
        commit(buf);
        __syncthreads();
        for (int r0 = wg_r0; r0 < wg_r1; r0 += TILE) {
            const bool more = r0 + TILE < wg_r1;
            const int nslot = slot == 2 ? 0 : slot + 1;
            if (more) fetch(r0 + TILE, nslot);
            uint32_t *bt = bits + buf * (TILE * BW);
            if (wave * 32 < ncols) {
                floatx16_t acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
                const float4 *src = (const float4 *)(kt + (buf * TILE + n) * ROWW + g * (D / 2));
#pragma unroll
                for (int s4 = 0; s4 < KS / 4; ++s4) {
                    const float4 kf = src[s4];
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[4 * s4], kf.x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[4 * s4 + 1], kf.y, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[4 * s4 + 2], kf.z, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[4 * s4 + 3], kf.w, acc, 0, 0, 0);
                }
                // accumulator i of lane (n, g) is plane 8 (i/4) + 4g + i%4 of key n
                uint32_t word = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) word |= (acc[i] >= 0.0f ? 1u : 0u) << (8 * (i / 4) + i % 4);
                word <<= 4 * g;
                auto both = __builtin_amdgcn_permlane32_swap(word, word, false, false);
                if (lane < 32) bt[n * BW + wave] = both[0] | both[1];
            }
            if (more) commit(buf ^ 1);
            __syncthreads();   // bit matrix complete, next tile staged, every wave done with this key tile
            const int *tk = tok + slot * TILE;
            const int64_t *gr = grow + slot * TILE;
            if (a.GT)
                pack_codes_packed(bt, BW, TILE, tk, gr, a.codes, a.L, a.P, a.Lpad, a.GT, first_table, ntab, 1, tid, nt);
            else
                pack_codes(bt, BW, TILE, tk, gr, a.codes, a.L, a.P, a.Lpad, a.S, a.cb, first_table, ntab, whole, tid, nt);
            buf ^= 1;
            slot = nslot;
        }
        if (!SHARE || left <= 0) return;
        do {                                   // (tiles are left, so a sequence behind has them)
            if (++b >= a.batch) return;
            count = min(a.row_count[b], a.max_rows);
        } while (count <= 0);
        begin = a.row_begin[b];
        wg_r0 = 0;
        take();
        fetch(wg_r0, slot);
    }
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA kernel.  512 threads = 8 waves; wave w owns projection columns
// [64w, 64w+64) of the workgroup's column chunk and keeps that slab of W in registers
// for the whole kernel.  The workgroup walks its rows in tiles of 64 keys, staged through
// LDS; a tile is multiplied as two halves of 32 keys so that the accumulators take 32
// registers and two workgroups fit a CU.
// MFMA operands: A = W^T (32 planes x 16 channels), B = K^T (16 channels x 32 keys), so
// lane (key n, half g) of the accumulator holds planes 8a + 4g + b (a,b in 0..3) of key n.
// One barrier per tile: the bit matrix is double-buffered and the row bookkeeping
// triple-buffered, so the waves that have finished a tile's products pack its ids while the
// others still multiply, and nobody waits a second time.
// ---------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(512, D <= 128 ? 4 : 2) void hash_mfma_kernel(HashArgs a) {
    constexpr int KS = D / 16;                 // MFMA k-steps
    constexpr int TILE = 64;                   // keys per tile
    constexpr int KSTRIDE = D * 2 + 16;        // bytes per staged key row (padded)
    constexpr int BSTRIDE = 17;                // words per bit row (16 + 1 pad)
    extern __shared__ uint32_t smem[];
    char *const kbase = (char *)smem;                  // two staged key tiles
    auto ktile = [&](int bf) { return kbase + bf * (TILE * KSTRIDE); };
    uint32_t *bits = smem + 2 * TILE * KSTRIDE / 4;   // [2][TILE][BSTRIDE]
    int *tok = (int *)(bits + 2 * TILE * BSTRIDE);    // [3][TILE]
    int64_t *grow = (int64_t *)(tok + 4 * TILE);      // [3][TILE] (8-byte aligned)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = blockIdx.y % a.n_chunks, h = blockIdx.y / a.n_chunks, b = blockIdx.z;
    const int count = a.row_count[b];
    const int wg_r0 = blockIdx.x * a.rows_per_wg;
    if (wg_r0 >= count) return;
    const int wg_r1 = min(count, wg_r0 + a.rows_per_wg);
    const int begin = a.row_begin[b];

    const int first_table = chunk * a.tables_per_chunk;
    const int ntab = max(0, min(a.tables_per_chunk, a.L - first_table));   // 0: a group of padding tables only
    const int ncols = ntab * a.P;              // live columns of this chunk (<= 512)
    const int col0 = first_table * a.P;

    // ---- this wave's slab of W as MFMA A-operand fragments: plane m = lane%32, channels
    //      16*ks + 8*(lane/32) .. +7
    const uint16_t *W = (const uint16_t *)a.W + (int64_t)h * D * a.LP;
    bf16x8_t wfrag[2][KS];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const int j = wave * 64 + mb * 32 + (lane & 31);      // chunk-local column
        const bool live = j < ncols;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            union { bf16x8_t v; uint16_t u[8]; } f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int c = ks * 16 + (lane >> 5) * 8 + e;
                f.u[e] = live ? W[(int64_t)c * a.LP + col0 + j] : (uint16_t)0;
            }
            wfrag[mb][ks] = f.v;
        }
    }

    // ---- tile staging: thread -> (row = tid / 8, 1/8 of the row)
    constexpr int SEG = D * 2 / 8;             // bytes of a row each thread stages (16, 32 or 64)
    const int srow = tid >> 3, sseg = tid & 7;
    uint4 stage[SEG / 16];

    auto fetch = [&](int tile_r0, int slot) {  // slot: which third of the row bookkeeping
        int r = tile_r0 + srow;
        int t = begin + r;
        bool live = r < wg_r1 && t >= 0 && t < a.map.max_n;
        int64_t g = live ? a.map.row(b, h, t) : -1;
        if (sseg == 0) {
            tok[slot * TILE + srow] = t;
            grow[slot * TILE + srow] = g;
        }
        const char *src = (const char *)a.K + g * (int64_t)(D * 2) + sseg * SEG;
#pragma unroll
        for (int v = 0; v < SEG / 16; ++v)
            stage[v] = g >= 0 ? ((const uint4 *)src)[v] : make_uint4(0, 0, 0, 0);
    };
    auto commit = [&](int buf) {
        char *dst = ktile(buf) + srow * KSTRIDE + sseg * SEG;
#pragma unroll
        for (int v = 0; v < SEG / 16; ++v) ((uint4 *)dst)[v] = stage[v];
    };

    // ids of P = 8 planes are the bytes of a bit row, and the rotated order moves whole bytes:
    // position 64c + 16 sub + s of token t holds table 64c + sub + 4 ((t + s) mod 16)
    const bool byte_ids = a.P == 8 && a.S == 4 && (a.tables_per_chunk == 64 || a.n_chunks == 1);
    const bool whole = a.n_chunks == 1 || (a.tables_per_chunk & 63) == 0;

    fetch(wg_r0, 0);
    commit(0);
    __syncthreads();

    int buf = 0, slot = 0;
    for (int tile_r0 = wg_r0; tile_r0 < wg_r1; tile_r0 += TILE) {
        const bool more = tile_r0 + TILE < wg_r1;
        const int nslot = slot == 2 ? 0 : slot + 1;
        if (more) fetch(tile_r0 + TILE, nslot);
        uint32_t *bt = bits + buf * (TILE * BSTRIDE);

#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            // ---- MFMA: acc[mb] = W^T slab (32 planes) x K^T (32 keys)
            floatx16_t acc[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mb][i] = 0.0f;
            const char *src = ktile(buf) + (nb * 32 + (lane & 31)) * KSTRIDE + (lane >> 5) * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8_t kf = *(const bf16x8_t *)(src + ks * 32);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag[0][ks], kf, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag[1][ks], kf, acc[1], 0, 0, 0);
            }
            // ---- sign bits: accumulator i of lane (n, g) is plane 8*(i/4) + 4g + i%4.
            //      Funnel-shift the 16 sign bits into one 16-bit value per lane, exchange with
            //      the other half-wave, and interleave nibbles into the 32 planes of the block.
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                uint32_t neg = __float_as_uint(acc[mb][15]) >> 31;
#pragma unroll
                for (int i = 14; i >= 0; --i)
                    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[mb][i]), 31);
                neg &= 0xffffu;                         // bit 4a+b = sign of plane 8a+4g+b
                auto both = __builtin_amdgcn_permlane32_swap(neg, neg, false, false);
                uint32_t lo = both[0], hi = both[1];    // the g = 0 and g = 1 halves of key n, in every lane
                lo = (lo | (lo << 8)) & 0x00ff00ffu;
                lo = (lo | (lo << 4)) & 0x0f0f0f0fu;
                hi = (hi | (hi << 8)) & 0x00ff00ffu;
                hi = (hi | (hi << 4)) & 0x0f0f0f0fu;
                const uint32_t word = ~(lo | (hi << 4)); // bit p = 1 when plane p projects >= 0
                if (lane < 32) bt[(nb * 32 + lane) * BSTRIDE + wave * 2 + mb] = word;
            }
        }
        if (more) commit(buf ^ 1);
        __syncthreads();   // bit matrix complete, next tile staged, every wave done with this key tile

        const int *tk = tok + slot * TILE;
        const int64_t *gr = grow + slot * TILE;
        if (byte_ids) {
            // thread -> (row, 16-position group, half of it): 8 ids = 8 byte reads, one 8-byte store
            const int r = tid >> 3, sub = (tid >> 1) & 3, half = tid & 1;
            const int64_t g = gr[r];
            if (g >= 0) {
                const int t = tk[r];
                const uint8_t *rowb = (const uint8_t *)(bt + r * BSTRIDE);
                uint32_t out[2] = {0u, 0u};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int tbl = sub + 4 * ((t + half * 8 + e) & 15);     // chunk-local table
                    const uint32_t id = tbl < ntab ? rowb[tbl] : 0u;
                    out[e >> 2] |= id << (8 * (e & 3));
                }
                const int pos0 = (first_table >> 6) << 6;
                *(uint2 *)((char *)a.codes + g * (int64_t)a.Lpad + pos0 + sub * 16 + half * 8) = make_uint2(out[0], out[1]);
            }
        } else if (a.GT) {
            pack_codes_packed(bt, BSTRIDE, TILE, tk, gr, a.codes, a.L, a.P, a.Lpad, a.GT, first_table, ntab, 1,
                              tid, 512);
        } else {
            pack_codes(bt, BSTRIDE, TILE, tk, gr, a.codes, a.L, a.P, a.Lpad, a.S, a.cb, first_table, ntab,
                       whole, tid, 512);
        }
        buf ^= 1;
        slot = nslot;
    }
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA kernel for 8- and 4-plane tables (one-byte ids): the fast path (fp32 keys: in pieces, CloseList).
// A workgroup keeps the W slab of one 64-table chunk (512 columns) in LDS, already cut into
// MFMA A-operand fragments, and each of its 16 wavefronts works on 64-key blocks of its own:
// the keys go from memory straight into B-operand registers, so there is no staging, no
// barrier in the main loop, and the wavefronts drift apart - some multiply while others pack.
//
// Column order (S = 4 position groups of 16 ids per 64-table chunk; rows of 16 or 32 ids have
// S = 1 or 2 and read 4 as S below).  Position 16 sub + s of token t holds table
// sub + 4 ((t + s) mod 16).  The
// 32-column block p = 4 sub + q therefore holds tables sub + 4 (4q + e), e = 0..3: after four
// blocks the wavefront has, for each key, the 16 ids of position group `sub` in table order
// j = 4q + e as the 16 bytes of four sign words, and the stored group is those bytes rotated
// by t mod 16.
// Row order inside a block.  MFMA operands: A = W^T (32 rows x 16 channels), B = K^T
// (16 channels x 32 keys); accumulator i of lane (key n, half g) is row 8 (i/4) + 4g + i%4.
// Row m is given plane (table e, plane pl) with 8e + pl = 16 g + i, so that the 16 sign bits a
// lane collects from its accumulators are, in order, one half of the key's 32-bit sign word.
// cut_fragments lays W out that way.
// ---------------------------------------------------------------------------------------
template <int V> struct IntTag { static constexpr int value = V; };

constexpr int kHash8Threads = 1024;

typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// Two adjacent channels in two bf16 pieces, rounded to nearest: the hi pieces, lo gets the others.
__device__ __forceinline__ uint32_t cut_pair(floatx2_t v, uint32_t *lo) {
    const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
    const floatx2_t left = {v.x - __uint_as_float(hi << 16), v.y - __uint_as_float(hi & 0xffff0000u)};
    *lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(left, bf16x2_t));
    return hi;
}

// The A fragments of a workgroup of the two fast kernels, cut from W into LDS by the workgroup itself:
// a thread takes one table (P columns) and eight channels, eight loads of 2 P bytes in flight, and
// transposes them in registers into P pieces of eight channels each.  (A launch of its own that laid
// the fragments out in memory first cost 4 to 5 us by itself, 2 to 3 back to back with this one:
// 777 + 333 rows of (10, 60) with their value norms 18.8 us with it, 16.2 without (15.4 since short runs
// share blocks); 4 heads x 32768 keys, d = 256, 37.8 / 35.1; 4 sequences of 65536 keys, 8 heads of
// (8, 64), 241.6 / 240.3, where two runs of one side differ by 0.7.)
// The workgroup's tables are tab0 + (i / NG) * S + i % NG: NG of the S interleaved position groups.
// Column P j + pl of position group `sub` (j = its j-th table) is bit u % 32 of sign word u / 32,
// u = P j + pl; wl holds word q of the workgroup's group sl as block sl BPG + q.
// Pieces of a block are kept at lane ^ frag_turn(sl, q), or the tables that the lanes of a
// wavefront write side by side would share banks.
__device__ __forceinline__ int frag_turn(int sl, int q) { return (sl ^ q) & 3; }

// fp32: W goes in two bf16 pieces, a block's hi fragments before its lo fragments.  Columns without a
// table repeat the last one's there (a sum of zero would look like a sign too close to call).
// `meanwhile` is called once, the thread's last loads of W on their way.
template <typename T, int D, int S, int P, int NG, int NT, typename F>
__device__ __forceinline__ void cut_fragments(uint4 *wl, const HashArgs &a, int h, int first_table, int ntab, int sub0, int tid, F &&meanwhile) {
    constexpr bool SPLIT = sizeof(T) == 4;
    constexpr int KS = D / 16, KF = SPLIT ? 2 * KS : KS, BPG = P / 2, NTAB = 16 * NG, ITEMS = NTAB * (D / 8);
    constexpr int ND = P * (int)sizeof(T) / 4;         // dwords of a table's row
    constexpr int PER = (ITEMS + NT - 1) / NT;
    static_assert(P == 4 || P == 8 || P == 10, "whole dwords");
    // rows of W start at any element: L P and the caller's pointer say nothing about alignment
    struct __attribute__((packed, aligned(sizeof(T)))) Row { uint32_t w[ND]; };
    const T *W = (const T *)a.W + ((int64_t)h * D * a.LP + (int64_t)first_table * P);
    auto cut = [&](int i, auto &&between) __attribute__((always_inline)) {
        int ti = i % NTAB;
        const int oct = i / NTAB;                      // channels 8 oct .. 8 oct + 7
        // (eight adjacent lanes: four groups, both halves of a sign word)
        if (S == 4 && NG == 4 && P == 8) ti = (ti & ~12) | ((ti >> 1) & 4) | ((ti << 1) & 8);
        const int j = ti / NG, sl = ti % NG;
        int tt = j * S + sub0 + sl;                    // chunk-local table
        if (SPLIT) tt = min(tt, ntab - 1);
        Row r[8];
        if ((ITEMS % NT == 0 || i < ITEMS) && (SPLIT ? ntab > 0 : tt < ntab)) {
#pragma unroll
            for (int c = 0; c < 8; ++c) r[c] = *(const Row *)(W + (int64_t)(oct * 8 + c) * a.LP + tt * P);
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int w = 0; w < ND; ++w) r[c].w[w] = 0u;
        }
        between();
        if (ITEMS % NT != 0 && i >= ITEMS) return;
#pragma unroll
        for (int pl = 0; pl < P; ++pl) {
            const int u = P * j + pl, q = u >> 5, bit = u & 31;
            const int m = 8 * ((bit >> 2) & 3) + 4 * (bit >> 4) + (bit & 3);   // the MFMA row that becomes this bit
            uint4 *dst = wl + ((sl * BPG + q) * KF + (oct >> 1)) * 64 + (((oct & 1) * 32 + m) ^ frag_turn(sl, q));
            uint32_t o[4];
            if constexpr (SPLIT) {
                uint32_t lo[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = cut_pair(floatx2_t{__uint_as_float(r[2 * c].w[pl]), __uint_as_float(r[2 * c + 1].w[pl])}, lo + c);
                dst[KS * 64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            } else {
                const uint32_t pick = pl & 1 ? 0x07060302u : 0x05040100u;   // the high or the low halves of two words
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = __builtin_amdgcn_perm(r[2 * c + 1].w[pl >> 1], r[2 * c].w[pl >> 1], pick);
            }
            dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
        }
    };
#pragma unroll 1
    for (int k = 0; k + 1 < PER; ++k) cut(tid + k * NT, []() {});
    cut(tid + (PER - 1) * NT, meanwhile);
}

// ---------------------------------------------------------------------------------------
// fp32 keys on the bf16 matrix cores.  Keys and W are cut into two bf16 pieces each, x = hi + lo + rest
// with |lo| <= 2^-8 |x| and |rest| <= 2^-8 |lo|, and lo*hi + hi*lo, then hi*hi, are summed: three
// products at 16 times the fp32 matrix rate a product.  An id only takes the sign of a sum, so what the
// pieces leave out matters near zero alone: where |sum| is not above a bound on its distance to the sum
// that the FMA kernel forms (three projections in ten thousand for normal keys), the projection goes on
// the wavefront's list and is formed anew, channel by channel as the FMA kernel does; if the sign is the
// other one (one in ten million) the id is stored again.  A block with more of them than the list holds is
// formed anew whole, on the fp32 matrix cores.  The ids are those of the FMA kernel bit for bit.
// That block makes the time depend on the data where sums are close to zero by the dozen (8 heads, 8192
// keys, 32 tables, 28 us else and 48 on the fp32 matrix cores alone): all keys or all of W too small or too
// large for the bound 100, one key in a hundred of that kind 91, every key at right angles to one column
// of W 70.  (Sum by sum, a lane each, these took 1130, 201 and 88.)
// 8 heads, 32 tables of 8 planes, 128 channels, many calls on two caches in turn: 8192 keys 28 us (45 on the
// fp32 matrix cores), 32768 67 (154), where a block's matrix work is 12 of its 20 us and the rest the keys' way
// from memory, two wavefronts a SIMD being all that the registers allow; of a short run's time 14 us are
// launch, W and instructions that come cold.
// The bound, for a key k and a column w, with A >= the norm of a vector and B = the norm of its lo
// pieces (Cauchy-Schwarz turns norms into sums of magnitudes):
//   dropped products  lo*lo <= B_k B_w, rest*w <= 2^-8 B_k A_w, k*rest <= 2^-8 A_k B_w
//   FMA kernel        D roundings of 2^-24 of at most A_k A_w
//   matrix cores      D additions to the sum of hi*hi and a rounding of the result every 16, each off by
//                     2^-23 of at most A_k A_w if it truncates; the 2 D additions of lo products before
//                     them likewise, to sums 2^-7 as large
// together (2^-24 + 1.08 * 2^-23) D A_k A_w = 1.885e-7 D A_k A_w for the last two; 1.9e-7 and a hundredth more
// are taken (2.1e-7: a tenth more close sums, 0.4 us of 27).  That the matrix cores lose no more than the
// last place of an addition is an assumption, not documented; the tests compare the ids with the FMA
// kernel's where sums are rounding errors and nothing else.
// close_part gives a key's (x, y), bound = x A_w + y B_w.  Where squares leave the range of floats, with
// infinities and NaN, the bound is infinite and every projection formed anew.  The sums of an all-zero
// key or column are zero: they need none.
// ---------------------------------------------------------------------------------------
template <int D> __device__ __forceinline__ float2 close_part(float A, float B) {
    float2 e = make_float2(1.01f * (A * (D * 1.9e-7f) + B * 0.00391f), 1.01f * (B * 1.01f + A * 0.00391f));
    if (!(A > 1e-10f && A < 1e15f)) e = A == 0.0f ? make_float2(-1.0f, 0.0f) : make_float2(__builtin_inff(), __builtin_inff());
    return e;
}
// sum of the squares of eight bf16 pieces, on top of `sum`
__device__ __forceinline__ float add_squares(bf16x8_t v, float sum) {
    const uint4 w = __builtin_bit_cast(uint4, v);
    sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.x), __builtin_bit_cast(bf16x2_t, w.x), sum, false);
    sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.y), __builtin_bit_cast(bf16x2_t, w.y), sum, false);
    sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.z), __builtin_bit_cast(bf16x2_t, w.z), sum, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.w), __builtin_bit_cast(bf16x2_t, w.w), sum, false);
}
// What a block's columns have in common: the largest A and B (an infinity where one of them is out of
// range), and which of them are all zero, a bit for each as in a sign word.
struct CloseColumns {
    float A, B;
    uint32_t zero;
};
// frag: the block's fragments, of lane's MFMA row.  w: the row's column of W (the pieces of a number too
// small for bf16 are zero, its products may not be)
template <int D> __device__ __forceinline__ CloseColumns close_columns(const uint4 *frag, const float *w, int LP) {
    constexpr int KS = D / 16;
    float hi = 0.0f, lo = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        hi = add_squares(__builtin_bit_cast(bf16x8_t, frag[ks * 64]), hi);
        lo = add_squares(__builtin_bit_cast(bf16x8_t, frag[(KS + ks) * 64]), lo);
    }
    const float h2 = xor32_sum(hi), B = 1.01f * sqrtf(xor32_sum(lo)), A = 1.001f * sqrtf(h2) + B;
    const bool odd = __ballot(!(A < 1e15f)) != 0;              // (a NaN would be lost in the largest)
    const float most = wave_max(A);
    uint32_t zero = 0;
    if (__ballot(h2 == 0.0f) != 0) {
        uint32_t any = 0;
        for (int c = 0; c < D; ++c) any |= __float_as_uint(w[(int64_t)c * LP]) << 1;
        const uint32_t rows = (uint32_t)__ballot(any == 0);    // by MFMA row: nibbles 0, 2, .. are the first half of the word
        for (int i = 0; i < 8; ++i) zero |= (rows >> (4 * i) & 15u) << (4 * (i >> 1) + 16 * (i & 1));
    }
    return CloseColumns{odd || !(most > 1e-10f) ? __builtin_inff() : most, wave_max(B), zero};
}

struct CloseEntry {
    int64_t row;       // the key's row in K and in the ids
    int tok;
    uint32_t col;      // column of the workgroup's tables, and from bit 16 on the id as it was stored
};

// A wavefront's list.  Entries are settled when it is half full and after the last block.
// An id is mended by storing it whole, as the list knows it, and never from what memory holds: the
// row may be another wavefront's too (sequences that share a block), whose ids come before or after.
template <int D, int P, int S, int CAP> struct CloseList {
    static_assert(CAP <= 64, "a lane an entry");
    const HashArgs &a;
    CloseEntry *list;
    const float *W;                            // [D][LP], the workgroup's tables from column 0 on
    int first_table, ntab, n = 0;

    __device__ __forceinline__ CloseList(const HashArgs &args, CloseEntry *mine, int h, int first, int tables)
        : a(args), list(mine), W((const float *)args.W + (int64_t)h * D * args.LP + (int64_t)first * P), first_table(first), ntab(tables) {}

    // The column of W that is the lane's MFMA row in block q of position group `sub` (cut_fragments)
    __device__ __forceinline__ const float *column(int q, int sub) const {
        const int lane = threadIdx.x & 63, u = 32 * q + (lane & 3) + 4 * ((lane >> 3) & 3) + 16 * ((lane >> 2) & 1);
        return W + max(min(u / P * S + sub, ntab - 1), 0) * P + u % P;
    }

    // The signs (as in add) of a block's first or second keys, or both, where one of them is `near`: on the
    // fp32 matrix cores, whose sums are the FMA kernel's bit for bit (hash_f32_kernel), both operands
    // straight from memory.
    __device__ __forceinline__ uint32_t block_signs(uint32_t neg, uint32_t near, int q, int sub, int64_t row0, int64_t row1) const {
        const int lane = threadIdx.x & 63, g = lane >> 5;
        const float *w = column(q, sub) + (int64_t)g * a.LP;
#pragma unroll 1
        for (int nb = 0; nb < 2; ++nb) {
            if (__ballot((near >> (16 * nb) & 0xffffu) != 0) == 0) continue;
            const int64_t row = nb ? row1 : row0;
            const f32x4_t *k = (const f32x4_t *)((const float *)a.K + (row >= 0 ? row : 0) * D);
            floatx16_t acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll 4
            for (int c = 0; c < D / 4; ++c) {          // channels 4 c + g, then 4 c + 2 + g
                const f32x4_t x = k[c];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[(int64_t)(4 * c) * a.LP], g ? x.y : x.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[(int64_t)(4 * c + 2) * a.LP], g ? x.w : x.z, acc, 0, 0, 0);
            }
            uint32_t signs = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) signs |= (acc[i] >= 0.0f ? 0u : 1u) << i;
            neg = nb ? (neg & 0xffffu) | signs << 16 : (neg & 0xffff0000u) | signs;
        }
        return neg;
    }

    // The sums of a block's two keys of a lane: accumulator i of half g is bit 32 q + 16 g + i of position
    // group `sub`.  neg: their signs, the second key's from bit 16 on.  row(nb): the key's row in K, or -1.
    template <typename F>
    __device__ __forceinline__ void add(const floatx16_t &acc0, const floatx16_t &acc1, uint32_t &neg, const float2 *key, CloseColumns cols, int q, int sub, int tok, F &&row) {
        const int lane = threadIdx.x & 63, u0 = 32 * q + 16 * (lane >> 5);
        // one of the two: the sums that are not above the bound (near zero); none of a key without a row,
        // or of a column of zeros, whose sums are zero (but for infinities and NaN)
        auto look = [&](const floatx16_t &acc, int nb, int64_t *at) __attribute__((always_inline)) {
            const float inf = __builtin_inff(), bound = cols.A < inf ? fmaf(key[nb].x, cols.A, key[nb].y * cols.B) : inf;
            float least = fabsf(acc[0]);
#pragma unroll
            for (int i = 1; i < 16; ++i) least = fminf(least, fabsf(acc[i]));   // (a NaN comes with an infinite bound)
            uint32_t near = 0;
            if (__ballot(!(least > bound)) == 0) return near;
#pragma unroll
            for (int i = 15; i >= 0; --i) near = __builtin_amdgcn_alignbit(near, __float_as_uint(fabsf(acc[i]) - bound), 31);
            *at = row(nb);
            const uint32_t zero = key[nb].x < inf ? cols.zero >> (lane & 32 ? 16 : 0) : 0u;
            return *at < 0 ? 0u : (bound < inf ? near : 0xffffu) & ~zero;
        };
        int64_t row0 = -1, row1 = -1;
        uint32_t near = look(acc0, 0, &row0);
        near |= look(acc1, 1, &row1) << 16;
        if (__ballot(near != 0) == 0 || ntab <= 0) return;
        auto table = [&](int i) { return (u0 + (i & 15)) / P * S + sub; };
        if ((32 * q + 31) / P * S + sub >= ntab) {
#pragma unroll
            for (int i = 0; i < 16; i += P)
                if (table(i) >= ntab) near &= ~(0x10001u * (((1u << P) - 1) << i));
        }
        const int before = n;
        uint64_t m;
        for (uint32_t left = near; (m = __ballot(left != 0)) != 0; left &= left - 1) {
            const int i = __ffs((int)left) - 1, more = (int)__popcll(m);
            if (n + more > CAP) {                      // (keys by the hundred at right angles to W, or out of range)
                n = before;
                neg = block_signs(neg, near, q, sub, row0, row1);
                return;
            }
            const uint32_t id = ~(neg >> (i & ~(P - 1))) & ((1u << P) - 1);
            if (left != 0)
                list[n + __popcll(m & ((1ull << lane) - 1))] = CloseEntry{i < 16 ? row0 : row1, tok + (i < 16 ? 0 : 32), (uint32_t)(table(i) * P + i % P) | id << 16};
            n += more;
        }
    }

    // The list's projections anew, and the ids that have the other sign mended: eight lanes to an entry,
    // each with an eighth of the channels, all loads at once; the sum goes from lane to lane.  (A lane to
    // an entry, 32 channels a round of loads, took 14 thousand cycles for one entry: memory latencies, and
    // instructions that come cold.)
    __device__ __forceinline__ void settle() {
        constexpr int CH = D / 8;
        const int lane = threadIdx.x & 63, part = lane & 7;
        for (int base = 0; base < n; base += 8) {
            const int at = min(base + (lane >> 3), n - 1);
            const CloseEntry e = list[at];
            const int col = (int)(e.col & 0xffffu);
            const f32x4_t *k = (const f32x4_t *)((const float *)a.K + e.row * D + part * CH);
            const float *wc = W + (int64_t)(part * CH) * a.LP + col;
            f32x4_t x[CH / 4];
            float w[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) w[c] = wc[(int64_t)c * a.LP];
#pragma unroll
            for (int c = 0; c < CH / 4; ++c) x[c] = k[c];
            float sum = 0.0f;
#pragma unroll 1
            for (int s = 0; s < 8; ++s) {              // lane s is right from round s on
                const float before = dpp_f32<0x111>(sum);   // row_shr:1
                sum = part == 0 ? 0.0f : before;
#pragma unroll
                for (int c = 0; c < CH; ++c) sum = fmaf(x[c / 4][c % 4], w[c], sum);
            }
            const bool flip = part == 7 && base + (lane >> 3) < n && (sum >= 0.0f) != ((e.col >> (16 + col % P) & 1) != 0);
            const uint64_t flips = __ballot(flip);
            if (flips == 0) continue;
            for (uint64_t todo = flips; todo != 0; todo &= todo - 1) {   // all entries of the id learn of its new bit
                const int from = __ffsll((unsigned long long)todo) - 1;
                const int64_t row = list[base + (from >> 3)].row;
                const uint32_t was = (uint32_t)__builtin_amdgcn_readlane((int)e.col, from), bit = 1u << (16 + (was & 0xffffu) % P);
                const CloseEntry mine = list[min(lane, n - 1)];
                if (lane < n && mine.row == row && (mine.col & 0xffffu) / P == (was & 0xffffu) / P) list[lane].col = (mine.col & ~bit) | (~was & bit);
            }
            __builtin_amdgcn_wave_barrier();           // (the list as the other lanes left it)
            __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0): behind the ids themselves
            if (flip) ((uint8_t *)a.codes)[e.row * a.Lpad + code_pos(first_table + col / P, e.tok, S)] = (uint8_t)(list[at].col >> 16);
        }
        n = 0;
    }
};

// The keys of a wavefront's 64-key block as B operands: bf16 as stored, fp32 in pieces
template <typename T, int KS> struct KeyBlock;
template <int KS> struct KeyBlock<uint16_t, KS> {
    bf16x8_t hi[2][KS];
    __device__ __forceinline__ void load(int nb, const char *src, int g) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) hi[nb][ks] = *(const bf16x8_t *)(src + g * 16 + ks * 32);
    }
    __device__ __forceinline__ void cut() {}
};
template <int KS> struct KeyBlock<float, KS> {
    Row8<float> raw[2][KS];
    bf16x8_t hi[2][KS], lo[2][KS];
    float2 close[2];
    __device__ __forceinline__ void load(int nb, const char *src, int g) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) raw[nb][ks].load(src + g * 32 + ks * 64);
    }
    __device__ __forceinline__ void cut() {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            uint32_t any = 0;
            float h2 = 0.0f, l2 = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                float f[8];
                raw[nb][ks].get(f);
                uint32_t h[4], l[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    any |= __float_as_uint(f[2 * c]) | __float_as_uint(f[2 * c + 1]);
                    h[c] = cut_pair(floatx2_t{f[2 * c], f[2 * c + 1]}, l + c);
                }
                hi[nb][ks] = __builtin_bit_cast(bf16x8_t, make_uint4(h[0], h[1], h[2], h[3]));
                lo[nb][ks] = __builtin_bit_cast(bf16x8_t, make_uint4(l[0], l[1], l[2], l[3]));
                h2 = add_squares(hi[nb][ks], h2);
                l2 = add_squares(lo[nb][ks], l2);
            }
            const float B = 1.01f * __builtin_amdgcn_sqrtf(xor32_sum(l2)), A = 1.001f * __builtin_amdgcn_sqrtf(xor32_sum(h2)) + B;
            const uint64_t some = __ballot((any << 1) != 0);   // (zero but for signs)
            const bool zero = ((some | (some >> 32)) >> (threadIdx.x & 31) & 1) == 0;
            close[nb] = close_part<16 * KS>(zero ? 0.0f : fmaxf(A, 1e-30f), B);
        }
    }
};

struct OneSequence {                                   // (what stands for SeqUnits where there is nothing to share out)
    __device__ __forceinline__ explicit OneSequence(const HashArgs &) {}
    __device__ __forceinline__ int total() const { return 0; }
    __device__ __forceinline__ void find(int, int *, int *, int *, int *) const {}
};

// What a launch of the fast kernels knows of its runs of keys
enum HashRuns {
    kRunsLong = 0,      // a wavefront works on several 64-key blocks of its sequence, or on none
    kRunsShared = 1,    // the blocks of several sequences are dealt out as one row (SeqUnits)
    kRunsShort = 2,     // no wavefront has more than one block
};

// Shape of a workgroup: NG of the chunk's S position groups (a chunk's workgroups are its S / NG
// parts), their fragments in LDS.  d = 256: a block's fragments are 16 KB, so eight blocks, and a
// 64-key block of keys takes 128 registers, so eight wavefronts; the keys are read once per part
// (4 heads x 32768 keys, 64 tables of 8 planes: 35.1 us = 0.98 PFLOP/s, against 72.9 through
// hash_mfma_kernel, which stages the keys through LDS and packs ids generically).
template <int D, int S, int P> constexpr int hash8_groups() { return D <= 128 || S * P / 2 <= 8 ? S : S / 2; }
template <int D> constexpr int hash8_threads() { return D <= 128 ? kHash8Threads : 512; }
// which launches may deal the blocks of several sequences out as one (launch_blocks)
template <typename T, int D> constexpr bool hash_shares() { return sizeof(T) == 4 || D == 256; }

// fp32: the shape of bf16 rows of 256 channels, d = 64 too (eight wavefronts, registers for a block's raw
// keys beside the pieces).
template <typename T, int D> constexpr int hash_width() { return sizeof(T) == 4 ? 256 : D; }

template <typename T, int D, int S, int P, int RUNS>
__global__ __launch_bounds__((hash8_threads<hash_width<T, D>()>())) void hash_mfma8_kernel(HashArgs a) {
    static_assert(P == 8 || P == 4, "one-byte ids of 8 planes, or of 4 (a block's eight nibbles are spread over two words)");
    constexpr bool SHARE = RUNS == kRunsShared, SHORT = RUNS == kRunsShort;
    constexpr bool SPLIT = sizeof(T) == 4;     // bf16 pieces of fp32
    constexpr int KS = D / 16;                 // MFMA k-steps
    constexpr int KF = SPLIT ? 2 * KS : KS;    // fragments of a block
    constexpr int WD = hash_width<T, D>();
    constexpr int BPG = P / 2;                 // 32-column blocks per position group of 16 ids
    constexpr int NG = hash8_groups<WD, S, P>();
    constexpr int NCB = BPG * NG;              // 32-column blocks of the workgroup
    constexpr int NT = hash8_threads<WD>(), NW = NT / 64;
    extern __shared__ __align__(16) uint32_t hash8_lds_words[];
    uint32_t *smem = hash8_lds_words;
    uint4 *wl = (uint4 *)smem;                         // [NCB][KF][64 lanes] A fragments
    uint32_t *bits = smem + NCB * KF * 64 * 4;         // [NW waves][64 keys][4 words]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = SHARE ? blockIdx.x : blockIdx.y, slot = SHARE ? blockIdx.y : blockIdx.x, slots = SHARE ? gridDim.y : gridDim.x;
    const int part = row % (S / NG), hc = row / (S / NG);
    const int chunk = hc % a.n_chunks, h = hc / a.n_chunks;
    // the 64-key blocks it takes part in: those of sequence blockIdx.z, or (SHARE) of that group
    int b = blockIdx.z, count = 0, begin = 0, shared_r0 = 0;
    const typename std::conditional<SHARE && !SPLIT, SeqUnits<6>, OneSequence>::type runs(a);
    if (!SHARE) {
        count = a.row_count[b];
        begin = a.row_begin[b];
    }
    const int sub0 = part * NG;                        // the workgroup's first position group
    const int first_table = chunk * 64;
    const int ntab = min(64, a.L - first_table);

    uint32_t *mybits = bits + wave * 256;
    const int n = lane & 31, g = lane >> 5;
    constexpr int CAP = SPLIT ? 64 : 1;                // entries of a CloseList
    __shared__ CloseColumns cols[SPLIT ? NCB : 1];     // of each block
    __shared__ CloseEntry close_lds[SPLIT ? NW : 1][CAP];
    CloseList<D, P, S, CAP> close(a, close_lds[SPLIT ? wave : 0], h, first_table, ntab);
    const char *Kb = (const char *)a.K;
    char *Cb = (char *)a.codes;

    auto key_row = [&](int r) -> int64_t {
        const int t = begin + r;
        return (r < count && t >= 0 && t < a.map.max_n) ? a.map.row(b, h, t) : -1;
    };
    // Branch-free: a key that does not exist reads row 0 of the cache instead (its ids are never
    // stored).
    KeyBlock<T, KS> keys;
    auto load_keys = [&](int blk) {
        if (SHARE && !SPLIT) runs.find(blk, &b, &count, &begin, &shared_r0);
        const int r0 = SHARE && !SPLIT ? shared_r0 : blk * 64;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int64_t row = key_row(r0 + nb * 32 + n);
            keys.load(nb, Kb + (row >= 0 ? row : 0) * (int64_t)(D * sizeof(T)), g);
        }
    };
    // 32 sign bits of one key from the accumulators of a 32-row block: bit p = 1 when the
    // projection onto plane p is >= 0.  A lane's 16 accumulators are bits 16g .. 16g+15.
    auto signs = [&](const floatx16_t &acc) -> uint32_t {
        uint32_t neg = __float_as_uint(acc[15]) >> 31;
#pragma unroll
        for (int i = 14; i >= 0; --i) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[i]), 31);
        return neg;
    };
    auto sign_word = [&](uint32_t neg) -> uint32_t {
        auto both = __builtin_amdgcn_permlane32_swap(neg, neg, false, false);   // g = 0 and g = 1 halves, in every lane
        return ~(both[0] | (both[1] << 16));
    };

    // 64-key blocks are dealt round-robin, to the workgroups before their wavefronts: short runs and
    // last rounds then spread over the compute units (8 heads, 64 tables of 8 planes, both ways with
    // the launch that cut W: 8192 keys 18.6 us, 29.0 with whole workgroups filled first; 40000 keys
    // 44 / 55; full rounds alike.  Without that launch 16.9 and 42.6)
    // Short runs: while that leaves wavefronts without a block, two or four of them share one, NG / parts
    // of its position groups each, and the keys are fetched while W is cut (8 heads, (8, 64): 777 keys
    // 15.9 us with the launch that cut W, 7.1 now; 4096 16.7 / 10.3; (10, 60) 777 keys 12.9 / 6.8.  Long
    // runs keep the loop of whole blocks: with bounds of its own for every wavefront 131072 keys took
    // 132 us, 127 without).
    int nblocks = 0, stride = slots * NW, blk = slot + wave * slots, parts = 1, p0 = 0;
    cut_fragments<T, D, S, P, NG, NT>(wl, a, h, first_table, ntab, sub0, tid, [&]() __attribute__((always_inline)) {
        if (!SHORT) return;
        nblocks = (count + 63) >> 6;
        if (SPLIT) nblocks = min(nblocks, slots * NW);   // (a row_count beyond max_rows: a wavefront's keys are fetched once)
        parts = NG;
        while (parts > 1 && nblocks > slots * (NW / parts)) parts >>= 1;
        stride = slots * (NW / parts);
        const int w = __builtin_amdgcn_readfirstlane(wave);
        p0 = (w % parts) * (NCB / parts);
        blk = slot + (w / parts) * slots;
        if (blk < nblocks) load_keys(blk);
    });
    __syncthreads();                           // (waits for LDS only: a short run's keys stay under way)
    if constexpr (SPLIT) {
        for (int p = wave; p < NCB; p += NW) {
            const int sl = p / BPG, q = p % BPG;
            const CloseColumns c = close_columns<D>(wl + (p * KF) * 64 + (lane ^ frag_turn(sl, q)), close.column(q, sub0 + sl), a.LP);
            if (lane == 0) cols[p] = c;
        }
        __syncthreads();
    }
    // SPLIT && SHARE: from sequence to sequence with the blocks counted on, in scalar registers (the keys
    // and their pieces leave none for SeqUnits); blk is the block of sequence b
    const int b_end = min(a.batch, (b + 1) * a.group);
    auto walk = [&]() {
        while (blk >= nblocks && b + 1 < b_end) {
            blk -= nblocks;
            ++b;
            count = min(a.row_count[b], a.max_rows);
            begin = a.row_begin[b];
            nblocks = (max(count, 0) + 63) >> 6;
        }
    };
    if constexpr (SPLIT && SHARE) {
        blk = slot + __builtin_amdgcn_readfirstlane(wave) * slots;
        b = b * a.group - 1;
        walk();
    } else if (SPLIT && !SHORT) {
        nblocks = (count + 63) >> 6;
    } else if (!SHORT) {
        nblocks = SHARE ? runs.total() : (count + 63) >> 6;   // (not before the slab: nothing there waits for the lengths)
        if (blk < nblocks) load_keys(blk);
    }
    const int pb = SHORT ? p0 : 0, pe = SHORT ? p0 + NCB / parts : NCB;
    while (blk < nblocks) {
        const int r0 = SHARE && !SPLIT ? shared_r0 : blk * 64;
        if (SPLIT && !SHORT) load_keys(blk);
        keys.cut();
        const int64_t prow = key_row(r0 + lane);        // the key this lane packs
        const int rot = (begin + r0 + lane) & 15;
        uint4 done[NG > 1 ? NG - 1 : 1];                // the key's position groups before the last, kept until the row is whole
#pragma unroll 1
        for (int p = pb; p < pe; ++p) {
            const int sl = p / BPG, sub = sub0 + sl, q = p % BPG;
            const uint4 *af = wl + (p * KF) * 64 + (lane ^ frag_turn(sl, q));
            floatx16_t acc0, acc1;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc0[i] = acc1[i] = 0.0f;
            auto frag = [&](int i) { return __builtin_bit_cast(bf16x8_t, af[i * 64]); };
            if constexpr (SPLIT) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {               // (the small products first)
                    const bf16x8_t fh = frag(ks), fl = frag(KS + ks);
                    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fl, keys.hi[0][ks], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fl, keys.hi[1][ks], acc1, 0, 0, 0);
                    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fh, keys.lo[0][ks], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fh, keys.lo[1][ks], acc1, 0, 0, 0);
                }
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8_t fa = frag(ks);
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, keys.hi[0][ks], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, keys.hi[1][ks], acc1, 0, 0, 0);
            }
            uint32_t neg0 = signs(acc0), neg1 = signs(acc1);
            if constexpr (SPLIT) {
                uint32_t neg = neg0 | neg1 << 16;
                close.add(acc0, acc1, neg, keys.close, cols[p], q, sub, begin + r0 + n, [&](int nb) { return key_row(r0 + 32 * nb + n); });
                neg0 = neg & 0xffffu;
                neg1 = neg >> 16;
            }
            const uint32_t w0 = sign_word(neg0), w1 = sign_word(neg1);
            const uint32_t w = lane < 32 ? w0 : w1;                     // lane = key n or 32 + n
            if (P == 8) {
                // bytes whose table (sub + S (4q + e)) lies beyond the chunk's live tables stay zero
                const int nlive = (ntab - sub - 4 * S * q + S - 1) >> (S == 4 ? 2 : S == 2 ? 1 : 0);   // live tables among e = 0..3 (<= 0: none)
                const uint32_t live_mask = nlive >= 4 ? 0xffffffffu : nlive <= 0 ? 0u : (1u << (8 * nlive)) - 1u;
                mybits[lane * 4 + q] = w & live_mask;
            } else {
                // eight 4-bit ids: each nibble becomes the byte of its table (sub + S (8q + e))
                auto spread = [](uint32_t x) {          // nibbles 0..3 of x -> bytes 0..3
                    const uint32_t t = (x | (x << 8)) & 0x00ff00ffu;
                    return (t | (t << 4)) & 0x0f0f0f0fu;
                };
                const int nlive = (ntab - sub - 8 * S * q + S - 1) >> (S == 4 ? 2 : S == 2 ? 1 : 0);   // live tables among e = 0..7
                const int n0 = nlive < 4 ? nlive : 4, n1 = nlive - 4 < 4 ? nlive - 4 : 4;
                const uint32_t m0 = n0 >= 4 ? 0xffffffffu : n0 <= 0 ? 0u : (1u << (8 * n0)) - 1u;
                const uint32_t m1 = n1 >= 4 ? 0xffffffffu : n1 <= 0 ? 0u : (1u << (8 * n1)) - 1u;
                mybits[lane * 4 + 2 * q] = spread(w & 0xffffu) & m0;
                mybits[lane * 4 + 2 * q + 1] = spread(w >> 16) & m1;
            }
            if (q == BPG - 1) {
                // ---- the 16 ids of position group `sub`, rotated by the token position
                const uint4 wv = *(const uint4 *)(mybits + lane * 4);
                const bool r1 = rot & 4, r2 = rot & 8;
                const uint32_t y0 = r1 ? wv.y : wv.x, y1 = r1 ? wv.z : wv.y, y2 = r1 ? wv.w : wv.z, y3 = r1 ? wv.x : wv.w;
                const uint32_t x0 = r2 ? y2 : y0, x1 = r2 ? y3 : y1, x2 = r2 ? y0 : y2, x3 = r2 ? y1 : y3;
                const uint32_t sh = rot & 3;
                uint4 o;
                o.x = __builtin_amdgcn_alignbyte(x1, x0, sh);
                o.y = __builtin_amdgcn_alignbyte(x2, x1, sh);
                o.z = __builtin_amdgcn_alignbyte(x3, x2, sh);
                o.w = __builtin_amdgcn_alignbyte(x0, x3, sh);
                // the groups of a key go out together: 64 adjacent bytes (four groups), written back
                // as one whole line instead of four partial ones a quarter of the block apart
                if (NG > 1 && SHORT && parts > 1) {
                    if (prow >= 0) ((uint4 *)(Cb + prow * (int64_t)a.Lpad + first_table))[sub] = o;
                } else if (NG > 1 && sl == 0) done[0] = o;
                else if (NG > 2 && sl == 1) done[NG > 2 ? 1 : 0] = o;
                else if (NG > 2 && sl == 2) done[NG > 2 ? 2 : 0] = o;
                else if (prow >= 0) {
                    uint4 *dst = (uint4 *)(Cb + prow * (int64_t)a.Lpad + first_table) + sub0;
#pragma unroll
                    for (int i = 0; i + 1 < NG; ++i) dst[i] = done[i];
                    dst[NG - 1] = o;
                }
            }
        }
        if (SPLIT && close.n > CAP / 2) close.settle();
        blk += stride;
        if (SPLIT && SHARE) walk();
        else if (!SPLIT && blk < nblocks) load_keys(blk);
    }
    if (SPLIT) close.settle();
}

// ---------------------------------------------------------------------------------------
// The same structure for 10-plane tables with packed ids (groups of 16 S tables, S = 1 or 2): a
// workgroup keeps the W slab of one group (S x 160 columns = 5 S 32-column blocks; one string's
// 5 at d = 256) in LDS as MFMA fragments; every wavefront works on 64-key blocks of its own.
//
// Column order.  String `sub` (< S) of a token's group holds, before its rotation by the token
// position, the ids of tables sub, sub + S, .., sub + 15 S in bits [10 j, 10 j + 10): 160 bits =
// five sign words.  Block p = 5 sub + q produces word q: bit u = 32 q + (bit of the word) of the
// string is plane u % 10 of table sub + S (u / 10).  The stored string is that one rotated right
// by 10 (t mod 16) bits: a rotation of the five words and one funnel shift.
// ---------------------------------------------------------------------------------------
// (d = 256: one string per workgroup, 80 KB of fragments)
template <int D, int S> constexpr int hash10_strings() { return D <= 128 ? S : 1; }

template <int D, int S, int RUNS>
__global__ __launch_bounds__(hash8_threads<D>()) void hash_mfma10_kernel(HashArgs a) {
    constexpr bool SHARE = RUNS == kRunsShared, SHORT = RUNS == kRunsShort;
    constexpr int KS = D / 16;                 // MFMA k-steps
    constexpr int NS = hash10_strings<D, S>(); // strings of the workgroup
    constexpr int NCB = 5 * NS;                // its 32-column blocks
    constexpr int GT = 16 * S;                 // tables of a group
    constexpr int NT = hash8_threads<D>(), NW = NT / 64;
    extern __shared__ uint32_t smem[];
    uint4 *wl = (uint4 *)smem;                         // [NCB][KS][64 lanes] A fragments
    uint32_t *bits = smem + NCB * KS * 64 * 4;         // [NW waves][64 keys][5 words]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = SHARE ? blockIdx.x : blockIdx.y, slot = SHARE ? blockIdx.y : blockIdx.x, slots = SHARE ? gridDim.y : gridDim.x;
    const int sub0 = row % (S / NS), hc = row / (S / NS);   // (S / NS > 1: the workgroup's string)
    const int grp = hc % a.n_chunks, h = hc / a.n_chunks;
    // the 64-key blocks it takes part in: those of sequence blockIdx.z, or (SHARE) of that group
    int b = blockIdx.z, count = 0, begin = 0, shared_r0 = 0;
    const typename std::conditional<SHARE, SeqUnits<6>, OneSequence>::type runs(a);
    if (!SHARE) {
        count = a.row_count[b];
        begin = a.row_begin[b];
    }
    const int ntab = max(0, min(GT, a.L - grp * GT));

    uint32_t *mybits = bits + wave * 320;
    const int n = lane & 31, g = lane >> 5;
    const char *Kb = (const char *)a.K;
    char *Cb = (char *)a.codes;

    auto key_row = [&](int r) -> int64_t {
        const int t = begin + r;
        return (r < count && t >= 0 && t < a.map.max_n) ? a.map.row(b, h, t) : -1;
    };
    // (a key that does not exist reads row 0 of the cache instead; its ids are never stored)
    bf16x8_t kf[2][KS];
    auto load_keys = [&](int blk) {
        if (SHARE) runs.find(blk, &b, &count, &begin, &shared_r0);
        const int r0 = SHARE ? shared_r0 : blk * 64;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int64_t row = key_row(r0 + nb * 32 + n);
            const char *src = Kb + (row >= 0 ? row : 0) * (int64_t)(D * 2) + g * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[nb][ks] = *(const bf16x8_t *)(src + ks * 32);
        }
    };
    auto sign_word = [&](const floatx16_t &acc) -> uint32_t {
        uint32_t neg = __float_as_uint(acc[15]) >> 31;
#pragma unroll
        for (int i = 14; i >= 0; --i) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[i]), 31);
        auto both = __builtin_amdgcn_permlane32_swap(neg, neg, false, false);
        return ~(both[0] | (both[1] << 16));
    };

    // (as in hash_mfma8_kernel: workgroups first; of short runs the keys while W is cut, a block's strings
    // by two wavefronts where there are enough)
    int nblocks = 0, stride = slots * NW, blk = slot + wave * slots, parts = 1, p0 = 0;
    cut_fragments<uint16_t, D, S, 10, NS, NT>(wl, a, h, grp * GT, ntab, sub0, tid, [&]() __attribute__((always_inline)) {
        if (!SHORT) return;
        nblocks = (count + 63) >> 6;
        parts = NS == 2 && nblocks <= slots * (NW / 2) ? 2 : 1;
        stride = slots * (NW / parts);
        const int w = __builtin_amdgcn_readfirstlane(wave);
        p0 = (w % parts) * (NCB / parts);
        blk = slot + (w / parts) * slots;
        if (blk < nblocks) load_keys(blk);
    });
    __syncthreads();                           // (waits for LDS only: a short run's keys stay under way)
    if (!SHORT) {
        nblocks = SHARE ? runs.total() : (count + 63) >> 6;   // (not before the slab: nothing there waits for the lengths)
        if (blk < nblocks) load_keys(blk);
    }
    const int pb = SHORT ? p0 : 0, pe = SHORT ? p0 + NCB / parts : NCB;
    for (; blk < nblocks; blk += stride) {
        const int r0 = SHARE ? shared_r0 : blk * 64;
        const int64_t prow = key_row(r0 + lane);        // the key this lane packs
        const uint32_t turn = 10u * (uint32_t)((begin + r0 + lane) & 15);   // bits the string is rotated by
        uint4 head0 = make_uint4(0, 0, 0, 0);           // string 0, kept until string 1 is there too
        uint32_t tail0 = 0;
#pragma unroll 1
        for (int p = pb; p < pe; ++p) {
            const int sl = p >= 5 ? 1 : 0, sub = sub0 + sl, q = p - 5 * sl;
            const uint4 *af = wl + (p * KS) * 64 + (lane ^ frag_turn(sl, q));
            floatx16_t acc0, acc1;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc0[i] = acc1[i] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                union { uint4 u; bf16x8_t v; } fa;
                fa.u = af[ks * 64];
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.v, kf[0][ks], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.v, kf[1][ks], acc1, 0, 0, 0);
            }
            // ids of tables beyond the live ones stay zero: the string's first 10 nj bits are live
            const int nj = max(0, (ntab - sub + S - 1) / S);
            const int nlive = 10 * nj - 32 * q;
            const uint32_t live_mask = nlive >= 32 ? 0xffffffffu : nlive <= 0 ? 0u : (1u << nlive) - 1u;
            const uint32_t w0 = sign_word(acc0), w1 = sign_word(acc1);
            mybits[lane * 5 + q] = (lane < 32 ? w0 : w1) & live_mask;   // lane = key n or 32 + n
            if (q == 4) {
                uint32_t x0 = mybits[lane * 5], x1 = mybits[lane * 5 + 1], x2 = mybits[lane * 5 + 2];
                uint32_t x3 = mybits[lane * 5 + 3], x4 = mybits[lane * 5 + 4];
                // stored word k = bits [32 k + turn, +32) of the string, cyclically: words turned
                // by turn / 32, then a funnel shift by turn % 32
                const uint32_t wo = turn >> 5, sh = turn & 31;
                if (wo & 1) { const uint32_t t0 = x0; x0 = x1; x1 = x2; x2 = x3; x3 = x4; x4 = t0; }
                if (wo & 2) { const uint32_t t0 = x0, t1 = x1; x0 = x2; x1 = x3; x2 = x4; x3 = t0; x4 = t1; }
                if (wo & 4) { const uint32_t t4 = x4; x4 = x3; x3 = x2; x2 = x1; x1 = x0; x0 = t4; }
                uint4 o;
                o.x = __builtin_amdgcn_alignbit(x1, x0, sh);
                o.y = __builtin_amdgcn_alignbit(x2, x1, sh);
                o.z = __builtin_amdgcn_alignbit(x3, x2, sh);
                o.w = __builtin_amdgcn_alignbit(x4, x3, sh);
                const uint32_t ot = __builtin_amdgcn_alignbit(x0, x4, sh);
                if (NS == 2 && (!SHORT || parts == 1) && sl == 0) {
                    head0 = o;
                    tail0 = ot;
                } else if (prow >= 0) {
                    // the strings of the key's group together: 16 S adjacent bytes of the tile's
                    // main rows and 4 S of its tail rows
                    uint4 *dst = (uint4 *)(Cb + packed_main_row(prow, grp, a.Lpad, GT));
                    if (NS == 2 && (!SHORT || parts == 1)) {
                        dst[0] = head0;
                        dst[1] = o;
                        *(uint2 *)(Cb + packed_tail_row(prow, grp, a.Lpad, GT)) = make_uint2(tail0, ot);
                    } else {
                        dst[sub] = o;
                        ((uint32_t *)(Cb + packed_tail_row(prow, grp, a.Lpad, GT)))[sub] = ot;
                    }
                }
            }
        }
        if (blk + stride < nblocks) load_keys(blk + stride);
    }
}

template <typename T>
static int launch_rows(const HashArgs &a, int Hkv, int batch, int max_rows, hipStream_t st) {
    const int bw = 2 * ((a.LP + 63) / 64);
    if (max_rows <= 4) {
        constexpr int ROWS = 1;
        size_t lds = (size_t)ROWS * a.d * 4 + (size_t)ROWS * bw * 4 + (ROWS + 1) * 4 + ROWS * 8 + 16;
        dim3 grid(max_rows, Hkv, batch);
        hipLaunchKernelGGL((hash_rows_kernel<T, ROWS>), grid, dim3(256), lds, st, a);
    } else {
        constexpr int ROWS = 16;
        size_t lds = (size_t)ROWS * a.d * 4 + (size_t)ROWS * bw * 4 + (ROWS + 1) * 4 + ROWS * 8 + 16;
        dim3 grid((max_rows + ROWS - 1) / ROWS, Hkv, batch);
        hipLaunchKernelGGL((hash_rows_kernel<T, ROWS>), grid, dim3(256), lds, st, a);
    }
    return SOCKET_OK;
}

// the sequences in groups of equal size, for SeqUnits; returns their number
static int share_groups(HashArgs *a) {
    const int groups = (a->batch + 63) / 64;
    a->group = (a->batch + groups - 1) / groups;
    return (a->batch + a->group - 1) / a->group;
}

// Launch of a kernel that deals 64-key blocks to wavefronts: one workgroup per CU (the W slab fills
// most of its LDS) over `rows` heads, chunks and parts.  `shared` (null: there is none): the kernel
// that deals the blocks of several sequences out as one, for batches in which a wavefront of
// `alone` would have more than one block of the longest run, or one round of workgroups would not do.
// (A workgroup without a block cuts its slab for nothing; asking for the run's length first cost
// every short run 0.3 us, 4 % at 5000 keys of 16 tables, and gained nothing in ragged batches.)
typedef void (*fragment_kernel_t)(HashArgs);
static void launch_blocks(fragment_kernel_t alone, fragment_kernel_t brief, fragment_kernel_t shared, HashArgs a, int rows,
                          int batch, int max_rows, int threads, size_t lds, hipStream_t st) {
    const int nblocks = (max_rows + 63) / 64;
    int groups = batch, per = std::max(1, std::min(nblocks, 256 / (rows * batch)));
    const bool share = shared && batch > 1 && (nblocks > per * (threads / 64) || rows * batch > 256);
    if (share) {
        groups = share_groups(&a);
        per = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)nblocks * a.group, 256 / (rows * groups)));
    }
    if (!share && nblocks <= per * (threads / 64)) alone = brief;
    // (shared: slab by slab, so that few of the slabs go through each XCD's L2)
    hipLaunchKernelGGL(share ? shared : alone, share ? dim3(rows, per, groups) : dim3(per, rows, groups), dim3(threads), lds, st, a);
}

// dynamic LDS of hash_mfma8_kernel: the W slab as fragments, one id-word row per key of every wavefront's block
template <typename T, int D, int S, int P> constexpr size_t hash8_lds() {
    constexpr int WD = hash_width<T, D>();
    return (size_t)(P / 2 * hash8_groups<WD, S, P>()) * (D * sizeof(T) / 32) * 64 * 16 + (size_t)hash8_threads<WD>() * 16;
}

template <int D, int S> constexpr size_t hash10_lds() {
    return (size_t)(5 * hash10_strings<D, S>()) * (D / 16) * 64 * 16 + (size_t)hash8_threads<D>() * 20;
}

// once per context that uses a fast hash: more than 64 KB of dynamic LDS has to be allowed
// before the first launch
template <typename T, int D> static int hash_prepare_d() {
    hipError_t e = hipSuccess;
    auto allow = [&](auto kernel, size_t lds) {
        if (e == hipSuccess && lds > 64 * 1024)
            e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    };
    auto all = [&](auto runs) {
        constexpr int RUNS = decltype(runs)::value;
        allow(hash_mfma8_kernel<T, D, 4, 8, RUNS>, hash8_lds<T, D, 4, 8>());
        allow(hash_mfma8_kernel<T, D, 2, 8, RUNS>, hash8_lds<T, D, 2, 8>());
        allow(hash_mfma8_kernel<T, D, 1, 8, RUNS>, hash8_lds<T, D, 1, 8>());
        allow(hash_mfma8_kernel<T, D, 4, 4, RUNS>, hash8_lds<T, D, 4, 4>());
        allow(hash_mfma8_kernel<T, D, 2, 4, RUNS>, hash8_lds<T, D, 2, 4>());
        if constexpr (sizeof(T) == 2) {
            allow(hash_mfma10_kernel<D, 2, RUNS>, hash10_lds<D, 2>());
            allow(hash_mfma10_kernel<D, 1, RUNS>, hash10_lds<D, 1>());
        }
    };
    all(IntTag<kRunsLong>());
    all(IntTag<kRunsShort>());
    if constexpr (hash_shares<T, D>()) all(IntTag<kRunsShared>());
    return e == hipSuccess ? SOCKET_OK : SOCKET_EHIP;
}
int hash_prepare(int d, int kv_dtype) {
    if (kv_dtype == SOCKET_F32) return d == 64 ? hash_prepare_d<float, 64>() : hash_prepare_d<float, 128>();
    return d == 64 ? hash_prepare_d<uint16_t, 64>() : d == 128 ? hash_prepare_d<uint16_t, 128>() : hash_prepare_d<uint16_t, 256>();
}

template <typename T, int D, int S, int P>
static int launch_mfma8(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    constexpr int WD = hash_width<T, D>(), NT = hash8_threads<WD>(), PARTS = S / hash8_groups<WD, S, P>();
    a.tables_per_chunk = 16 * S;
    a.n_chunks = S == 4 ? (a.L + 63) / 64 : 1;
    const int rows = Hkv * a.n_chunks * PARTS;
    fragment_kernel_t shared = nullptr;
    if constexpr (hash_shares<T, D>()) shared = hash_mfma8_kernel<T, D, S, P, kRunsShared>;
    launch_blocks(hash_mfma8_kernel<T, D, S, P, kRunsLong>, hash_mfma8_kernel<T, D, S, P, kRunsShort>, shared, a, rows, batch, max_rows, NT, hash8_lds<T, D, S, P>(), st);
    return SOCKET_OK;
}
template <typename T, int D, int P>
static int launch_mfma8(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    return a.S == 4 ? launch_mfma8<T, D, 4, P>(a, Hkv, batch, max_rows, st)
         : a.S == 2 ? launch_mfma8<T, D, 2, P>(a, Hkv, batch, max_rows, st)
                    : launch_mfma8<T, D, 1, P>(a, Hkv, batch, max_rows, st);
}
template <typename T, int D>
static int launch_mfma8(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    return a.P == 8 ? launch_mfma8<T, D, 8>(a, Hkv, batch, max_rows, st)
                    : launch_mfma8<T, D, 4>(a, Hkv, batch, max_rows, st);
}

template <int D, int S>
static int launch_mfma10(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    constexpr int NT = hash8_threads<D>(), PARTS = S / hash10_strings<D, S>();
    a.tables_per_chunk = 16 * S;
    a.n_chunks = a.Lpad / (16 * S);            // groups, padding groups included (their ids are zero)
    fragment_kernel_t shared = nullptr;
    if constexpr (D == 256) shared = hash_mfma10_kernel<D, S, kRunsShared>;
    launch_blocks(hash_mfma10_kernel<D, S, kRunsLong>, hash_mfma10_kernel<D, S, kRunsShort>, shared, a, Hkv * a.n_chunks * PARTS, batch, max_rows, NT, hash10_lds<D, S>(), st);
    return SOCKET_OK;
}
template <int D>
static int launch_mfma10(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    return a.GT == 32 ? launch_mfma10<D, 2>(a, Hkv, batch, max_rows, st)
                      : launch_mfma10<D, 1>(a, Hkv, batch, max_rows, st);
}

// Runs of up to four rows stay with the FMA kernel's one-row workgroups while W is small: both are a
// prologue of W loads, and theirs are spread over more workgroups (rows = 4, 8 heads: 512 columns x
// 128 channels 11.6 us there, 13.2 here; 600 x 128 16.1 / 10.9; 512 x 256 19.5 / 13.2; five rows of
// 512 x 128, where that kernel takes sixteen rows a workgroup: 32.6 / 13.2).
static bool f32_fma_rows(const HashArgs &a, int max_rows) { return max_rows <= 4 && (a.LP + 255) / 256 * a.d <= 256; }
// columns of W a workgroup of hash_f32_kernel holds at most (32 a wavefront)
template <int D> constexpr int f32_columns() { return D <= 128 ? 512 : 256; }

// `split`: the context's ids are hash_mfma8_kernel's, which takes fp32 keys of up to 128 channels
template <typename T, int D>
static int launch_f32(HashArgs a, int Hkv, int batch, int max_rows, bool split, hipStream_t st) {
    if (a.GT) {
        a.tables_per_chunk = a.GT;             // packed ids: whole groups, padding groups included
        a.n_chunks = a.Lpad / a.GT;
    } else {
        a.tables_per_chunk = f32_columns<D>() / a.P;
        if (a.tables_per_chunk > a.L) a.tables_per_chunk = a.L;
        a.n_chunks = (a.L + a.tables_per_chunk - 1) / a.tables_per_chunk;
    }
    int waves = (a.tables_per_chunk * a.P + 31) / 32;
    if (waves < f32_min_threads<D>() / 64) waves = f32_min_threads<D>() / 64;
    // one round of resident workgroups (16 wavefronts a CU, 8 at d = 256), at most 16 tiles each
    const int slots = 256 * ((D <= 128 ? 16 : 8) / waves), rows = Hkv * a.n_chunks;
    const int seq_tiles = (max_rows + kF32Tile - 1) / kF32Tile;
    int64_t share = ((int64_t)seq_tiles * rows * batch + slots - 1) / slots;
    // More than one tile to a workgroup: the pieces on the bf16 matrix cores.  One tile is over before
    // their W is cut and their first instructions are there (8 heads, us here / there, many calls on two
    // caches in turn: 32 tables of 8 planes 1024 keys 9.9 / 15.1, 2048 16.9 / 15.8 (still one tile), 8192
    // 45 / 28, 32768 154 / 67; 64 tables 1024 16.7 / 17.2, 2048 25.6 / 20.4, 8192 74 / 40; d = 64, 64 tables
    // 1024 9.4 / 11.1, 2048 14.3 / 12.6, 32768 160 / 63; on one cache, d = 128, 16 tables 3072 keys 14.9 /
    // 13.6, 8192 27.7 / 17.0; 31 tables of 4 planes 3072 15.3 / 13.0; d = 64, 16 of 4 8192 11.8 / 8.7).
    if constexpr (sizeof(T) == 4 && D <= 128)
        if (split && share > 1) return launch_mfma8<float, D>(a, Hkv, batch, max_rows, st);
    if (share > 16) share = 16;
    a.rows_per_wg = (int)share * kF32Tile;
    int64_t per = (seq_tiles + share - 1) / share;
    int groups = batch;
    // Batches with more than three tiles to a workgroup, by the bound on the lengths: shares of
    // all sequences' tiles, in up to four rounds where 16 tiles a share or a last round that is an
    // eighth empty ask for it
    const bool shared = batch > 1 && share > 3;
    if (shared) {
        groups = share_groups(&a);
        const int64_t tiles = (int64_t)seq_tiles * a.group, all = (int64_t)rows * groups;
        per = slots / all;
        for (int r = 1; r < 4 && (per * all * 8 < (int64_t)r * slots * 7 || tiles > 16 * per); ++r) per = (r + 1) * slots / all;
        if (per < 1) per = 1;
        share = (tiles + per - 1) / per;
        per = (tiles + share - 1) / share;
    }
    const auto kernel = shared ? hash_f32_kernel<T, D, true> : hash_f32_kernel<T, D, false>;
    constexpr size_t lds = 2 * kF32Tile * (D + 4) * 4 + 2 * kF32Tile * kF32BitWords * 4 + 3 * kF32Tile * 12;
    static_assert(lds <= 80 * 1024, "two workgroups a CU");
    if (lds > 64 * 1024 && hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return SOCKET_EHIP;
    hipLaunchKernelGGL(kernel, dim3((unsigned)per, rows, groups), dim3(64 * waves), lds, st, a);
    return SOCKET_OK;
}

template <typename T>
static int launch_f32(const HashArgs &a, int Hkv, int batch, int max_rows, bool split, hipStream_t st) {
    // (a group of 32 tables of 9 or 10 planes is wider than a workgroup at d = 256)
    if (f32_fma_rows(a, max_rows) || a.GT * a.P > (a.d <= 128 ? f32_columns<128>() : f32_columns<256>()))
        return launch_rows<T>(a, Hkv, batch, max_rows, st);
    switch (a.d) {
        case 64: return launch_f32<T, 64>(a, Hkv, batch, max_rows, split, st);
        case 128: return launch_f32<T, 128>(a, Hkv, batch, max_rows, split, st);
        case 256: return launch_f32<T, 256>(a, Hkv, batch, max_rows, split, st);
        default: return SOCKET_EUNSUPPORTED;
    }
}

template <int D>
static int launch_mfma(HashArgs a, int Hkv, int batch, int max_rows, hipStream_t st) {
    constexpr int TILE = 64, KSTRIDE = D * 2 + 16, BSTRIDE = 17;
    if (a.GT) {
        // packed ids: a workgroup owns whole groups of GT tables (the high bits of four ids
        // share a byte), padding groups included
        a.tables_per_chunk = a.GT;
        a.n_chunks = a.Lpad / a.GT;
    } else {
        a.tables_per_chunk = 512 / a.P;
        if (a.tables_per_chunk > a.L) a.tables_per_chunk = a.L;
        a.n_chunks = (a.L + a.tables_per_chunk - 1) / a.tables_per_chunk;
    }
    // rows per workgroup: enough workgroups to fill 256 CUs, at least 1024 rows each so the
    // one-time load of the W slab is amortised
    int64_t total = (int64_t)max_rows * Hkv * batch * a.n_chunks;
    int rows = (int)((total + 511) / 512);
    rows = (rows + TILE - 1) / TILE * TILE;
    if (rows < 1024) rows = 1024;
    a.rows_per_wg = rows;
    size_t lds = 2 * TILE * KSTRIDE + 2 * TILE * BSTRIDE * 4 + 4 * TILE * 4 + 3 * TILE * 8;
    dim3 grid((max_rows + rows - 1) / rows, Hkv * a.n_chunks, batch);
    hipLaunchKernelGGL((hash_mfma_kernel<D>), grid, dim3(512), lds, st, a);
    return SOCKET_OK;
}

int launch_hash_keys(socket_ctx *ctx, const void *K, const void *proj, const int32_t *block_table,
                     const int32_t *row_begin, const int32_t *row_count, int batch, int max_rows,
                     void *codes, hipStream_t st) {
    const Geometry &g = ctx->g;
    HashArgs a;
    a.K = K; a.W = proj; a.codes = codes; a.row_begin = row_begin; a.row_count = row_count;
    a.map = row_map(g, block_table);
    a.d = g.d; a.L = g.L; a.P = g.P; a.LP = g.L * g.P; a.Lpad = g.Lpad; a.S = g.S; a.cb = g.cb;
    a.GT = g.mode == kSplit ? g.GT : 0;
    a.rows_per_wg = 0; a.tables_per_chunk = g.L; a.n_chunks = 1; a.batch = batch; a.max_rows = max_rows; a.group = 0;
    int rc;
    if (max_rows == 1) {
        // one appended key per sequence: the projection kernel with its W slab staged in LDS
        return launch_project(ctx, nullptr, proj, 1.0f, K, codes, block_table, row_begin, row_count,
                              nullptr, batch, st);
    } else if (g.kv_dtype == SOCKET_F32) {
        rc = launch_f32<float>(a, g.Hkv, batch, max_rows, ctx->fast_hash, st);
    } else if (max_rows < 64) {
        rc = launch_f32<uint16_t>(a, g.Hkv, batch, max_rows, false, st);
    } else {
        const bool fast8 = ctx->fast_hash && (g.P == 8 || g.P == 4);   // one-byte ids of 8 or 4 planes
        const bool fast10 = ctx->fast_hash && g.P == 10;    // packed ids in groups of 32 or 16 tables
        switch (g.d) {
            case 64: rc = fast8 ? launch_mfma8<uint16_t, 64>(a, g.Hkv, batch, max_rows, st)
                          : fast10 ? launch_mfma10<64>(a, g.Hkv, batch, max_rows, st)
                                   : launch_mfma<64>(a, g.Hkv, batch, max_rows, st); break;
            case 128: rc = fast8 ? launch_mfma8<uint16_t, 128>(a, g.Hkv, batch, max_rows, st)
                           : fast10 ? launch_mfma10<128>(a, g.Hkv, batch, max_rows, st)
                                    : launch_mfma<128>(a, g.Hkv, batch, max_rows, st); break;
            case 256: rc = fast8 ? launch_mfma8<uint16_t, 256>(a, g.Hkv, batch, max_rows, st)
                           : fast10 ? launch_mfma10<256>(a, g.Hkv, batch, max_rows, st)
                                    : launch_mfma<256>(a, g.Hkv, batch, max_rows, st); break;
            default: return SOCKET_EUNSUPPORTED;
        }
    }
    if (rc != SOCKET_OK) return rc;
    return record_hip(ctx, hipGetLastError());
}

}  // namespace sk
