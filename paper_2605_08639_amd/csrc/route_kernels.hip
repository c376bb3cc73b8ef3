// Routing-side kernels: load histogram, token permutation, unpermute + combine.
// All three are bound by HBM traffic (or, for the index parts, by launch latency); none is
// a contraction, so there is no MFMA here: the work is coalesced 16-byte accesses,
// wave-level ballots and LDS-private counters.
#include "common.h"

#include <mutex>

namespace relibra {

constexpr int kMaxExperts = 4096;
constexpr int kHistThreads = 1024;   // one block per micro-batch
constexpr int kHistLdsBytes = 64 * 1024;
constexpr int kUnit = RELIBRA_PERM_UNIT;   // assignments per permutation unit (one wave): short units, many waves -
                                         // the rank kernel is a chain of dependent table reads per round of 64
constexpr int kPermThreads = 256;    // 4 waves = 4 units per block

// ---------------------------------------------------------------- histogram (Eq. 1)
// One block per micro-batch: it counts the micro-batch's ids in LDS and STORES the finished
// histogram, so there is no zero-fill launch in front, no global atomics, and the result does
// not depend on any execution order.  Hot experts (a Zipf router sends a fifth of the assignments
// to one expert) would serialise LDS atomics on one address; every bin is therefore kept in C
// copies, lane l adding to copy l % C, laid out so that the copies of a bin sit in different banks.
// A single micro-batch (<= 512 KiB of ids) is latency-sized whatever the kernel does; the
// bandwidth-bound use is many micro-batches at once (every layer's replayed routing, Section 3),
// where the grid is thousands of blocks.
__global__ void __launch_bounds__(kHistThreads)
hist_kernel(const int32_t *__restrict__ ids, int per_mb, int E, int copies_log2, int vec_ok,
            int32_t *__restrict__ counts, int32_t *err_flag)
{
    extern __shared__ int32_t bins[];          // [E << copies_log2]
    const int mb = blockIdx.x;
    const int n_bins = E << copies_log2;
    for (int i = threadIdx.x; i < n_bins; i += kHistThreads) bins[i] = 0;
    __syncthreads();
    const int32_t *src = ids + (size_t)mb * per_mb;
    const int copy = threadIdx.x & ((1 << copies_log2) - 1);
    bool bad = false;
    if (vec_ok) {                      // 16-byte aligned rows of the id tensor
        const int4 *v = reinterpret_cast<const int4 *>(src);
        const int n4 = per_mb / 4;
        int i = threadIdx.x;
        for (; i + 3 * kHistThreads < n4; i += 4 * kHistThreads) {       // four loads in flight per lane
            const int4 q[4] = {v[i], v[i + kHistThreads], v[i + 2 * kHistThreads], v[i + 3 * kHistThreads]};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e4[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if ((unsigned)e4[j] < (unsigned)E) atomicAdd(&bins[(e4[j] << copies_log2) + copy], 1);
                    else bad = true;
                }
            }
        }
        for (; i < n4; i += kHistThreads) {
            const int4 q = v[i];
            const int e4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((unsigned)e4[j] < (unsigned)E) atomicAdd(&bins[(e4[j] << copies_log2) + copy], 1);
                else bad = true;
            }
        }
    } else {
        for (int i = threadIdx.x; i < per_mb; i += kHistThreads) {
            const int e = src[i];
            if ((unsigned)e < (unsigned)E) atomicAdd(&bins[(e << copies_log2) + copy], 1);
            else bad = true;
        }
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_ID_RANGE);
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kHistThreads) {
        int c = 0;
        for (int j = 0; j < (1 << copies_log2); ++j) c += bins[(e << copies_log2) + ((j + e) & ((1 << copies_log2) - 1))];
        counts[(size_t)mb * E + e] = c;
    }
}

// ---------------------------------------------------------------- permutation indices
// The stable partition is a counting sort over experts in three passes:
//   1. every wave counts its unit of assignments per expert        -> unit_cnt[unit][e]
//   2. an exclusive scan over units, per expert                    -> unit_cnt[unit][e] = base
//   3. every wave walks its unit in order, 64 assignments at a time; a ballot-built mask of
//      the lanes holding the same expert gives each lane its ordinal inside the step, an LDS
//      counter per expert carries the ordinal across steps.
// The ordinal is then mapped through the expert's instance list to a row (Section 5.2).

__global__ void __launch_bounds__(kPermThreads)
perm_count_kernel(const int32_t *__restrict__ ids, int N, int E, int32_t *__restrict__ unit_cnt,
                  int32_t *__restrict__ src_of, int32_t *err_flag)
{
    extern __shared__ int32_t lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int32_t *bins = lds + wave * E;
    const int unit = blockIdx.x * (kPermThreads / 64) + wave;
    for (int e = lane; e < E; e += 64) bins[e] = 0;
    __builtin_amdgcn_wave_barrier();
    const int lo = unit * kUnit, hi = min(N, lo + kUnit);
    bool bad = false;
    for (int a = lo + lane; a < hi; a += 64) {
        const int e = ids[a];
        if ((unsigned)e < (unsigned)E) atomicAdd(&bins[e], 1);
        else bad = true;
        src_of[a] = -1;                // rows nobody claims stay marked
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_ID_RANGE);
    __builtin_amdgcn_wave_barrier();
    if (lo < N)
        for (int e = lane; e < E; e += 64) unit_cnt[(size_t)unit * E + e] = bins[e];
}

// One block per expert: exclusive scan of that expert's counts over the units.
__global__ void __launch_bounds__(256) perm_scan_kernel(int32_t *unit_cnt, int n_units, int E)
{
    __shared__ int32_t sums[4];
    const int e = blockIdx.x, tid = threadIdx.x;
    int carry = 0;
    for (int base = 0; base < n_units; base += 256) {
        const int u = base + tid;
        const int c = u < n_units ? unit_cnt[(size_t)u * E + e] : 0;
        int all;
        const int upto = block_scan256(c, sums, all);
        if (u < n_units) unit_cnt[(size_t)u * E + e] = carry + upto - c;
        carry += all;
    }
}

// Optional per-source split of the permutation (all null / zero: split in token order).
struct SrcSplit {
    const int32_t *src_first;       // [EP][E] ordinal, among e's assignments, of source j's first one
    const int32_t *inst_src_rows;   // [instances][EP] tokens of source j served by instance i
    const int32_t *inst_src_base;   // [instances][EP] exclusive prefix of inst_src_rows over j
    int EP, k, tokens_per_src;
};

// What the ranking step needs of the plan's tables.
struct PlanTables {
    const int32_t *__restrict__ inst_ptr, *__restrict__ inst_rows, *__restrict__ inst_group, *__restrict__ group_offset;
};
// First instance of an expert, kept in LDS by the one-block permutation: its rows and its first row.
struct FirstInst {
    int32_t rows, row0;
};

// Ranks assignments lo .. hi-1 (one wave, 64 at a time, in order).  next[e]: next ordinal of expert e
// in this range (LDS, private to the wave).  first: null, or every expert's first instance.
__device__ __forceinline__ int rank_range(const int32_t *__restrict__ ids, int lo, int hi, int N, int E, int G, int ebits, int32_t *next,
                                          const FirstInst *first, const PlanTables &t, int32_t *__restrict__ row_of,
                                          int32_t *__restrict__ src_of, const SrcSplit &sp)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int flags = 0;
    int e_next = lo + lane < hi ? ids[lo + lane] : -1;
    for (int base = lo; base < hi; base += 64) {
        const int a = base + lane;
        const bool live = a < hi;
        const int e_raw = e_next;
        e_next = a + 64 < hi ? ids[a + 64] : -1;
        const bool ok = live && (unsigned)e_raw < (unsigned)E;
        const int e = ok ? e_raw : 0;
        // lanes with the same expert: intersect ballots bit by bit
        uint64_t same = __ballot(ok);
        for (int b = 0; b < ebits; ++b) {
            const uint64_t vote = __ballot((e >> b) & 1);
            same &= ((e >> b) & 1) ? vote : ~vote;
        }
        int q = 0;
        if (ok) {
            const int before = __popcll(same & lt_mask);
            const int leader = __ffsll((long long)same) - 1;
            int start = 0;
            if (lane == leader) {          // one lane per expert touches the counter
                start = next[e];
                next[e] = start + __popcll(same);
            }
            start = __shfl(start, leader);
            q = start + before;
        }
        __builtin_amdgcn_wave_barrier();
        if (ok) {
            int skipped = 0, row = -1;
            if (sp.src_first) {
                // source-aware split: ordinal among the source's own tokens of e, runs of
                // inst_src_rows[i][j], rows of an instance laid out source after source
                int i = t.inst_ptr[e];
                const int end = t.inst_ptr[e + 1];
                const int j = min((a / sp.k) / sp.tokens_per_src, sp.EP - 1);
                const int qj = q - sp.src_first[(size_t)j * E + e];
                for (; qj >= 0 && i < end; ++i) {
                    const int n = sp.inst_src_rows[(size_t)i * sp.EP + j];
                    if (qj < skipped + n) {
                        const int g = t.inst_group[i];
                        if ((unsigned)g < (unsigned)G) row = t.group_offset[g] + sp.inst_src_base[(size_t)i * sp.EP + j] + (qj - skipped);
                        break;
                    }
                    skipped += n;
                }
            } else if (first && q < first[e].rows) {
                row = first[e].row0 + q;
            } else {
                int i = t.inst_ptr[e];
                const int end = t.inst_ptr[e + 1];
                for (; i < end; ++i) {
                    const int n = t.inst_rows[i];
                    if (q < skipped + n) {
                        const int g = t.inst_group[i];
                        if ((unsigned)g < (unsigned)G) row = t.group_offset[g] + (q - skipped);
                        break;
                    }
                    skipped += n;
                }
            }
            if ((unsigned)row < (unsigned)N) {
                row_of[a] = row;
                src_of[row] = a;
            } else {
                row_of[a] = -1;
                flags |= RELIBRA_ERR_PLAN_COVER;
            }
        } else if (live) {
            row_of[a] = -1;
            flags |= RELIBRA_ERR_ID_RANGE;
        }
    }
    return flags;
}

__global__ void __launch_bounds__(kPermThreads)
perm_rank_kernel(const int32_t *__restrict__ ids, int N, int E, int G, int ebits,
                 const int32_t *__restrict__ unit_base, PlanTables t,
                 int32_t *__restrict__ row_of, int32_t *__restrict__ src_of, int32_t *err_flag,
                 SrcSplit sp)
{
    extern __shared__ int32_t lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int32_t *next = lds + wave * E;        // next ordinal of each expert, private to the wave
    const int unit = blockIdx.x * (kPermThreads / 64) + wave;
    const int lo = unit * kUnit, hi = min(N, lo + kUnit);
    if (lo < N)
        for (int e = lane; e < E; e += 64) next[e] = unit_base[(size_t)unit * E + e];
    __builtin_amdgcn_wave_barrier();
    const int flags = rank_range(ids, lo, hi, N, E, G, ebits, next, nullptr, t, row_of, src_of, sp);
    if (flags) atomicOr(err_flag, flags);
}

// The three passes in one block, for small micro-batches: the three launches cost more than the work
// (each is a launch and a few dependent memory round trips).  Every wave takes a sixteenth of the
// assignments; counts, their scan over the waves and the experts' first instances stay in LDS, so that a
// round of 64 assignments reads memory only where an expert is split over several instances.  A wave's rounds run one
// after the other, so the time goes in steps of 1024 assignments, and with the number of experts (the scan).  One
// block / three kernels, us, in a captured graph and called one by one (where launches are what three kernels cost):
//     assignments            1024       2048       3072       4096              1024        2048       3072       4096
//     8 experts, top-2    4.6  8.6   6.4  8.6   8.4  8.7  10.0  8.7           7.4 12.3   7.5 12.9   8.1 12.8   9.7 13.0
//     128 experts, top-8  4.0  8.4   7.0  9.6   6.2  8.9   7.2  9.1           7.4 12.7   7.3 12.7   7.4 12.7   7.3 12.8
//     512 experts, top-8  6.3 13.4   8.8 12.9  12.2 13.5  16.2 13.9           7.4 13.3   8.5 12.8  12.0 13.5  16.0 13.9
// (128 experts at 3584, with more experts split: 10.0 9.6 and 9.8 12.8.)  So up to 3072 assignments, and up to 4096 for
// 256 experts, where only a captured call loses, by about 1 us.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int kSmallE = 512;                               // (kSmallWaves + 2) * kSmallE ints of LDS
inline bool perm_in_one_block(int N, int E) { return E <= kSmallE && N <= (E <= 256 ? 4096 : 3072); }
__global__ void __launch_bounds__(kSmallThreads)
perm_small_kernel(const int32_t *__restrict__ ids, int N, int E, int G, int ebits, PlanTables t,
                  int32_t *__restrict__ row_of, int32_t *__restrict__ src_of, int32_t *err_flag, SrcSplit sp)
{
    extern __shared__ int32_t lds[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    int32_t *bins = lds + wave * E;
    FirstInst *first = reinterpret_cast<FirstInst *>(lds + kSmallWaves * E);
    for (int i = tid; i < kSmallWaves * E; i += kSmallThreads) lds[i] = 0;
    for (int i = tid; i < N; i += kSmallThreads) src_of[i] = -1;       // rows nobody claims stay marked
    int inst0 = 0, inst1 = 0;
    if (tid < E) { inst0 = t.inst_ptr[tid]; inst1 = t.inst_ptr[tid + 1]; }
    const int per_wave = ((N + kSmallThreads - 1) / kSmallThreads) * 64;
    const int lo = min(wave * per_wave, N), hi = min(lo + per_wave, N);
    __syncthreads();
    for (int a = lo + lane; a < hi; a += 64) {
        const int e = ids[a];
        if ((unsigned)e < (unsigned)E) atomicAdd(&bins[e], 1);         // ids out of range are flagged by the ranking
    }
    __syncthreads();
    if (tid < E) {                         // exclusive scan over the waves
        int at = 0;
        for (int w = 0; w < kSmallWaves; ++w) {
            const int c = lds[w * E + tid];
            lds[w * E + tid] = at;
            at += c;
        }
        FirstInst f{0, 0};
        if (at > 0 && inst0 < inst1 && !sp.src_first) {
            const int g = t.inst_group[inst0];
            if ((unsigned)g < (unsigned)G) f = FirstInst{t.inst_rows[inst0], t.group_offset[g]};
        }
        first[tid] = f;
    }
    __syncthreads();
    const int flags = rank_range(ids, lo, hi, N, E, G, ebits, bins, sp.src_first ? nullptr : first, t, row_of, src_of, sp);
    if (flags) atomicOr(err_flag, flags);
}

// Thread mapping of the row-streaming kernels: a row of vec_per_row 16-byte pieces is walked by
// LPR = 2^lpr_log2 consecutive threads, each taking every LPR-th piece (LPR = the smallest power
// of two that leaves a thread at most `pieces` pieces, at most the block), so a block of 256
// threads serves 256 / LPR rows at a time and no index needs a division.
constexpr int kRowThreads = 256;
inline int lanes_per_row_log2(int vec_per_row, int pieces)
{
    int l = 0;
    while ((1 << l) * pieces < vec_per_row && (1 << l) < kRowThreads) ++l;
    return l;
}

// Row gather: Xrows[row] = X[src_of[row] / k], 16 bytes per piece.  Rows nobody claims stay untouched.
// Two forms.  Token by token: a token's pieces are read once into registers and stored to the rows of its k
// assignments (a row is written by the assignment that src_of names for it); the write stream alone bounds it, where
// walked row by row the gather fetched every token k times through the caches and ran at the copy rate.  Row by row:
// k times the threads and one lookup less in the chain, for copies that do not fill the chip.  Row by row / token by
// token, us: 777 tokens x 256, k = 4 2.0 3.2; 32 x 7168, k = 8 2.0 3.0; 16384 x 128, k = 1 2.6 3.0; 4096 x 512, k = 2
// 3.4 3.6; 128 x 7168, k = 8 4.9 5.4; 8192 x 128, k = 8 (16 MiB of rows) 4.3 5.3; 256 x 7168, k = 8 (28 MiB) 9.4 7.4;
// 2048 x 4096, k = 2 12.0 9.1; 16384 x 4096, k = 2 83 79; 8192 x 4096, k = 8 (512 MiB) 159 103.
constexpr size_t kGatherByRow = (size_t)16 << 20;          // bytes of rows up to which they are walked one by one
__global__ void __launch_bounds__(kRowThreads)
gather_by_row_kernel(const uint4 *__restrict__ X, const int32_t *__restrict__ src_of, int N, int T, int k, int vec_per_row, int lpr_log2,
                     uint4 *__restrict__ Xrows)
{
    const int lpr = 1 << lpr_log2, rows_per_block = kRowThreads >> lpr_log2;
    const int r_local = threadIdx.x >> lpr_log2, c0 = threadIdx.x & (lpr - 1);
    for (int row = blockIdx.x * rows_per_block + r_local; row < N; row += gridDim.x * rows_per_block) {
        const int a = src_of[row];
        if (a < 0) continue;
        const int t = a / k;
        if (t >= T) continue;
        const uint4 *__restrict__ src = X + (size_t)t * vec_per_row;
        uint4 *__restrict__ dst = Xrows + (size_t)row * vec_per_row;
        int c = c0;
        for (; c + 3 * lpr < vec_per_row; c += 4 * lpr) {
            const uint4 v0 = src[c], v1 = src[c + lpr], v2 = src[c + 2 * lpr], v3 = src[c + 3 * lpr];
            dst[c] = v0; dst[c + lpr] = v1; dst[c + 2 * lpr] = v2; dst[c + 3 * lpr] = v3;
        }
        for (; c < vec_per_row; c += lpr) dst[c] = src[c];
    }
}

constexpr int kGatherRows = 8;                             // row lookups in flight
__global__ void __launch_bounds__(kRowThreads)
gather_by_token_kernel(const uint4 *__restrict__ X, const int32_t *__restrict__ row_of, const int32_t *__restrict__ src_of, int N, int T,
                       int k, int vec_per_row, int lpr_log2, uint4 *__restrict__ Xrows)
{
    const int lpr = 1 << lpr_log2, tokens_per_block = kRowThreads >> lpr_log2;
    const int t_local = threadIdx.x >> lpr_log2, c0 = threadIdx.x & (lpr - 1);
    for (int t = blockIdx.x * tokens_per_block + t_local; t < T; t += gridDim.x * tokens_per_block) {
        const uint4 *__restrict__ src = X + (size_t)t * vec_per_row;
        for (int c = c0; c < vec_per_row; c += 4 * lpr) {
            const int last = vec_per_row - 1;              // pieces past the end: the last one again, not stored
            const int c1 = c + lpr, c2 = c + 2 * lpr, c3 = c + 3 * lpr;
            const uint4 v0 = src[c], v1 = src[min(c1, last)], v2 = src[min(c2, last)], v3 = src[min(c3, last)];
            for (int s0 = 0; s0 < k; s0 += kGatherRows) {
                int row[kGatherRows], owner[kGatherRows];
#pragma unroll
                for (int u = 0; u < kGatherRows; ++u) row[u] = s0 + u < k ? row_of[t * k + s0 + u] : -1;
#pragma unroll
                for (int u = 0; u < kGatherRows; ++u) owner[u] = (unsigned)row[u] < (unsigned)N ? src_of[row[u]] : -1;
#pragma unroll
                for (int u = 0; u < kGatherRows; ++u) {
                    if (owner[u] != t * k + s0 + u) continue;
                    uint4 *__restrict__ dst = Xrows + (size_t)row[u] * vec_per_row;
                    dst[c] = v0;
                    if (c1 <= last) dst[c1] = v1;
                    if (c2 <= last) dst[c2] = v2;
                    if (c3 <= last) dst[c3] = v3;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- combine
__device__ __forceinline__ void unpack8(const uint4 &v, float *f)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = __uint_as_float(w[j] << 16);
        f[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float *f)
{
    uint4 v;
    v.x = pack2bf(f[0], f[1]);
    v.y = pack2bf(f[2], f[3]);
    v.z = pack2bf(f[4], f[5]);
    v.w = pack2bf(f[6], f[7]);
    return v;
}

// out[t] = sum_s gate[t,s] * rows[row_of[t,s]]; fp32 accumulation in slot order.
template <bool GATED>
__global__ void __launch_bounds__(256)
combine_fwd_kernel(const uint4 *__restrict__ rows, const float *__restrict__ gates,
                   const int32_t *__restrict__ row_of, int T, int k, int N, int vec_per_row,
                   uint4 *__restrict__ out, int32_t *err_flag)
{
    const size_t total = (size_t)T * vec_per_row;
    bool bad = false;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const int t = (int)(i / vec_per_row), c = (int)(i % vec_per_row);
        float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int s0 = 0; s0 < k; s0 += 8) {                 // eight row fetches in flight
            uint4 v[8];
            float g[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                g[u] = 0.0f;
                v[u] = make_uint4(0, 0, 0, 0);
                if (s0 + u < k) {
                    const int row = row_of[(size_t)t * k + s0 + u];
                    if ((unsigned)row < (unsigned)N) {
                        g[u] = GATED ? gates[(size_t)t * k + s0 + u] : 1.0f;
                        v[u] = rows[(size_t)row * vec_per_row + c];
                    } else {
                        bad = true;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {                   // fp32 sum in slot order
                float f[8];
                unpack8(v[u], f);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaf(g[u], f[j], acc[j]);
            }
        }
        out[i] = pack8(acc);
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_PLAN_COVER);
}

// One wave per assignment (t,s): dYrows[row] = gate * dOut[t]; dgate = <dOut[t], Yrows[row]>.
__global__ void __launch_bounds__(256)
combine_bwd_kernel(const uint4 *__restrict__ Yrows, const uint4 *__restrict__ dOut,
                   const float *__restrict__ gates, const int32_t *__restrict__ row_of,
                   int N, int vec_per_row, int k, uint4 *__restrict__ dYrows, float *__restrict__ dgate,
                   int32_t *err_flag)
{
    const int lane = threadIdx.x & 63;
    const int a = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (a >= N) return;
    const int row = row_of[a];
    if ((unsigned)row >= (unsigned)N) {
        if (lane == 0) { atomicOr(err_flag, RELIBRA_ERR_PLAN_COVER); dgate[a] = 0.0f; }
        return;
    }
    const int t = a / k;
    const float g = gates[a];
    float dot = 0.0f;
    for (int c = lane; c < vec_per_row; c += 64) {
        float d[8], y[8], o[8];
        unpack8(dOut[(size_t)t * vec_per_row + c], d);
        unpack8(Yrows[(size_t)row * vec_per_row + c], y);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            o[j] = g * d[j];
            dot = fmaf(d[j], y[j], dot);
        }
        dYrows[(size_t)row * vec_per_row + c] = pack8(o);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
    if (lane == 0) dgate[a] = dot;
}

// row -> token: row_tok[row] = src_of[row] / k (assignment a = t*k + s belongs to token t).
__global__ void __launch_bounds__(256)
row_tokens_kernel(const int32_t *__restrict__ src_of, int N, int k, int T, int32_t *__restrict__ row_tok,
                  int32_t *__restrict__ err_flag)
{
    bool bad = false;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < N; i += gridDim.x * 256) {
        const int a = src_of[i];
        int t = 0;
        if (a < 0 || a / k >= T) bad = true; else t = a / k;
        row_tok[i] = t;
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_PLAN_COVER);
}

// row -> gate of the assignment the row serves: row_gate[row] = gates[src_of[row]] (gates flat [T*k]).
__global__ void __launch_bounds__(256)
row_gates_kernel(const int32_t *__restrict__ src_of, const float *__restrict__ gates, int N, float *__restrict__ row_gate,
                 int32_t *__restrict__ err_flag)
{
    bool bad = false;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < N; i += gridDim.x * 256) {
        const int a = src_of[i];
        float g = 0.0f;
        if (a < 0 || a >= N) bad = true; else g = gates[a];
        row_gate[i] = g;
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_PLAN_COVER);
}

inline int grid_for(size_t work_items, int per_block, int cap)
{
    size_t b = (work_items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (size_t)cap) b = cap;
    return (int)b;
}

}  // namespace relibra

using namespace relibra;

extern "C" int relibra_route_hist(const int32_t *ids_dev, int n_mb, int T, int k, int E,
                                  int32_t *counts_dev, int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (n_mb < 0 || T < 0 || k < 1 || E < 1 || E > kMaxExperts || k > E) return RELIBRA_EINVAL;
    if ((size_t)T * k > 0x7fffffffull) return RELIBRA_EINVAL;
    if (n_mb == 0) return RELIBRA_OK;
    if (!counts_dev || !err_flag_dev) return RELIBRA_EINVAL;
    const int per_mb = T * k;
    if (per_mb > 0 && !ids_dev) return RELIBRA_EINVAL;
    int copies_log2 = 4;                     // up to 16 copies of every bin, as many as fit the LDS budget
    while (copies_log2 > 0 && ((size_t)E << copies_log2) * sizeof(int32_t) > (size_t)kHistLdsBytes) --copies_log2;
    RELIBRA_LAUNCH(RELIBRA_K_HIST, stream, hist_kernel<<<(unsigned)n_mb, kHistThreads, ((size_t)E << copies_log2) * sizeof(int32_t), stream>>>(
        ids_dev, per_mb, E, copies_log2, ((per_mb & 3) == 0 && aligned16(ids_dev)) ? 1 : 0, counts_dev, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

static int permute_impl(const int32_t *ids_dev, const int32_t *inst_ptr_dev, const int32_t *inst_rows_dev,
                        const int32_t *inst_group_dev, const int32_t *group_offset_dev, const SrcSplit &split,
                        const void *X_dev, int T, int k, int E, int G, int h,
                        int32_t *row_of_dev, int32_t *src_of_dev, void *Xrows_dev,
                        void *workspace_dev, size_t workspace_bytes,
                        int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (T < 0 || k < 1 || E < 1 || E > kMaxExperts || k > E || G < 1 || h < 0) return RELIBRA_EINVAL;
    if ((size_t)T * k > 0x7fffffffull) return RELIBRA_EINVAL;
    const int N = T * k;
    if (N == 0) return RELIBRA_OK;
    if (!ids_dev || !inst_ptr_dev || (!inst_rows_dev && !split.src_first) || !inst_group_dev || !group_offset_dev ||
        !row_of_dev || !src_of_dev || !err_flag_dev || !workspace_dev)
        return RELIBRA_EINVAL;
    const bool with_rows = X_dev != nullptr || Xrows_dev != nullptr;
    if (with_rows && (!X_dev || !Xrows_dev || h < 8 || h % 8 || !aligned16(X_dev) || !aligned16(Xrows_dev)))
        return RELIBRA_EINVAL;
    if (workspace_bytes < relibra_workspace_bytes(RELIBRA_WS_PERMUTE, T, k, E, G, h, 0)) return RELIBRA_EWORKSPACE;
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    const PlanTables tables{inst_ptr_dev, inst_rows_dev, inst_group_dev, group_offset_dev};
    if (perm_in_one_block(N, E)) {
        const size_t lds = (size_t)(kSmallWaves + 2) * E * sizeof(int32_t);
        RELIBRA_LAUNCH(RELIBRA_K_PERM_SMALL, stream, perm_small_kernel<<<1, kSmallThreads, lds, stream>>>(ids_dev, N, E, G, ebits, tables,
                                                                row_of_dev, src_of_dev, err_flag_dev, split));
        RELIBRA_HIP_TRY(launch_check());
    } else {
        int32_t *unit_cnt = (int32_t *)workspace_dev;
        const int n_units = (N + kUnit - 1) / kUnit;
        const int blocks = (n_units + 3) / 4;
        const size_t lds = (size_t)4 * E * sizeof(int32_t);
        RELIBRA_LAUNCH(RELIBRA_K_PERM_COUNT, stream, perm_count_kernel<<<blocks, kPermThreads, lds, stream>>>(ids_dev, N, E, unit_cnt, src_of_dev, err_flag_dev));
        RELIBRA_HIP_TRY(launch_check());
        RELIBRA_LAUNCH(RELIBRA_K_PERM_SCAN, stream, perm_scan_kernel<<<E, 256, 0, stream>>>(unit_cnt, n_units, E));
        RELIBRA_HIP_TRY(launch_check());
        RELIBRA_LAUNCH(RELIBRA_K_PERM_RANK, stream, perm_rank_kernel<<<blocks, kPermThreads, lds, stream>>>(ids_dev, N, E, G, ebits, unit_cnt, tables,
                                                                row_of_dev, src_of_dev, err_flag_dev, split));
        RELIBRA_HIP_TRY(launch_check());
    }
    if (with_rows) {
        const int vpr = h / 8, lpr_log2 = lanes_per_row_log2(vpr, 4);
        const bool by_row = (size_t)N * h * sizeof(bf16_t) <= kGatherByRow;
        const int grid = grid_for((size_t)(by_row ? N : T), kRowThreads >> lpr_log2, 256 * 32);
        if (by_row) RELIBRA_LAUNCH(RELIBRA_K_GATHER, stream, gather_by_row_kernel<<<grid, kRowThreads, 0, stream>>>((const uint4 *)X_dev, src_of_dev,
                                                                 N, T, k, vpr, lpr_log2, (uint4 *)Xrows_dev));
        else RELIBRA_LAUNCH(RELIBRA_K_GATHER, stream, gather_by_token_kernel<<<grid, kRowThreads, 0, stream>>>((const uint4 *)X_dev, row_of_dev,
                                                          src_of_dev, N, T, k, vpr, lpr_log2, (uint4 *)Xrows_dev));
        RELIBRA_HIP_TRY(launch_check());
    }
    return RELIBRA_OK;
}

extern "C" int relibra_permute(const int32_t *ids_dev, const int32_t *inst_ptr_dev, const int32_t *inst_rows_dev,
                               const int32_t *inst_group_dev, const int32_t *group_offset_dev,
                               const void *X_dev, int T, int k, int E, int G, int h,
                               int32_t *row_of_dev, int32_t *src_of_dev, void *Xrows_dev,
                               void *workspace_dev, size_t workspace_bytes,
                               int32_t *err_flag_dev, relibra_stream stream_)
{
    if (T > 0 && !inst_rows_dev) return RELIBRA_EINVAL;
    return permute_impl(ids_dev, inst_ptr_dev, inst_rows_dev, inst_group_dev, group_offset_dev, SrcSplit{},
                        X_dev, T, k, E, G, h, row_of_dev, src_of_dev, Xrows_dev, workspace_dev, workspace_bytes,
                        err_flag_dev, stream_);
}

// The permutation for callers that cannot allocate: its unit-count matrix lives in a static device
// array instead of a caller's workspace.  Every GPU holds its own copy of the array at its own
// address; host code never uses the array's name as an address, only what hipGetSymbolAddress
// returned for the device that is current.
static __device__ __align__(256) int32_t scratch[RELIBRA_PERMUTE_STATIC_BYTES / sizeof(int32_t)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
int32_t *g_scratch_ptr[kMaxDevices] = {};     // per device: the device address of `scratch`
}  // namespace

// Device address of this device's copy of `scratch` (looked up once per device); null on failure.
static int32_t *scratch_for_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = (int32_t *)ptr;
    }
    return g_scratch_ptr[dev];
}

extern "C" int relibra_permute_static(const int32_t *ids_dev, const int32_t *inst_ptr_dev, const int32_t *inst_rows_dev,
                                      const int32_t *inst_group_dev, const int32_t *group_offset_dev,
                                      const void *X_dev, int T, int k, int E, int G, int h,
                                      int32_t *row_of_dev, int32_t *src_of_dev, void *Xrows_dev,
                                      int32_t *err_flag_dev, relibra_stream stream_)
{
    if (T > 0 && !inst_rows_dev) return RELIBRA_EINVAL;
    if (T < 0 || k < 1 || E < 1 || G < 1) return RELIBRA_EINVAL;
    const size_t need = relibra_workspace_bytes(RELIBRA_WS_PERMUTE, T, k, E, G, h, 0);
    if (need == 0 && (size_t)T * k > 0) return RELIBRA_EINVAL;
    if (need > (size_t)RELIBRA_PERMUTE_STATIC_BYTES) return RELIBRA_EWORKSPACE;     // beyond the static array
    int32_t *ws = scratch_for_current_device();
    if (!ws) return RELIBRA_EHIP;
    // Nothing in the array has to start at zero: the counting kernel overwrites every entry the other
    // two kernels read.
    return permute_impl(ids_dev, inst_ptr_dev, inst_rows_dev, inst_group_dev, group_offset_dev, SrcSplit{},
                        X_dev, T, k, E, G, h, row_of_dev, src_of_dev, Xrows_dev, ws, (size_t)RELIBRA_PERMUTE_STATIC_BYTES,
                        err_flag_dev, stream_);
}

extern "C" int relibra_permute_src(const int32_t *ids_dev, const int32_t *inst_ptr_dev,
                                   const int32_t *inst_group_dev, const int32_t *group_offset_dev,
                                   int EP, const int32_t *src_first_dev, const int32_t *inst_src_rows_dev,
                                   const int32_t *inst_src_base_dev,
                                   const void *X_dev, int T, int k, int E, int G, int h,
                                   int32_t *row_of_dev, int32_t *src_of_dev, void *Xrows_dev,
                                   void *workspace_dev, size_t workspace_bytes,
                                   int32_t *err_flag_dev, relibra_stream stream_)
{
    if (EP < 1 || T < 0 || T % EP) return RELIBRA_EINVAL;
    if (T > 0 && (!src_first_dev || !inst_src_rows_dev || !inst_src_base_dev)) return RELIBRA_EINVAL;
    const SrcSplit split{src_first_dev, inst_src_rows_dev, inst_src_base_dev, EP, k, T > 0 ? T / EP : 1};
    return permute_impl(ids_dev, inst_ptr_dev, nullptr, inst_group_dev, group_offset_dev, split,
                        X_dev, T, k, E, G, h, row_of_dev, src_of_dev, Xrows_dev, workspace_dev, workspace_bytes,
                        err_flag_dev, stream_);
}

extern "C" int relibra_unpermute_combine(int mode, const void *rows_dev, const void *tok_dev,
                                         const float *gates_dev, const int32_t *row_of_dev,
                                         int T, int k, int h,
                                         void *out_tok_dev, void *out_rows_dev, float *dgate_dev,
                                         int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (T < 0 || k < 1 || k > 64 || h < 8 || h % 8) return RELIBRA_EINVAL;
    if ((size_t)T * k > 0x7fffffffull) return RELIBRA_EINVAL;
    if (mode != RELIBRA_COMBINE_FWD && mode != RELIBRA_COMBINE_BWD && mode != RELIBRA_COMBINE_SUM)
        return RELIBRA_EINVAL;
    if (T == 0) return RELIBRA_OK;
    if (!rows_dev || !row_of_dev || !err_flag_dev || !aligned16(rows_dev)) return RELIBRA_EINVAL;
    const int N = T * k, vpr = h / 8;
    if (mode == RELIBRA_COMBINE_BWD) {
        if (!tok_dev || !gates_dev || !out_rows_dev || !dgate_dev || !aligned16(tok_dev) || !aligned16(out_rows_dev))
            return RELIBRA_EINVAL;
        RELIBRA_LAUNCH(RELIBRA_K_COMBINE_BWD, stream, combine_bwd_kernel<<<(N + 3) / 4, 256, 0, stream>>>((const uint4 *)rows_dev, (const uint4 *)tok_dev,
                                                            gates_dev, row_of_dev, N, vpr, k,
                                                            (uint4 *)out_rows_dev, dgate_dev, err_flag_dev));
    } else {
        if (!out_tok_dev || !aligned16(out_tok_dev)) return RELIBRA_EINVAL;
        const int grid = grid_for((size_t)T * vpr, 256, 256 * 64);
        if (mode == RELIBRA_COMBINE_FWD) {
            if (!gates_dev) return RELIBRA_EINVAL;
            RELIBRA_LAUNCH(RELIBRA_K_COMBINE_FWD, stream, combine_fwd_kernel<true><<<grid, 256, 0, stream>>>((const uint4 *)rows_dev, gates_dev, row_of_dev,
                                                               T, k, N, vpr, (uint4 *)out_tok_dev, err_flag_dev));
        } else {
            RELIBRA_LAUNCH(RELIBRA_K_COMBINE_SUM, stream, combine_fwd_kernel<false><<<grid, 256, 0, stream>>>((const uint4 *)rows_dev, nullptr, row_of_dev,
                                                                T, k, N, vpr, (uint4 *)out_tok_dev, err_flag_dev));
        }
    }
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" int relibra_row_tokens(const int32_t *src_of_dev, int N, int k, int T, int32_t *row_tok_dev,
                                  int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (N < 0 || k < 1 || T < 1) return RELIBRA_EINVAL;
    if (N == 0) return RELIBRA_OK;
    if (!src_of_dev || !row_tok_dev || !err_flag_dev) return RELIBRA_EINVAL;
    RELIBRA_LAUNCH(RELIBRA_K_ROW_TOKENS, stream, row_tokens_kernel<<<grid_for((size_t)N, 256, 1024), 256, 0, stream>>>(
        src_of_dev, N, k, T, row_tok_dev, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" int relibra_row_gates(const int32_t *src_of_dev, const float *gates_dev, int N, float *row_gate_dev,
                                 int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (N < 0) return RELIBRA_EINVAL;
    if (N == 0) return RELIBRA_OK;
    if (!src_of_dev || !gates_dev || !row_gate_dev || !err_flag_dev) return RELIBRA_EINVAL;
    RELIBRA_LAUNCH(RELIBRA_K_ROW_GATES, stream, row_gates_kernel<<<grid_for((size_t)N, 256, 1024), 256, 0, stream>>>(
        src_of_dev, gates_dev, N, row_gate_dev, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" const char *relibra_status_string(int status)
{
    switch (status) {
    case RELIBRA_OK: return "ok";
    case RELIBRA_EINVAL: return "invalid argument";
    case RELIBRA_ERANGE: return "table value out of range";
    case RELIBRA_EWORKSPACE: return "workspace too small";
    case RELIBRA_EHIP: return "HIP runtime error";
    case RELIBRA_EUNSUPPORTED: return "unsupported shape";
    case RELIBRA_ENOMEM: return "out of host memory";
    default: return "unknown status";
    }
}
