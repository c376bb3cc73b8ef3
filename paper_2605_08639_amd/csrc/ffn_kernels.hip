// Expert FFN forward / backward as grouped bf16 MFMA GEMMs (gfx950, v_mfma_f32_32x32x16_bf16).
//
// A wavefront always owns 64 rows x 128 columns of the output as 2 x 4 MFMA tiles with fp32
// accumulators, two wavefronts per SIMD.  Row-tiled kernels (forward, data gradients) come in two
// workgroup shapes: narrow, 4 waves = 128 rows x 256 columns, 72 KiB of LDS, two workgroups per
// compute unit; wide, 8 waves = 128 rows x 512 columns (gate/up: 2 x 256), one workgroup per
// compute unit, used where the wide tile divides the output width (the rows' slab is loaded once
// for twice the columns).  A group's tail of at most 64 rows runs as a 64-row tile.  Operand slabs
// of 32 k-values go global -> LDS directly (global_load_lds, 16 bytes per lane) through a ring of
// three slabs (four in the wide weight-gradient tile); the wide row tiles stage their rows 64
// k-values deep (full 128-byte lines) in a ring of their own, 144 KiB of LDS in all, and weights that lie
// k-contiguous too, half of their columns (or the gate, the up projection) at a time; see gemm_tile.h
// for the tile layouts and the pipeline.
//
// MFMA operand roles: the lanes carry the index that is contiguous in the output's memory
// only for the fp32 weight gradients (128-byte runs per store); for the bf16 row tensors the
// lanes carry the row index and each lane holds 4 consecutive columns, re-laid through per-wave
// LDS staging so that global accesses are 16 bytes per lane along rows.
// The ragged dimension is always clamped (reads) and masked (writes); a ragged contraction
// (weight gradients) is masked to zero in the fragments.
//
// Block index -> tile: XCD x (blockIdx % 8) takes the x-th eighth of the ordered tile list, so
// that operand tiles shared by neighbouring tiles are served by one L2.
//
// Weight gradients exist in two forms: per micro-batch (read-add-write of fp32 dW, replica slots
// summed into the home slot) and once per batch over every resident micro-batch, contracted in
// registers (wgrad_batched_kernel), which avoids the dW traffic that dominates short groups.
#include "gemm_tile.h"

#include <mutex>
#include <type_traits>

namespace relibra {

// Tile geometry: 4 waves, 128-row x 256-column tiles, three LDS slabs, two workgroups per
// compute unit (one group's prologue and epilogue overlap the other's MFMAs).
constexpr int BM = 128;                     // rows of a full row tile
constexpr int NWAVES = BM / 32;
constexpr int THREADS = NWAVES * 64;
constexpr int NSTAGES = 3;
constexpr int WGN = BM;                     // output columns of a weight-gradient tile

// ---------------------------------------------------------------- schedule tables
// Sanitised copies of the caller's group tables plus the list of row tiles, built on the
// device so that no host synchronisation is needed.
struct Sched {
    int32_t *hdr;          // [0] row tiles, [1] replica pairs
    int32_t *grp_row0, *grp_rows, *grp_expert, *grp_slot;   // [Gr]
    int32_t *tile_prefix;  // [Gr+1]
    int32_t *tile_group, *tile_row0, *tile_rows;            // [Rmax]
    int32_t *tile_band;    // [Rmax] band of the row tile: first row tile | number of row tiles << 24
    int32_t *pair_slot, *pair_expert;                       // [Gr]
    bf16_t *dGt, *dU;      // [n_rows, hff] (backward only)
};

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }
inline int max_row_tiles(int n_rows, int Gr) { return (n_rows + BM - 1) / BM + Gr; }
constexpr int kLdsBytes = NSTAGES * (256 + BM) * BK * 2;   // NSTAGES slabs of 256 + BM operand rows
// The row-tiled GEMMs also come with a tile twice as wide (512 columns, or 2 x 256 for gate and up)
// run by eight waves, one workgroup per compute unit: the same 128 x 64 per wave and two waves
// per SIMD, but the rows' slab is loaded once for twice the columns (five load instructions per
// wave and slab instead of six, one of them instead of two on the half-line k-contiguous rows);
// measured on dense problems of these shapes: 17-20 % faster.
constexpr int kWideRowWaves = 8;
// In the wide tiles the rows (the k-contiguous operand) are staged 64 k-values deep, in full 128-byte
// lines, through a ring of their own (KLoop, deep B side): three slabs of 512 weight rows plus three
// 64-deep tiles of 128 rows.
constexpr int kRowDepthWide = 2 * BK;
constexpr int kLdsBytesWide = NSTAGES * 512 * BK * 2 + ((NSTAGES + 3) / 2) * BM * kRowDepthWide * 2;
static_assert(kLdsBytesWide >= NSTAGES * (512 + BM) * BK * 2 && kLdsBytesWide >= 8 * 64 * 128 * 2 && kLdsBytesWide <= 160 * 1024,
              "slabs and the epilogue's staging (8 waves x 64 x 128 bf16) fit");
constexpr int kDgateParts = 4;                 // partial gate-gradient sums per row and 256-column tile (one per wave column at most)
inline size_t dgate_scratch_bytes(int n_rows, int hff) { return round256((size_t)kDgateParts * ((hff + 255) / 256) * n_rows * sizeof(float)); }
inline size_t sched_ints(int n_rows, int Gr) { return 8 + 4 * (size_t)Gr + (Gr + 1) + 4 * (size_t)max_row_tiles(n_rows, Gr) + 2 * (size_t)Gr; }
inline size_t ffn_ws_bytes(int n_rows, int Gr, int hff, bool bwd)
{
    size_t b = round256(sched_ints(n_rows, Gr) * sizeof(int32_t));
    if (bwd) b += 2 * round256((size_t)n_rows * hff * sizeof(bf16_t));
    return b;
}
inline Sched carve(void *ws, int n_rows, int Gr, int hff, bool bwd)
{
    Sched s;
    int32_t *p = (int32_t *)ws;
    const int R = max_row_tiles(n_rows, Gr);
    s.hdr = p; p += 8;
    s.grp_row0 = p; p += Gr;
    s.grp_rows = p; p += Gr;
    s.grp_expert = p; p += Gr;
    s.grp_slot = p; p += Gr;
    s.tile_prefix = p; p += Gr + 1;
    s.tile_group = p; p += R;
    s.tile_row0 = p; p += R;
    s.tile_rows = p; p += R;
    s.tile_band = p; p += R;
    s.pair_slot = p; p += Gr;
    s.pair_expert = p; p += Gr;
    char *q = (char *)ws + round256(sched_ints(n_rows, Gr) * sizeof(int32_t));
    s.dGt = s.dU = nullptr;
    if (bwd) {
        s.dGt = (bf16_t *)q;
        s.dU = (bf16_t *)(q + round256((size_t)n_rows * hff * sizeof(bf16_t)));
    }
    return s;
}

// Order of the tiles.  A group's row tiles are cut into bands of kBand; the tiles of a band run
// column tile by column tile, the band's row tiles innermost, so that the tiles a set of compute
// units works on at one time share weight column tiles as well as row tiles.  Against row-major
// order over the group this takes 15 to 27 % off the HBM reads of the forward gate/up and the
// dX kernels (measured, bands of 8) and about 1 % off their time: the L2 misses are not what
// bounds them.
constexpr int kBand = 8;
constexpr int kMaxSchedGroups = 8192;          // groups of one call (g_end - g_begin)

// The caller's group tables, for the kernel that works the schedule out (group_offset null: another one has).
struct SchedIn {
    const int32_t *group_offset, *group_expert, *group_dw_slot;
    int g_begin, Gr, n_rows, E, n_dw_slots, max_tiles;
    int32_t *err_flag;
};
struct SchedGroup {
    int lo, hi, expert, slot;
    bool bad;
};
// Group number i of the call, validated: a bad one is empty.
__device__ __forceinline__ SchedGroup sched_group(const SchedIn &in, int i)
{
    const int g = in.g_begin + i;
    SchedGroup r;
    r.lo = in.group_offset[g];
    r.hi = in.group_offset[g + 1];
    r.expert = in.group_expert[g];
    r.slot = in.group_dw_slot ? in.group_dw_slot[g] : 0;
    r.bad = r.lo < 0 || r.hi < r.lo || r.hi > in.n_rows || r.expert < -1 || r.expert >= in.E;
    if (in.group_dw_slot && r.expert >= 0 && (r.slot < 0 || r.slot >= in.n_dw_slots)) r.bad = true;
    if (r.bad) { r.lo = r.hi = 0; r.expert = -1; }
    if (r.expert < 0) r.hi = r.lo;
    return r;
}
// 256 threads.  prefix [Gr + 1] (LDS): row tiles in front of every group; returns their number.  WRITE: the
// groups go to the workspace too, and what is wrong with them to the flag.
template <bool WRITE>
__device__ __forceinline__ int sched_prefix(const SchedIn &in, const Sched &s, int32_t *prefix, int32_t *sums)
{
    const int tid = threadIdx.x;
    if (tid == 0) prefix[0] = 0;
    bool bad_any = false;
    int carry = 0;                             // tiles so far, the same in every thread
    for (int base = 0; base < in.Gr; base += 256) {
        const int i = base + tid;
        int tiles = 0;
        if (i < in.Gr) {
            const SchedGroup g = sched_group(in, i);
            bad_any |= g.bad;
            if (WRITE) {
                s.grp_row0[i] = g.lo;
                s.grp_rows[i] = g.hi - g.lo;
                s.grp_expert[i] = g.expert;
                s.grp_slot[i] = g.slot;
            }
            tiles = min((g.hi - g.lo + BM - 1) / BM, in.max_tiles + 1);
        }
        int all;
        const int upto = block_scan256(tiles, sums, all);
        if (tiles > 0 && carry + upto > in.max_tiles) bad_any = true;
        if (i < in.Gr) prefix[i + 1] = min(carry + upto, in.max_tiles);
        carry = min(carry + all, in.max_tiles);
    }
    if (WRITE && bad_any) atomicOr(in.err_flag, RELIBRA_ERR_GROUP_TABLE);
    __threadfence_block();
    __syncthreads();
    return carry;
}
// Last group whose prefix <= t: the one that holds row tile t (0 <= t < prefix[Gr]).
__device__ __forceinline__ int sched_group_of(const int32_t *prefix, int Gr, int t)
{
    int lo = 0, hi = Gr;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// 256 threads.  Validates the group tables of [g_begin, g_end) (bad groups become empty and raise
// the flag), lists the row tiles group by group, and lists the live replica slots.  The lists hold
// max_tiles: enough for any table whose groups do not overlap; an overlapping one ends there, flagged.
// prefix: Gr + 1 ints of LDS.
__device__ __forceinline__ void sched_write(const SchedIn &in, const Sched &s, int32_t *prefix, int32_t *sums)
{
    const int tid = threadIdx.x, Gr = in.Gr;
    const int total = sched_prefix<true>(in, s, prefix, sums);
    if (tid == 0) s.hdr[0] = total;
    for (int i = tid; i <= Gr; i += 256) s.tile_prefix[i] = prefix[i];
    for (int t = tid; t < total; t += 256) {
        const int lo = sched_group_of(prefix, Gr, t);
        const int j = t - prefix[lo];
        s.tile_group[t] = lo;
        s.tile_row0[t] = s.grp_row0[lo] + j * BM;
        s.tile_rows[t] = min(BM, s.grp_rows[lo] - j * BM);
        const int m = prefix[lo + 1] - prefix[lo], b0 = j / kBand * kBand;
        s.tile_band[t] = (prefix[lo] + b0) | (min(kBand, m - b0) << 24);
    }
    // live replica slots, in group order (256 groups at a time)
    int carry = 0;
    if (in.group_dw_slot) {
        for (int base = 0; base < Gr; base += 256) {
            const int i = base + tid;
            const bool live = i < Gr && s.grp_expert[i] >= 0 && s.grp_slot[i] >= in.E;
            int all;
            const int at = carry + block_scan256(live ? 1 : 0, sums, all) - 1;
            if (live) {
                s.pair_slot[at] = s.grp_slot[i];
                s.pair_expert[at] = s.grp_expert[i];
            }
            carry += all;
        }
    }
    if (tid == 0) s.hdr[1] = carry;
}

__global__ void __launch_bounds__(256)
sched_kernel(SchedIn in, Sched s)
{
    extern __shared__ int32_t prefix[];        // [Gr + 1]
    __shared__ int32_t sums[4];
    sched_write(in, s, prefix, sums);
}

// ---------------------------------------------------------------- tile lookup
struct RowTile {
    int group, row0, rows, expert, col0;
    bool valid;
};

// Order of the tiles of an n_r x n_c grid (weight gradients): bands of kGridBand rows; inside a
// band column by column, the band's rows innermost.  The ~64 tiles a set of compute units works
// on at one time then form a roughly square patch (8 x 8), which shares 8 + 8 operand tiles
// instead of 1 + 64.
constexpr int kGridBand = 8;
__device__ __forceinline__ void band_order(int idx, int n_r, int n_c, int &r, int &c)
{
    const int band = idx / (kGridBand * n_c), within = idx - band * (kGridBand * n_c);
    const int rows_here = min(kGridBand, n_r - band * kGridBand);
    c = within / rows_here;
    r = band * kGridBand + within - c * rows_here;
}

// Physical block -> tile.  The hardware deals blocks to the 8 XCDs round-robin (blockIdx % 8);
// XCD x takes the x-th eighth of the ordered tile list, so neighbouring tiles share one L2.
__device__ __forceinline__ RowTile find_row_tile(const Sched &s, int n_col_tiles, int col_tile_width, bool w_from_slot = false)
{
    RowTile t;
    const int n_rt = s.hdr[0];
    const int total = n_rt * n_col_tiles;
    const int per_xcd = (total + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    t.valid = logical < total && (int)(blockIdx.x >> 3) < per_xcd;
    if (!t.valid) return t;
    // the band that holds row tile logical / n_col_tiles holds tile `logical`
    const int band = s.tile_band[logical / n_col_tiles];
    const int first = band & 0xffffff, rows_here = band >> 24;
    const int within = logical - first * n_col_tiles;
    const int ct = within / rows_here, rt = first + within - ct * rows_here;
    t.group = s.tile_group[rt];
    t.row0 = s.tile_row0[rt];
    t.rows = s.tile_rows[rt];
    t.expert = w_from_slot ? s.grp_slot[t.group] : s.grp_expert[t.group];   // index of the parameter block
    t.col0 = ct * col_tile_width;
    return t;
}

// The k-loop's operand bases are scalar: says that the tile is the same in every lane, which the compiler cannot
// see of values that came through LDS.
__device__ __forceinline__ void make_uniform(RowTile &t)
{
    t.valid = __builtin_amdgcn_readfirstlane(t.valid ? 1 : 0) != 0;
    t.group = __builtin_amdgcn_readfirstlane(t.group);
    t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
    t.rows = __builtin_amdgcn_readfirstlane(t.rows);
    t.expert = __builtin_amdgcn_readfirstlane(t.expert);
    t.col0 = __builtin_amdgcn_readfirstlane(t.col0);
}

// The same from the caller's tables, for the first kernel of a call of few tiles: every block works out the part
// of the schedule that it needs (one read of the groups and a scan, about as long as the chain of lookups above),
// and the grid's last block, which has no tile, writes the tables for the kernels that follow.  Saves the
// scheduling kernel and the gap behind it.  lds: 4 ints and Gr + 1 more, free again afterwards.
__device__ __forceinline__ RowTile schedule_row_tile(const SchedIn &in, const Sched &s, int n_col_tiles, int col_tile_width, bool w_from_slot, char *lds)
{
    int32_t *sums = reinterpret_cast<int32_t *>(lds), *prefix = sums + 4;
    RowTile t{};
    if (blockIdx.x == gridDim.x - 1) {
        sched_write(in, s, prefix, sums);
        return t;
    }
    const int total = sched_prefix<false>(in, s, prefix, sums) * n_col_tiles;
    const int per_xcd = (total + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    t.valid = logical < total && (int)(blockIdx.x >> 3) < per_xcd;
    if (t.valid) {
        const int rt0 = logical / n_col_tiles, lo = sched_group_of(prefix, in.Gr, rt0);
        const int m = prefix[lo + 1] - prefix[lo], b0 = (rt0 - prefix[lo]) / kBand * kBand;
        const int first = prefix[lo] + b0, rows_here = min(kBand, m - b0);
        const int within = logical - first * n_col_tiles;
        const int ct = within / rows_here, j = b0 + within - ct * rows_here;
        const SchedGroup g = sched_group(in, lo);
        t.group = lo;
        t.row0 = g.lo + j * BM;
        t.rows = min(BM, g.hi - g.lo - j * BM);
        t.expert = w_from_slot ? g.slot : g.expert;
        t.col0 = ct * col_tile_width;
    }
    __syncthreads();                                          // the LDS goes to the operand slabs
    return t;
}

// 1 / (1 + e^-x) with the hardware reciprocal (1 ulp; the result is rounded to bf16 anyway): a
// plain division expands to the ten-instruction IEEE sequence, 128 times per lane and tile.
__device__ __forceinline__ float sigmoidf_(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

__device__ __forceinline__ uint2 pack4bf(float a, float b, float c, float d)
{
    uint2 w;
    w.x = pack2bf(a, b);
    w.y = pack2bf(c, d);
    return w;
}
__device__ __forceinline__ void unpack4bf(uint2 w, float (&f)[4])
{
    f[0] = __uint_as_float(w.x << 16);
    f[1] = __uint_as_float(w.x & 0xffff0000u);
    f[2] = __uint_as_float(w.y << 16);
    f[3] = __uint_as_float(w.y & 0xffff0000u);
}

// Per-wave LDS staging between the accumulator layout (a lane holds 4 consecutive columns of
// its row) and the row-major layout (a row's columns spread over consecutive lanes), so that
// global accesses of the epilogue are 16 bytes per lane along rows: full cache lines.
// A wave stages 64 rows x NCOLS bf16; 16-byte pieces of a row are XOR-ed with the row number.
template <int NCOLS>
struct WaveStage {
    static constexpr int PIECES = NCOLS / 8;
    static constexpr int BYTES = 64 * NCOLS * 2;
    static constexpr int ROWS_PER_PASS = 64 / PIECES;
    static constexpr int PASSES = 64 / ROWS_PER_PASS;

    // accumulator side: 8 bytes = columns col..col+3 (col % 4 == 0) of `row`
    static __device__ __forceinline__ int acc_addr(int row, int col)
    {
        return row * (NCOLS * 2) + ((((col >> 3) ^ row) & (PIECES - 1)) << 4) + ((col >> 2) & 1) * 8;
    }
    static __device__ __forceinline__ void put(char *buf, int row, int col, uint2 v) { *reinterpret_cast<uint2 *>(buf + acc_addr(row, col)) = v; }
    static __device__ __forceinline__ uint2 get(const char *buf, int row, int col) { return *reinterpret_cast<const uint2 *>(buf + acc_addr(row, col)); }

    // row-major side: stage -> global, rows grow0.. of a tensor with leading dimension ld.
    // All LDS reads first, then the (predicated) stores: left to itself the compiler moves every
    // read into the branch of its store, and each store then waits for its own read in turn.
    // Only columns col_from <= c < n_dim are stored.
    static __device__ __forceinline__ void flush(const char *buf, bf16_t *out, int ld, int grow0, int row_end,
                                                 int gcol0, int n_dim, int lane, int col_from = 0)
    {
        uint4 v[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            v[p] = *reinterpret_cast<const uint4 *>(buf + r * (NCOLS * 2) + (((piece ^ r) & (PIECES - 1)) << 4));
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p)          // the values are needed here: the reads stay above
            asm volatile("" : "+v"(v[p].x), "+v"(v[p].y), "+v"(v[p].z), "+v"(v[p].w));
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            if (grow0 + r < row_end && gcol0 + piece * 8 < n_dim && gcol0 + piece * 8 >= col_from)
                *reinterpret_cast<uint4 *>(out + (size_t)(grow0 + r) * ld + gcol0 + piece * 8) = v[p];
        }
    }
    // global -> stage.  Rows and columns beyond the tensor are read from clamped (valid) addresses
    // instead of being skipped: what lands in their places is never stored by flush, and without
    // the predicates all loads of the fill are in flight together (predicated, every load was
    // waited for before the next one went out: one memory round trip per pass).
    // Needs grow0 < row_end and n_dim >= 8.
    // two tensors of the same shape into two staging areas, all loads in flight together
    static __device__ __forceinline__ void fill2(char *buf0, char *buf1, const bf16_t *in0, const bf16_t *in1, int ld, int grow0,
                                                 int row_end, int gcol0, int n_dim, int lane)
    {
        uint4 v0[PASSES], v1[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            const size_t at = (size_t)min(grow0 + r, row_end - 1) * ld + min(gcol0 + piece * 8, n_dim - 8);
            v0[p] = *reinterpret_cast<const uint4 *>(in0 + at);
            v1[p] = *reinterpret_cast<const uint4 *>(in1 + at);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            const int at = r * (NCOLS * 2) + (((piece ^ r) & (PIECES - 1)) << 4);
            *reinterpret_cast<uint4 *>(buf0 + at) = v0[p];
            *reinterpret_cast<uint4 *>(buf1 + at) = v1[p];
        }
    }
    static __device__ __forceinline__ void fill(char *buf, const bf16_t *in, int ld, int grow0, int row_end,
                                                int gcol0, int n_dim, int lane)
    {
        uint4 v[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            const int gr = min(grow0 + r, row_end - 1), gc = min(gcol0 + piece * 8, n_dim - 8);
            v[p] = *reinterpret_cast<const uint4 *>(in + (size_t)gr * ld + gc);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + lane / PIECES, piece = lane % PIECES;
            *reinterpret_cast<uint4 *>(buf + r * (NCOLS * 2) + (((piece ^ r) & (PIECES - 1)) << 4)) = v[p];
        }
    }
};

// LDS operations of one wave execute in order; this keeps the compiler from moving them across
// the hand-over between the two layouts and waits for the data.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The k-loops issue a slab's loads one by one between the MFMAs of a slab period instead of in one
// burst behind the barrier (gemm_tile.h); needs a ring of at least three slabs to pay.
constexpr bool kSpreadLoads = true;

// Wave layouts: every wave owns 64 rows; the waves left over split the columns.
template <int BB, int NWV = NWAVES> struct Waves { static constexpr int B = BB / 64, A = NWV / B; };

// ---------------------------------------------------------------- forward
// Gt = X Wg^T, U = X Wu^T (one pass over X), A = silu(Gt) * U.   Column tile: 128 of h'.
template <int BB, bool WT, int AW = 128>
__device__ __forceinline__ void fwd_gate_up_body(const RowTile &t, const bf16_t *X, const int32_t *row_tok, int tok_last,
                                                 const bf16_t *Wg, const bf16_t *Wu,
                                                 int h, int hff, bf16_t *Gt, bf16_t *U, bf16_t *Aout,
                                                 const float *row_gate, bf16_t *Agout, char *lds)
{
    constexpr int NWV = AW == 128 ? NWAVES : kWideRowWaves;
    using WV = Waves<BB, NWV>;
    constexpr bool ALT = !WT && AW != 128;                    // k-contiguous weights in the wide tile: gate and up slabs in turn
    using WTile = typename std::conditional<WT, KsTile<AW>, KcTile<AW, (ALT ? kRowDepthWide : BK), ALT>>::type;
    using KL = KLoop<WTile, KcTile<BB, (AW == 128 ? BK : kRowDepthWide)>, 2, 1, AW, BB, WV::A, WV::B, 1, false, NSTAGES, kSpreadLoads, false, ALT>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t wofs = (size_t)t.expert * hff * h;
    const int ldw = WT ? hff : h;                             // (n in h', k in h) at [n*h + k], or at [k*h' + n]
    const int col0 = ALT ? min(t.col0, hff - AW) : t.col0;    // ALT tiles are whole: the last one starts earlier and stores its own columns only
    const Operand A[1][2] = {{{Wg + wofs, ldw, col0, hff - 1}, {Wu + wofs, ldw, col0, hff - 1}}};
    // rows of the group: a gathered copy (row_tok == nullptr), or token rows fetched through row_tok
    const Operand B[1][1] = {{{X, h, t.row0, t.row0 + t.rows - 1, row_tok, tok_last}}};
    typename KL::Acc acc;
    KL::zero(acc);
    KL::run(acc, A, B, h / BK, h, lds, tid);
    // epilogue: three tensors, one after the other through this wave's staging area
    constexpr int WCOLS = AW / WV::A;                         // columns of this wave per tensor
    using ST = WaveStage<WCOLS>;
    static_assert(KL::TB == 2, "a wave owns 64 rows");
    __syncthreads();                                          // every wave is done with the operand slabs
    char *buf = lds + wave * ST::BYTES;
    const int wrow0 = t.row0 + (wave % WV::B) * 64, row_end = t.row0 + t.rows;
    const int wcol0 = col0 + (wave / WV::B) * WCOLS;
    // With row gates: the activations scaled by the gate of the row's assignment, as a fourth tensor
    // (Agout) or, with Agout == Aout, in place of the plain ones (the down projection then yields
    // gated rows and the combine is a plain sum).
    const bool gated = row_gate != nullptr, in_place = gated && Agout == Aout;
    float gate[KL::TB];
#pragma unroll
    for (int tb = 0; tb < KL::TB; ++tb) gate[tb] = gated ? row_gate[min(wrow0 + tb * 32 + (lane & 31), row_end - 1)] : 0.0f;
#pragma unroll
    for (int which = 0; which < 4; ++which) {
        if (which == 3 && !gated) break;
        if (which == 2 && in_place) continue;                 // the fourth pass writes A's place
#pragma unroll
        for (int tb = 0; tb < KL::TB; ++tb)
#pragma unroll
            for (int ta = 0; ta < KL::TA; ++ta)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float g = acc[0][ta][tb][q * 4 + e], u = acc[1][ta][tb][q * 4 + e];
                        v[e] = which == 0 ? g : which == 1 ? u : which == 2 ? g * sigmoidf_(g) * u : gate[tb] * (g * sigmoidf_(g) * u);
                    }
                    ST::put(buf, tb * 32 + (lane & 31), ta * 32 + q * 8 + (lane >> 5) * 4, pack4bf(v[0], v[1], v[2], v[3]));
                }
        wave_lds_fence();
        ST::flush(buf, which == 0 ? Gt : which == 1 ? U : which == 2 ? Aout : Agout, hff, wrow0, row_end, wcol0, hff, lane, t.col0);
        wave_lds_fence();
    }
}

// WT: Wg, Wu given as transposed copies [h][h'] (contraction index strided, transposing LDS reads).
template <bool WT, int AW = 128>
__global__ void __launch_bounds__(AW == 128 ? THREADS : kWideRowWaves * 64, AW == 128 ? 2 : 1)
fwd_gate_up_kernel(Sched s, const bf16_t *__restrict__ X, const int32_t *__restrict__ row_tok, int tok_last,
                   const bf16_t *__restrict__ Wg, const bf16_t *__restrict__ Wu, int h, int hff, int n_col_tiles,
                   bf16_t *__restrict__ Gt, bf16_t *__restrict__ U, bf16_t *__restrict__ Aout,
                   const float *__restrict__ row_gate, bf16_t *__restrict__ Agout, SchedIn in)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    RowTile t;
    if (AW == 128 && in.group_offset) t = schedule_row_tile(in, s, n_col_tiles, AW, false, lds);
    else t = find_row_tile(s, n_col_tiles, AW);
    if (AW == 128) make_uniform(t);
    if (!t.valid) return;
    if (t.rows > BM / 2) fwd_gate_up_body<BM, WT, AW>(t, X, row_tok, tok_last, Wg, Wu, h, hff, Gt, U, Aout, row_gate, Agout, lds);
    else fwd_gate_up_body<BM / 2, WT, AW>(t, X, row_tok, tok_last, Wg, Wu, h, hff, Gt, U, Aout, row_gate, Agout, lds);
}

// Gate-side fusion of the activation backward (EPI = 2).  With the upstream gradient of row r
// taken straight from the token tensor, dY'[r] = dOut[tok(r)] (the combine's gate left out), the
// accumulators hold dA' = dY' Wd, and
//   dGt = gate * dA' * U * silu'(Gt),  dU = gate * dA' * silu(Gt),  dgate[r] = sum_n dA'[r][n] * A[r][n]
// with A = silu(Gt) * U recomputed in place: the same values as scaling dOut by the gate first
// and reducing dOut against the down projection's output, without either pass over the rows.
struct GateFusion {
    const int32_t *row_tok = nullptr;   // [n_rows] row -> token (null: P0 holds group-ordered rows)
    int tok_last = 0;
    const float *row_gate = nullptr;    // [n_rows]
    float *dgate_part = nullptr;        // [kDgateParts * column tiles][n_rows] partial row sums, summed later in slot order
    int n_rows = 0;
};

// Shared body of the three single-accumulator row-tiled GEMMs.  EPI: 0 = store bf16 (Y, dX);
// 1 = dA -> dGt, dU (needs Gt, U); 2 = the same with the gate fused in (GateFusion).
// W_KS: weights k-strided (data gradients).  NPH = 2 sums two products (dX = dGt Wg + dU Wu).
template <int BB, bool W_KS, int NPH, int EPI, int AW = 256>
__device__ __forceinline__ void row_gemm_body(const RowTile &t, const bf16_t *P0, const bf16_t *P1, int ldp,
                                              const bf16_t *W0, const bf16_t *W1, int ldw, int n_dim, int k_dim,
                                              bf16_t *out0, bf16_t *out1, const bf16_t *Gt, const bf16_t *U, char *lds,
                                              const GateFusion &gf = GateFusion{})
{
    constexpr int NWV = AW == 256 ? NWAVES : kWideRowWaves;
    using WV = Waves<BB, NWV>;
    // k-contiguous weights in the wide tile: every wave's columns in two halves that take turns (KLoop, ALT)
    constexpr bool ALT = !W_KS && AW != 256;
    constexpr int NA = ALT ? 2 : 1, BA = AW / NA, SEG = ALT ? BA / WV::A : 0;
    using WT = typename std::conditional<W_KS, KsTile<BA>, KcTile<BA, (ALT ? kRowDepthWide : BK), ALT>>::type;
    using KL = KLoop<WT, KcTile<BB, (AW == 256 ? BK : kRowDepthWide)>, NA, 1, BA, BB, WV::A, WV::B, NPH, false, NSTAGES, kSpreadLoads, false, ALT>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Operand A[NPH][NA], B[NPH][1];
    const int col0 = ALT ? min(t.col0, n_dim - AW) : t.col0;  // ALT tiles are whole: the last one starts earlier and stores its own columns only
#pragma unroll
    for (int a = 0; a < NA; ++a) A[0][a] = {W0, ldw, col0 + a * SEG, n_dim - 1, nullptr, 0, SEG};
    B[0][0] = {P0, ldp, t.row0, t.row0 + t.rows - 1};
    if (EPI == 2 && gf.row_tok) B[0][0] = {P0, ldp, t.row0, t.row0 + t.rows - 1, gf.row_tok, gf.tok_last};
    if (NPH == 2) {
#pragma unroll
        for (int a = 0; a < NA; ++a) A[NPH - 1][a] = {W1, ldw, col0 + a * SEG, n_dim - 1, nullptr, 0, SEG};
        B[NPH - 1][0] = {P1, ldp, t.row0, t.row0 + t.rows - 1};
    }
    typename KL::Acc acc;
    KL::zero(acc);
    KL::run(acc, A, B, k_dim / BK, k_dim, lds, tid);
    constexpr int WCOLS = AW / WV::A, TALL = NA * KL::TA;     // a wave's columns: MFMA tile ta of TALL is tile ta % TA of half ta / TA
    using ST = WaveStage<WCOLS>;
    static_assert(KL::TB == 2, "a wave owns 64 rows");
    __syncthreads();                                          // every wave is done with the operand slabs
    char *buf = lds + wave * ST::BYTES;
    const int wrow0 = t.row0 + (wave % WV::B) * 64, row_end = t.row0 + t.rows;
    const int wcol0 = col0 + (wave / WV::B) * WCOLS;
    if (EPI == 0) {
#pragma unroll
        for (int tb = 0; tb < KL::TB; ++tb)
#pragma unroll
            for (int ta = 0; ta < TALL; ++ta)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ST::put(buf, tb * 32 + (lane & 31), ta * 32 + q * 8 + (lane >> 5) * 4,
                            pack4bf(acc[ta / KL::TA][ta % KL::TA][tb][q * 4], acc[ta / KL::TA][ta % KL::TA][tb][q * 4 + 1],
                                    acc[ta / KL::TA][ta % KL::TA][tb][q * 4 + 2], acc[ta / KL::TA][ta % KL::TA][tb][q * 4 + 3]));
        wave_lds_fence();
        ST::flush(buf, out0, n_dim, wrow0, row_end, wcol0, n_dim, lane, t.col0);
    } else {
        // dA (in the accumulators) -> dGt, dU, half of the wave's columns at a time: Gt and U come
        // in through two staging areas and are overwritten in place by dGt and dU.
        using SH = WaveStage<WCOLS / 2>;
        constexpr int TAH = TALL / 2;
        static_assert(TAH >= 1, "at least 64 columns per wave");
        char *buf_g = buf, *buf_u = buf + SH::BYTES;
        float gate[KL::TB], dsum[KL::TB];
#pragma unroll
        for (int tb = 0; tb < KL::TB; ++tb) {
            gate[tb] = EPI == 2 ? gf.row_gate[min(wrow0 + tb * 32 + (lane & 31), row_end - 1)] : 1.0f;
            dsum[tb] = 0.0f;
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int hcol0 = wcol0 + half * (WCOLS / 2);
            SH::fill2(buf_g, buf_u, Gt, U, n_dim, wrow0, row_end, hcol0, n_dim, lane);
            wave_lds_fence();
            // this half's share of the row sums; a half (32 or 64 columns, n_dim % 64 == 0) lies inside
            // the tensor or outside it as a whole, and outside it holds clamped copies
            float hsum[KL::TB];
#pragma unroll
            for (int tb = 0; tb < KL::TB; ++tb) hsum[tb] = 0.0f;
#pragma unroll
            for (int tb = 0; tb < KL::TB; ++tb)
#pragma unroll
                for (int th = 0; th < TAH; ++th)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int ta = half * TAH + th;
                        const int row = tb * 32 + (lane & 31), col = th * 32 + q * 8 + (lane >> 5) * 4;
                        float g[4], u[4], dg[4], du[4], pa[4];
                        unpack4bf(SH::get(buf_g, row, col), g);
                        unpack4bf(SH::get(buf_u, row, col), u);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float da = acc[ta / KL::TA][ta % KL::TA][tb][q * 4 + e];
                            const float sg = sigmoidf_(g[e]);
                            if (EPI == 2) {
                                pa[e] = da * (g[e] * sg * u[e]);
                                const float dag = gate[tb] * da;
                                dg[e] = dag * u[e] * (sg * (1.0f + g[e] * (1.0f - sg)));
                                du[e] = dag * (g[e] * sg);
                            } else {
                                dg[e] = da * u[e] * (sg * (1.0f + g[e] * (1.0f - sg)));
                                du[e] = da * (g[e] * sg);
                            }
                        }
                        SH::put(buf_g, row, col, pack4bf(dg[0], dg[1], dg[2], dg[3]));
                        SH::put(buf_u, row, col, pack4bf(du[0], du[1], du[2], du[3]));
                        // The running sum is needed only after the loop, and the compiler would sink all
                        // of its arithmetic down there, parking every operand in scratch memory on the
                        // way; an assembly statement that "uses" the sum keeps each add where it is.
                        if (EPI == 2) {
                            hsum[tb] += (pa[0] + pa[1]) + (pa[2] + pa[3]);
                            asm volatile("" : "+v"(hsum[tb]));
                        }
                    }
            wave_lds_fence();
            SH::flush(buf_g, out0, n_dim, wrow0, row_end, hcol0, n_dim, lane);
            SH::flush(buf_u, out1, n_dim, wrow0, row_end, hcol0, n_dim, lane);
            wave_lds_fence();
            if (EPI == 2 && hcol0 < n_dim) {
#pragma unroll
                for (int tb = 0; tb < KL::TB; ++tb) dsum[tb] += hsum[tb];
            }
        }
        if (EPI == 2) {
            // a row's columns lie on lanes l and l + 32; one partial sum per row and wave column, in the
            // slot of its 256 columns (kDgateParts slots each; a wave column is 64 or 128 wide)
            constexpr int PER = 256 / WCOLS;
            static_assert(PER >= 1 && PER <= kDgateParts, "wave columns per 256 columns");
            const int slot = (wcol0 / 256) * kDgateParts + (wcol0 % 256) / WCOLS;
#pragma unroll
            for (int tb = 0; tb < KL::TB; ++tb) {
                const float total = dsum[tb] + __shfl_xor(dsum[tb], 32);
                const int r = wrow0 + tb * 32 + (lane & 31);
                if (lane < 32 && r < row_end) {
                    gf.dgate_part[(size_t)slot * gf.n_rows + r] = total;
#pragma unroll
                    for (int extra = PER; extra < kDgateParts; extra += PER)      // the slots this tile shape does not fill
                        gf.dgate_part[(size_t)(slot + extra) * gf.n_rows + r] = 0.0f;
                }
            }
        }
    }
}

// Y = A Wd^T.  WT: Wd given as a transposed copy [h'][h].
template <bool WT, int AW = 256>
__global__ void __launch_bounds__(AW == 256 ? THREADS : kWideRowWaves * 64, AW == 256 ? 2 : 1)
fwd_down_kernel(Sched s, const bf16_t *__restrict__ Ain, const bf16_t *__restrict__ Wd, int h, int hff,
                int n_col_tiles, bf16_t *__restrict__ Y)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const RowTile t = find_row_tile(s, n_col_tiles, AW);
    if (!t.valid) return;
    const bf16_t *W = Wd + (size_t)t.expert * h * hff;
    const int ldw = WT ? h : hff;                             // (n in h, k in h') at [n*h' + k], or at [k*h + n]
    if (t.rows > BM / 2) row_gemm_body<BM, WT, 1, 0, AW>(t, Ain, nullptr, hff, W, nullptr, ldw, h, hff, Y, nullptr, nullptr, nullptr, lds);
    else row_gemm_body<BM / 2, WT, 1, 0, AW>(t, Ain, nullptr, hff, W, nullptr, ldw, h, hff, Y, nullptr, nullptr, nullptr, lds);
}

// ---------------------------------------------------------------- backward
// dA = dY Wd, then dGt = dA * U * silu'(Gt), dU = dA * silu(Gt).
// WT = false: Wd as the forward pass holds it, [h][h'], contraction index strided (transposing
// LDS reads, full-line loads: the faster operand path).  WT = true: a transposed copy [h'][h],
// contraction index contiguous.
template <bool WT, bool GATED = false, int AW = 256>
__global__ void __launch_bounds__(AW == 256 ? THREADS : kWideRowWaves * 64, AW == 256 ? 2 : 1)
bwd_act_kernel(Sched s, const bf16_t *__restrict__ dY, const bf16_t *__restrict__ Wd,
               const bf16_t *__restrict__ Gt, const bf16_t *__restrict__ U, int h, int hff, int n_col_tiles,
               int w_from_slot, GateFusion gf, SchedIn in)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    RowTile t;
    if (AW == 256 && in.group_offset) t = schedule_row_tile(in, s, n_col_tiles, AW, w_from_slot != 0, lds);
    else t = find_row_tile(s, n_col_tiles, AW, w_from_slot != 0);
    if (AW == 256) make_uniform(t);
    if (!t.valid) return;
    const bf16_t *W = Wd + (size_t)t.expert * h * hff;      // (n in h', k in h) at [k*h' + n], or at [n*h + k]
    const int ldw = WT ? h : hff;
    constexpr int EPI = GATED ? 2 : 1;
    if (t.rows > BM / 2) row_gemm_body<BM, !WT, 1, EPI, AW>(t, dY, nullptr, h, W, nullptr, ldw, hff, h, s.dGt, s.dU, Gt, U, lds, gf);
    else row_gemm_body<BM / 2, !WT, 1, EPI, AW>(t, dY, nullptr, h, W, nullptr, ldw, hff, h, s.dGt, s.dU, Gt, U, lds, gf);
}

// dgate of the gate-fused backward: the partial row sums of the activation backward added up in
// slot order (fixed order: bit-reproducible), written per row or, with src_of, at the assignment
// the row serves (the [T,k] layout of the gates).  Rows outside [group_offset[g_begin],
// group_offset[g_end]) were not computed and are left alone.
__global__ void __launch_bounds__(256)
dgate_reduce_kernel(const float *__restrict__ part, int n_slots, int n_rows, const int32_t *__restrict__ group_offset,
                    int g_begin, int g_end, const int32_t *__restrict__ src_of, float *__restrict__ dgate,
                    int32_t *__restrict__ err_flag)
{
    const int lo = max(0, min(group_offset[g_begin], n_rows)), hi = max(lo, min(group_offset[g_end], n_rows));
    bool bad = false;
    for (int r = lo + blockIdx.x * 256 + threadIdx.x; r < hi; r += gridDim.x * 256) {
        float sum = 0.0f;
        for (int p = 0; p < n_slots; ++p) sum += part[(size_t)p * n_rows + r];
        int at = r;
        if (src_of) {
            at = src_of[r];
            if (at < 0 || at >= n_rows) { bad = true; continue; }
        }
        dgate[at] = sum;
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_PLAN_COVER);
}

// dX = dGt Wg + dU Wu (one accumulator, the contraction runs over both products).
// WT as above: Wg, Wu [h'][h] as the forward pass holds them, or transposed copies [h][h'].
template <bool WT, int AW = 256>
__global__ void __launch_bounds__(AW == 256 ? THREADS : kWideRowWaves * 64, AW == 256 ? 2 : 1)
bwd_dx_kernel(Sched s, const bf16_t *__restrict__ Wg, const bf16_t *__restrict__ Wu, int h, int hff,
              int n_col_tiles, int w_from_slot, bf16_t *__restrict__ dX)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const RowTile t = find_row_tile(s, n_col_tiles, AW, w_from_slot != 0);
    if (!t.valid) return;
    const size_t wofs = (size_t)t.expert * hff * h;         // (n in h, k in h') at [k*h + n], or at [n*h' + k]
    const int ldw = WT ? hff : h;
    if (t.rows > BM / 2) row_gemm_body<BM, !WT, 2, 0, AW>(t, s.dGt, s.dU, hff, Wg + wofs, Wu + wofs, ldw, h, hff, dX, nullptr, nullptr, nullptr, lds);
    else row_gemm_body<BM / 2, !WT, 2, 0, AW>(t, s.dGt, s.dU, hff, Wg + wofs, Wu + wofs, ldw, h, hff, dX, nullptr, nullptr, nullptr, lds);
}

// Transposed copy of per-expert matrices, out[e][j][i] = in[e][i][j]: 128 x 128 tiles through LDS, 16-byte
// accesses on both global sides (256 contiguous bytes of a row), eight loads in flight per thread.  LDS holds the
// tile row by row, 16-byte pieces XOR-ed with the row's octet: the 64 lanes of a read (16 octets of rows x the
// four column pairs of a piece) fall into 64 banks.  A thread reads a pair of columns at a time and stores two
// output rows' pieces.  Bound by the copy rate; against 64 x 64 tiles read two bytes at a time: 128 experts of
// 4096 x 1536 632 -> 608 us a tensor (5.3 TB/s), 8 of 4096 x 14336 381 -> 365.
constexpr int kTrTile = 128;
__global__ void __launch_bounds__(256)
transpose_experts_kernel(const bf16_t *__restrict__ in, int rows, int cols, bf16_t *__restrict__ out)
{
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) char tile[kTrTile * kTrTile * 2];
    const size_t base = (size_t)blockIdx.z * rows * cols;
    const int r0 = blockIdx.y * kTrTile, c0 = blockIdx.x * kTrTile, tid = threadIdx.x;
    u32x4_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {          // beyond the matrix: its last row or piece again, not stored
        const int r = min(r0 + i * 16 + (tid >> 4), rows - 1), c = min(c0 + (tid & 15) * 8, cols - 8);
        v[i] = *reinterpret_cast<const u32x4_t *>(in + base + (size_t)r * cols + c);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = i * 16 + (tid >> 4), piece = (tid & 15) ^ ((r >> 3) & 15);
        *reinterpret_cast<u32x4_t *>(tile + r * 256 + piece * 16) = v[i];
    }
    __syncthreads();
    const int oct = tid & 15;              // rows r0 + oct * 8 .. of the matrix: one piece of the output rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (i * 16 + (tid >> 4)) * 2;
        uint32_t w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            w[j] = *reinterpret_cast<const uint32_t *>(tile + (oct * 8 + j) * 256 + (((c >> 3) ^ oct) * 16) + (c & 7) * 2);
        u32x4_t lo, hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x05040100);       // low halves of both words
            hi[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x07060302);       // high halves
        }
        if (r0 + oct * 8 < rows) {
            bf16_t *to = out + base + (size_t)(c0 + c) * rows + r0 + oct * 8;
            if (c0 + c < cols) *reinterpret_cast<u32x4_t *>(to) = lo;
            if (c0 + c + 1 < cols) *reinterpret_cast<u32x4_t *>(to + rows) = hi;
        }
    }
}

// Weight-gradient epilogue.  The accumulators hold, per lane, one column n and 16 rows m of each
// MFMA tile; each 32 x 64 fp32 block of the wave goes through this wave's 8 KiB of LDS and
// leaves as 16 bytes per lane along n: 1 KiB per store (or load-add-store) instruction.
// stream: gradients larger than the last-level cache leave with a streaming hint, so that they do not push
// out operands that other tiles still read (128 experts of 2048 x 768: 1 to 3 % of the kernel).
template <class KL, int NA, int BA, int NWV = NWAVES>
__device__ __forceinline__ void wgrad_epilogue(typename KL::Acc &acc, char *lds, float *out0, float *out1, size_t base,
                                               int m0, int n0, int m_dim, int n_dim, bool add, bool stream, int wave, int lane)
{
    static_assert(KL::TB % 2 == 0, "a wave owns a multiple of 64 columns");
    __syncthreads();                                          // every wave is done with the operand slabs
    float *buf = reinterpret_cast<float *>(lds + wave * 8192);
    const int wm0 = m0 + (wave / (NWV / 2)) * (BA / 2);
    const int col4 = lane & 15;
#pragma unroll
    for (int half = 0; half < KL::TB / 2; ++half)             // 64 columns of the wave at a time
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int ta = 0; ta < KL::TA; ++ta) {
            const int wn0 = n0 + (wave % (NWV / 2)) * (KL::TB * 32) + half * 64, gcol = wn0 + col4 * 4;
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    buf[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 64 + tb * 32 + (lane & 31)] = acc[a][ta][half * 2 + tb][v];
            wave_lds_fence();
            float *out = (a == 0 ? out0 : out1) + base;
            float4 val[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) val[p] = *reinterpret_cast<const float4 *>(buf + (p * 4 + (lane >> 4)) * 64 + col4 * 4);
            if (add) {
                float4 old[8];
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const int r = wm0 + ta * 32 + p * 4 + (lane >> 4);
                    old[p] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (r < m_dim && gcol < n_dim) old[p] = *reinterpret_cast<const float4 *>(out + (size_t)r * n_dim + gcol);
                }
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    val[p].x += old[p].x; val[p].y += old[p].y; val[p].z += old[p].z; val[p].w += old[p].w;
                }
            }
            typedef float f32x4_t __attribute__((ext_vector_type(4)));
            auto store = [&](auto streaming) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const int r = wm0 + ta * 32 + p * 4 + (lane >> 4);
                    const f32x4_t v = {val[p].x, val[p].y, val[p].z, val[p].w};
                    f32x4_t *to = reinterpret_cast<f32x4_t *>(out + (size_t)r * n_dim + gcol);
                    if (r < m_dim && gcol < n_dim) {
                        if (decltype(streaming)::value) __builtin_nontemporal_store(v, to);
                        else *to = v;
                    }
                }
            };
            if (stream) store(std::true_type{});
            else store(std::false_type{});
            wave_lds_fence();
        }
}

// The same for the eight-wave tiles.  When adding, a block's old values are requested one block ahead: with one
// workgroup per unit nobody else covers the round trip, and the registers are free.  (Four small workgroups
// per unit lose a fourth of their waves to the registers and 17 % of their time.)
template <class KL, int NA, int BA, int NWV>
__device__ __forceinline__ void wgrad_epilogue_ahead(typename KL::Acc &acc, char *lds, float *out0, float *out1, size_t base,
                                               int m0, int n0, int m_dim, int n_dim, bool add, bool stream, int wave, int lane)
{
    static_assert(KL::TB % 2 == 0, "a wave owns a multiple of 64 columns");
    constexpr int BLOCKS = (KL::TB / 2) * NA * KL::TA;        // 32 x 64 blocks of the wave: columns, operands, tiles
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    float *buf = reinterpret_cast<float *>(lds + wave * 8192);
    const int wm0 = m0 + (wave / (NWV / 2)) * (BA / 2), wn0 = n0 + (wave % (NWV / 2)) * (KL::TB * 32);
    const int col4 = lane & 15, row4 = lane >> 4;
    auto tensor = [&](int i) __attribute__((always_inline)) { return ((i / KL::TA) % NA == 0 ? out0 : out1) + base; };
    auto row_of = [&](int i, int p) __attribute__((always_inline)) { return wm0 + (i % KL::TA) * 32 + p * 4 + row4; };
    auto col_of = [&](int i) __attribute__((always_inline)) { return wn0 + i / (NA * KL::TA) * 64 + col4 * 4; };
    f32x4_t old[2][8];
    auto request = [&](int i, f32x4_t (&o)[8]) __attribute__((always_inline)) {      // clamped: what lies outside is not stored
#pragma unroll
        for (int p = 0; p < 8; ++p)
            o[p] = *reinterpret_cast<const f32x4_t *>(tensor(i) + (size_t)min(row_of(i, p), m_dim - 1) * n_dim + min(col_of(i), n_dim - 4));
    };
    if (add) request(0, old[0]);
    __syncthreads();                                          // every wave is done with the operand slabs
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) {
        const int half = i / (NA * KL::TA), a = (i / KL::TA) % NA, ta = i % KL::TA;
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                buf[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 64 + tb * 32 + (lane & 31)] = acc[a][ta][half * 2 + tb][v];
        if (add && i + 1 < BLOCKS) request(i + 1, old[(i + 1) % 2]);
        wave_lds_fence();
        f32x4_t val[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) val[p] = *reinterpret_cast<const f32x4_t *>(buf + (p * 4 + row4) * 64 + col4 * 4);
        if (add) {
#pragma unroll
            for (int p = 0; p < 8; ++p) val[p] += old[i % 2][p];
        }
        auto store = [&](auto streaming) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int r = row_of(i, p), c = col_of(i);
                f32x4_t *to = reinterpret_cast<f32x4_t *>(tensor(i) + (size_t)r * n_dim + c);
                if (r < m_dim && c < n_dim) {
                    if (decltype(streaming)::value) __builtin_nontemporal_store(val[p], to);
                    else *to = val[p];
                }
            }
        };
        if (stream) store(std::true_type{});
        else store(std::false_type{});
        wave_lds_fence();
    }
}

// Weight gradients: out[slot][m][n] (+)= sum over the group's rows of L[row][m] * R[row][n].
// NA = 2 computes two left operands against one right operand (dGt and dU against X).
// Tile: (NA x BA) x WN with BA = WGM / NA.  Three geometries: 256 x 256 (eight waves, see wgrad_tiles_wide);
// for outputs narrower than that WGM = 256 (three slabs, two
// workgroups per compute unit) for long groups, where the MFMA rate matters; and WGM = 128 (two
// slabs, four workgroups per compute unit) for short groups, where the kernel is a stream of
// fp32 read-add-writes and more waves in flight mean more HBM bandwidth.  DEEP, for calls of few
// tiles: a unit has one or two workgroups at most, so nothing but a workgroup's own ring hides the
// latency of its slabs.  24 groups of 130 rows, 256 x 192: both calls 27.6 -> 24.8 us (of which 9 are launches).
template <int WGM, bool DEEP, int WN = WGN> struct WgradCfg {
    static constexpr int NWV = WN == 256 ? 8 : NWAVES;
    static constexpr int STAGES = DEEP || WN == 256 ? 4 : WGM == 256 ? NSTAGES : 2;
    static constexpr int OCC = WN == 256 ? 1 : DEEP || WGM == 256 ? 2 : 4;          // waves per SIMD aimed at
    static constexpr int SLABS = STAGES * (WGM + WN) * BK * 2;
    static constexpr int LDS = SLABS > NWV * 8192 ? SLABS : NWV * 8192;
};
template <int NA, int WGM, bool DEEP, int WN = WGN>
__device__ __forceinline__ void wgrad_tile(const Sched &s, const bf16_t *__restrict__ L0, const bf16_t *__restrict__ L1,
                                           const bf16_t *__restrict__ R, int m_dim, int n_dim, int E, int accumulate, int stream,
                                           int total, float *__restrict__ out0, float *__restrict__ out1, int block, char *lds)
{
    constexpr int BA = WGM / NA;
    using CF = WgradCfg<WGM, DEEP, WN>;
    using KL = KLoop<KsTile<BA>, KsTile<WN>, NA, 1, BA, WN, 2, CF::NWV / 2, 1, true, CF::STAGES, (kSpreadLoads && CF::STAGES >= 3)>;
    const int n_nt = (n_dim + WN - 1) / WN, n_mt = (m_dim + BA - 1) / BA;
    const int per_group = n_nt * n_mt;
    const int per_xcd = (total + 7) >> 3;
    const int logical = (block & 7) * per_xcd + (block >> 3);
    if (logical >= total) return;
    const int gi = logical / per_group, rem = logical % per_group;
    const int e = s.grp_expert[gi];
    if (e < 0) return;
    const int slot = s.grp_slot[gi];
    const bool add = accumulate && slot < E;
    const int row0 = s.grp_row0[gi], rows = s.grp_rows[gi];
    if (rows == 0 && add) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int mt, nt;
    band_order(rem, n_mt, n_nt, mt, nt);
    const int m0 = mt * BA, n0 = nt * WN;
    Operand A[1][NA], B[1][1];
    A[0][0] = {L0 + (size_t)row0 * m_dim, m_dim, m0, m_dim - 1};
    if (NA == 2) A[0][NA - 1] = {L1 + (size_t)row0 * m_dim, m_dim, m0, m_dim - 1};
    B[0][0] = {R + (size_t)row0 * n_dim, n_dim, n0, n_dim - 1};
    typename KL::Acc acc;
    KL::zero(acc);
    KL::run(acc, A, B, (rows + BK - 1) / BK, rows, lds, tid);
    const size_t at = (size_t)slot * m_dim * n_dim;
    if constexpr (WN == 256) wgrad_epilogue_ahead<KL, NA, BA, CF::NWV>(acc, lds, out0, out1, at, m0, n0, m_dim, n_dim, add, stream != 0, wave, lane);
    else wgrad_epilogue<KL, NA, BA>(acc, lds, out0, out1, at, m0, n0, m_dim, n_dim, add, stream != 0, wave, lane);
}
template <int NA, int WGM, int WN = WGN>
__global__ void __launch_bounds__((WgradCfg<WGM, false, WN>::NWV * 64), (WgradCfg<WGM, false, WN>::OCC))
wgrad_kernel(Sched s, const bf16_t *__restrict__ L0, const bf16_t *__restrict__ L1,
             const bf16_t *__restrict__ R, int m_dim, int n_dim, int E, int accumulate, int stream, int total,
             float *__restrict__ out0, float *__restrict__ out1)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    wgrad_tile<NA, WGM, false, WN>(s, L0, L1, R, m_dim, n_dim, E, accumulate, stream, total, out0, out1, blockIdx.x, lds);
}
// dWd and dWg, dWu in one launch, for calls of few tiles: neither fills the chip, and both take the time of
// one tile, which they then spend side by side.  Blocks 0 .. blocks_gu - 1 do dWg, dWu.  24 groups of 130 rows,
// 256 x 192: 24.5 -> 13 us a call with the launches; 8 experts, 1024 rows, 128 x 256, batched: 39 -> 22.
template <int WGM>
__global__ void __launch_bounds__(THREADS, (WgradCfg<WGM, true>::OCC))
wgrad_pair_kernel(Sched s, const bf16_t *__restrict__ dY, const bf16_t *__restrict__ A, const bf16_t *__restrict__ X, int h, int hff, int E,
                  int accumulate, int stream, int total_down, int total_gu, int blocks_gu,
                  float *__restrict__ dWg, float *__restrict__ dWu, float *__restrict__ dWd)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    if ((int)blockIdx.x < blocks_gu) wgrad_tile<2, WGM, true>(s, s.dGt, s.dU, X, hff, h, E, accumulate, stream, total_gu, dWg, dWu, blockIdx.x, lds);
    else wgrad_tile<1, WGM, true>(s, dY, nullptr, A, h, hff, E, accumulate, stream, total_down, dWd, nullptr, blockIdx.x - blocks_gu, lds);
}

// ---------------------------------------------------------------- batched weight gradients
// One pass over every micro-batch of a training batch: the tile of expert e contracts over all
// rows e received, instance by instance, micro-batch by micro-batch, in registers, and writes
// dW once.  Per-micro-batch device pointers travel as a kernel argument of the ordering kernel,
// which turns them into one record per piece for the GEMM kernels.
constexpr int kMaxWgradMb = RELIBRA_MAX_WGRAD_MB;
constexpr int kWgradChunk = 64;
struct MbTable {
    const bf16_t *dY[kMaxWgradMb], *X[kMaxWgradMb], *A[kMaxWgradMb], *dGt[kMaxWgradMb], *dU[kMaxWgradMb];
    const int32_t *iptr[kMaxWgradMb], *igrp[kMaxWgradMb], *goff[kMaxWgradMb];
    const int32_t *rtok[kMaxWgradMb];      // null: X holds group-ordered rows; else X holds tokens and row r is X[rtok[r]]
    int tok_last[kMaxWgradMb];
    unsigned long long dy_tokens;          // bit mb set: dY[mb] is the token tensor dOut and row r is dOut[rtok[r]]
};

// Instance range of expert e in micro-batch mb, sanitised: [p0, p1) inside the instance table.
__device__ __forceinline__ bool inst_range(const MbTable &tb, int mb, int e, int inst_cap, int &p0, int &p1)
{
    p0 = tb.iptr[mb][e];
    p1 = tb.iptr[mb][e + 1];
    if (p0 < 0 || p1 < p0 || p1 > inst_cap) { p0 = p1 = 0; return false; }
    return true;
}
// Row range of instance p of micro-batch mb, sanitised: rows = 0 when a table entry is bad.
__device__ __forceinline__ bool inst_rows(const MbTable &tb, int mb, int p, int G, int n_rows, int &row0, int &rows)
{
    row0 = rows = 0;
    const int g = tb.igrp[mb][p];
    if (g < 0 || g >= G) return false;
    const int lo = tb.goff[mb][g], hi = tb.goff[mb][g + 1];
    if (lo < 0 || hi < lo || hi > n_rows) return false;
    row0 = lo;
    rows = hi - lo;
    return true;
}

// Workspace of the batched weight gradients.
struct WgradPlan {
    int32_t *exp_rows;     // [E] rows of the expert over the whole batch
    int32_t *exp_slabs;    // [E] k-loop slabs: sum over its pieces of ceil(rows / BK)
    int32_t *exp_order;    // [E] experts in descending order of rows (ties: lower id)
    int32_t *piece_ptr;    // [E+1] CSR over experts into the piece arrays
    int32_t *piece_mb, *piece_row0, *piece_rows;   // [S] micro-batch, first row, rows (> 0) of a piece
    // [S] what a tile's k-loop needs of a piece, as one record each (one wide scalar load per switch
    // of piece instead of a chain of single ones): operand addresses at the piece's first row, the
    // row table (0: none), rows, last token.  64-byte aligned.
    int32_t *rec_down, *rec_gu;
};
constexpr int kRecDownInts = 8, kRecGuInts = 16;
struct PieceRecDown { unsigned long long L, R, gather; int32_t rows, tok_last; };
struct PieceRecGu { unsigned long long L0, L1, R, gather; int32_t rows, tok_last; int32_t pad[6]; };
static_assert(sizeof(PieceRecDown) == kRecDownInts * 4 && sizeof(PieceRecGu) == kRecGuInts * 4, "record sizes");
inline size_t wgrad_plan_ints(int E, int G)
{
    const size_t S = (size_t)kMaxWgradMb * ((size_t)E + G);
    return 4 * (size_t)E + 1 + 3 * S + 16 + (kRecDownInts + kRecGuInts) * S;
}
inline WgradPlan carve_wgrad(void *ws, int E, int G)
{
    WgradPlan w;
    int32_t *p = (int32_t *)ws;
    const size_t S = (size_t)kMaxWgradMb * ((size_t)E + G);
    w.exp_rows = p; p += E;
    w.exp_slabs = p; p += E;
    w.exp_order = p; p += E;
    w.piece_ptr = p; p += E + 1;
    w.piece_mb = p; p += S;
    w.piece_row0 = p; p += S;
    w.piece_rows = p; p += S;
    p += (16 - ((p - (int32_t *)ws) & 15)) & 15;             // records: 64-byte aligned (the workspace is 256-byte aligned)
    w.rec_down = p; p += kRecDownInts * S;
    w.rec_gu = p;
    return w;
}

// One block.  Lists, per expert, the pieces of its contraction: every instance with rows, micro-
// batch by micro-batch in the order of the plan's instance table (entries out of range are left
// out and flagged), and ranks the experts by rows so that the tiles run heaviest first.
__global__ void __launch_bounds__(256)
wgrad_order_kernel(MbTable tb, int n_mb, int G, int inst_cap, int n_rows, int E, int h, int hff, WgradPlan w, int32_t *err_flag)
{
    extern __shared__ int32_t rows_of[];       // [E]
    __shared__ int32_t sums[4];
    const int tid = threadIdx.x;
    bool bad = false;
    int carry = 0;                             // pieces so far, the same in every thread
    if (tid == 0) w.piece_ptr[0] = 0;
    // The piece arrays hold S entries: enough for every instance of every micro-batch of a well-formed
    // (monotone) instance table.  A corrupted table whose ranges overlap could list more; pieces
    // beyond S are left out (and flagged), so that nothing is written past the arrays.
    const int S = kMaxWgradMb * (E + G);
    for (int base = 0; base < E; base += 256) {
        const int e = base + tid;
        int pieces = 0;
        if (e < E) {
            for (int mb = 0; mb < n_mb; ++mb) {
                int p0, p1;
                if (!inst_range(tb, mb, e, inst_cap, p0, p1)) bad = true;
                for (int p = p0; p < p1; ++p) {
                    int row0, rows;
                    if (!inst_rows(tb, mb, p, G, n_rows, row0, rows)) bad = true;
                    if (rows > 0) ++pieces;
                }
            }
        }
        pieces = min(pieces, S + 1);                 // saturate: the sums below stay inside an int
        int all;
        const int upto = block_scan256(pieces, sums, all);
        if (e < E) {
            int at = min(carry + upto - pieces, S);
            const int end = min(carry + upto, S);
            if (carry + upto > S) bad = true;
            w.piece_ptr[e + 1] = end;
            long long total = 0, slabs = 0;
            for (int mb = 0; mb < n_mb && at < end; ++mb) {
                int p0, p1;
                inst_range(tb, mb, e, inst_cap, p0, p1);
                for (int p = p0; p < p1 && at < end; ++p) {
                    int row0, rows;
                    inst_rows(tb, mb, p, G, n_rows, row0, rows);
                    if (rows > 0) {
                        total += rows;
                        slabs += (rows + BK - 1) / BK;
                        w.piece_mb[at] = mb; w.piece_row0[at] = row0; w.piece_rows[at] = rows;
                        const bool dy_tok = (tb.dy_tokens >> mb) & 1, x_tok = tb.rtok[mb] != nullptr;
                        const unsigned long long table = (unsigned long long)(uintptr_t)(tb.rtok[mb] + row0);
                        PieceRecDown d;     // dWd: L = dY rows (or dOut tokens through the table), R = A rows
                        d.L = (unsigned long long)(uintptr_t)(dy_tok ? tb.dY[mb] : tb.dY[mb] + (size_t)row0 * h);
                        d.R = (unsigned long long)(uintptr_t)(tb.A[mb] + (size_t)row0 * hff);
                        d.gather = dy_tok ? table : 0ull;
                        d.rows = rows;
                        d.tok_last = tb.tok_last[mb];
                        ((PieceRecDown *)w.rec_down)[at] = d;
                        PieceRecGu u;       // dWg, dWu: L = dGt, dU rows; R = X rows (or tokens through the table)
                        u.L0 = (unsigned long long)(uintptr_t)(tb.dGt[mb] + (size_t)row0 * hff);
                        u.L1 = (unsigned long long)(uintptr_t)(tb.dU[mb] + (size_t)row0 * hff);
                        u.R = (unsigned long long)(uintptr_t)(x_tok ? tb.X[mb] : tb.X[mb] + (size_t)row0 * h);
                        u.gather = x_tok ? table : 0ull;
                        u.rows = rows;
                        u.tok_last = tb.tok_last[mb];
                        for (int z = 0; z < 6; ++z) u.pad[z] = 0;
                        ((PieceRecGu *)w.rec_gu)[at] = u;
                        ++at;
                    }
                }
            }
            rows_of[e] = (int32_t)(total > 0x7fffffffLL ? 0x7fffffffLL : total);
            w.exp_rows[e] = rows_of[e];
            w.exp_slabs[e] = (int32_t)(slabs > 0x7fffffffLL ? 0x7fffffffLL : slabs);
        }
        carry = min(carry + all, S + 1);
    }
    if (bad) atomicOr(err_flag, RELIBRA_ERR_GROUP_TABLE);
    __syncthreads();
    for (int e = tid; e < E; e += 256) {
        const int mine = rows_of[e];
        int rank = 0;
        for (int o = 0; o < E; ++o) rank += (rows_of[o] > mine || (rows_of[o] == mine && o < e)) ? 1 : 0;
        w.exp_order[rank] = e;
    }
}

// The pieces of one expert's contraction as the k-loop sees them: one record per piece, written
// by the ordering kernel (an earlier launch, the same for every lane: read as scalars).
template <int NA>
struct WgradPieces {
    const_i32_ptr rows;                    // this expert's slice of the piece rows
    const_i32_ptr recs;                    // and of the records
    int m_dim, n_dim, m0, n0;
    __device__ __forceinline__ int valid(int i) const { return rows[i]; }
    __device__ __forceinline__ void piece(int i, Operand (&A)[1][NA], Operand (&B)[1][1], int &k_valid) const
    {
        constexpr int RI = NA == 1 ? kRecDownInts : kRecGuInts;
        typedef int32_t rec_vec __attribute__((ext_vector_type(RI)));
        typedef const __attribute__((address_space(4))) rec_vec *rec_ptr;
        const rec_vec r = *(rec_ptr)(recs + (size_t)i * RI);
        auto ptr = [&](int at) { return (const bf16_t *)(uintptr_t)(((unsigned long long)(uint32_t)r[at + 1] << 32) | (uint32_t)r[at]); };
        if (NA == 1) {
            const int32_t *table = (const int32_t *)ptr(4);
            k_valid = r[6];
            A[0][0] = {ptr(0), m_dim, m0, m_dim - 1, table, r[7]};
            B[0][0] = {ptr(2), n_dim, n0, n_dim - 1};
        } else {
            const int32_t *table = (const int32_t *)ptr(6);
            k_valid = r[8];
            A[0][0] = {ptr(0), m_dim, m0, m_dim - 1};
            A[0][NA - 1] = {ptr(2), m_dim, m0, m_dim - 1};
            B[0][0] = {ptr(4), n_dim, n0, n_dim - 1, table, r[9]};
        }
    }
};

// NA = 1: dWd.  NA = 2: dWg, dWu.  WN: columns of a tile.  128: four waves, three slabs, two
// workgroups per compute unit.  256: eight waves of 128 x 64 each, one workgroup per compute unit,
// four slabs: two thirds of the operand bytes (and load instructions) per flop, the same two
// waves per SIMD.  (Four waves of 128 x 128 on that tile, one per SIMD, were 5-10 % slower.)
constexpr int kWideWaves = 8;
template <int WN> struct WgradWide {
    static constexpr int STAGES = WN == 256 ? 4 : NSTAGES;
    static constexpr int OCC = WN == 256 ? 1 : 2;
    static constexpr int SLABS = STAGES * (256 + WN) * BK * 2;
    static constexpr int LDS = SLABS > 8 * 8192 ? SLABS : 8 * 8192;
};
template <int NA, int WN, int NWV>
__device__ __forceinline__ void wgrad_batched_tile(int E, int m_dim, int n_dim, const WgradPlan &w, int accumulate, int stream,
                                                   float *__restrict__ out0, float *__restrict__ out1, int block, char *lds)
{
    constexpr int WGM = 256, BA = WGM / NA;
    // NA = 1: the A side (dY) may be gathered; its loads go last in the window (see KLoop)
    // the operand that may come through a row table: dY of dWd (A side), X of dWg, dWu (B side)
    using KL = KLoop<KsTile<BA, BK, NA == 1>, KsTile<WN, BK, NA == 2>, NA, 1, BA, WN, 2, NWV / 2, 1, true, WgradWide<WN>::STAGES, kSpreadLoads, NA == 1>;
    const int n_nt = (n_dim + WN - 1) / WN, n_mt = (m_dim + BA - 1) / BA;
    const int per_expert = n_nt * n_mt;
    // Tile list: experts in descending order of rows, each expert's tiles in band order, cut into
    // chunks of kWgradChunk tiles (an 8 x 8 patch sharing operand tiles).  The chunks are dealt to
    // the XCDs back and forth (0..7, 7..0, ...), so every L2 gets near-equal work, heaviest first.
    const int x = block & 7, t = block >> 3;
    const int q = t / kWgradChunk;
    const long long tile = ((long long)q * 8 + ((q & 1) ? 7 - x : x)) * kWgradChunk + t % kWgradChunk;
    if (tile >= (long long)E * per_expert) return;
    const int e = w.exp_order[tile / per_expert];
    if ((unsigned)e >= (unsigned)E) return;
    const bool add = accumulate != 0;
    if (w.exp_rows[e] == 0 && add) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int mt, nt;
    band_order((int)(tile % per_expert), n_mt, n_nt, mt, nt);
    const int m0 = mt * BA, n0 = nt * WN;
    typename KL::Acc acc;
    KL::zero(acc);
    const int s0 = w.piece_ptr[e];
    const WgradPieces<NA> src{(const_i32_ptr)(uintptr_t)(w.piece_rows + s0),
                              (const_i32_ptr)(uintptr_t)((NA == 1 ? w.rec_down + (size_t)s0 * kRecDownInts : w.rec_gu + (size_t)s0 * kRecGuInts)),
                              m_dim, n_dim, m0, n0};
    KL::run_pieces(acc, src, w.piece_ptr[e + 1] - s0, w.exp_slabs[e], lds, tid);
    const size_t at = (size_t)e * m_dim * n_dim;
    if constexpr (WN == 256) wgrad_epilogue_ahead<KL, NA, BA, NWV>(acc, lds, out0, out1, at, m0, n0, m_dim, n_dim, add, stream != 0, wave, lane);
    else wgrad_epilogue<KL, NA, BA>(acc, lds, out0, out1, at, m0, n0, m_dim, n_dim, add, stream != 0, wave, lane);
}
template <int NA, int WN, int NWV = NWAVES>
__global__ void __launch_bounds__(NWV * 64, WgradWide<WN>::OCC)
wgrad_batched_kernel(int E, int m_dim, int n_dim, WgradPlan w, int accumulate, int stream,
                     float *__restrict__ out0, float *__restrict__ out1)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    wgrad_batched_tile<NA, WN, NWV>(E, m_dim, n_dim, w, accumulate, stream, out0, out1, blockIdx.x, lds);
}
// Both in one launch, for calls of few tiles, as wgrad_pair_kernel.
template <int WN, int NWV = NWAVES>
__global__ void __launch_bounds__(NWV * 64, WgradWide<WN>::OCC)
wgrad_batched_pair_kernel(int E, int h, int hff, WgradPlan w, int accumulate, int stream, int blocks_gu,
                          float *__restrict__ dWg, float *__restrict__ dWu, float *__restrict__ dWd)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    if ((int)blockIdx.x < blocks_gu) wgrad_batched_tile<2, WN, NWV>(E, hff, h, w, accumulate, stream, dWg, dWu, blockIdx.x, lds);
    else wgrad_batched_tile<1, WN, NWV>(E, h, hff, w, accumulate, stream, dWd, nullptr, blockIdx.x - blocks_gu, lds);
}

// Replica gradients return to the home copy (Section 5.1).  A thread owns element positions
// and walks the live replica slots in ascending slot order, so the sum has a fixed order.
// blockIdx.y selects the tensor (all three have h * h' elements per expert).
__global__ void __launch_bounds__(256)
replica_sum_kernel(Sched s, size_t per_expert_vec4, float4 *__restrict__ dWg, float4 *__restrict__ dWu,
                   float4 *__restrict__ dWd)
{
    const int n_pairs = s.hdr[1];
    float4 *__restrict__ dW = blockIdx.y == 0 ? dWg : blockIdx.y == 1 ? dWu : dWd;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < per_expert_vec4; i += (size_t)gridDim.x * 256)
        for (int p = 0; p < n_pairs; ++p) {
            const float4 src = dW[(size_t)s.pair_slot[p] * per_expert_vec4 + i];
            float4 *dst = &dW[(size_t)s.pair_expert[p] * per_expert_vec4 + i];
            float4 d = *dst;
            d.x += src.x; d.y += src.y; d.z += src.z; d.w += src.w;
            *dst = d;
        }
}

struct FfnArgs {
    int n_rows, G, g_begin, g_end, E, h, hff;
};

inline int check_ffn_args(const FfnArgs &a)
{
    if (a.n_rows < 0 || a.G < 1 || a.g_begin < 0 || a.g_end > a.G || a.g_begin > a.g_end || a.E < 1) return RELIBRA_EINVAL;
    if (a.g_end - a.g_begin > kMaxSchedGroups) return RELIBRA_EUNSUPPORTED;   // the schedule kernel keeps a prefix per group in LDS
    if (a.h < 64 || a.hff < 64 || a.h % 64 || a.hff % 64) return RELIBRA_EUNSUPPORTED;
    if ((size_t)a.n_rows * (size_t)(a.h > a.hff ? a.h : a.hff) > ((size_t)1 << 40)) return RELIBRA_EUNSUPPORTED;
    return RELIBRA_OK;
}

}  // namespace relibra

using namespace relibra;

extern "C" size_t relibra_workspace_bytes(int which, int T, int k, int E, int G, int h, int hff)
{
    if (T < 0 || k < 1 || E < 1 || G < 1 || (size_t)T * k > 0x7fffffffull) return 0;
    const int N = T * k;
    switch (which) {
    case RELIBRA_WS_PERMUTE: return round256((size_t)((N + RELIBRA_PERM_UNIT - 1) / RELIBRA_PERM_UNIT + 4) * E * sizeof(int32_t));
    case RELIBRA_WS_FFN_FWD: return ffn_ws_bytes(N, G, hff, false);
    case RELIBRA_WS_FFN_BWD: return ffn_ws_bytes(N, G, hff, true);
    case RELIBRA_WS_WGRAD_BATCHED: return round256(wgrad_plan_ints(E, G) * sizeof(int32_t));
    case RELIBRA_WS_DGATE: return dgate_scratch_bytes(N, hff);
    default: return 0;
    }
    (void)h;
}

// Kernels use more than 64 KiB of dynamic LDS: raise the per-kernel limit (an attribute of the
// loaded kernel, not of a call) once per process, whichever thread calls first.
static int set_lds_limits()
{
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_gate_up_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_gate_up_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_down_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_down_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<false, false, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<true, false, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<false, true, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_act_kernel<true, true, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_dx_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_dx_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_gate_up_kernel<false, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_gate_up_kernel<true, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_down_kernel<false, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)fwd_down_kernel<true, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_dx_kernel<false, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)bwd_dx_kernel<true, 512>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesWide));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<1, 256, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<256, false, 256>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<1, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<256, false>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<2, 256, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<256, false, 256>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<2, 256>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<256, false>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_kernel<1, 128>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<128>::LDS));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_kernel<2, 128>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<128>::LDS));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_kernel<1, 256, kWideWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<256>::LDS));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_kernel<2, 256, kWideWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<256>::LDS));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<1, 128>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<128, false>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_pair_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<128, true>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_kernel<2, 128>, hipFuncAttributeMaxDynamicSharedMemorySize, (WgradCfg<128, false>::LDS)));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_pair_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<128>::LDS));
    RELIBRA_HIP_TRY(hipFuncSetAttribute((const void *)wgrad_batched_pair_kernel<256, kWideWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, WgradWide<256>::LDS));
    return RELIBRA_OK;
}
static int ensure_lds_limits()
{
    static std::once_flag once;
    static int status = RELIBRA_OK;
    std::call_once(once, [] { status = set_lds_limits(); });
    return status;
}

static inline unsigned grid8(long long tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

// The wide column tiles are taken where they pad the output's columns no further than the narrow ones do
// (half of all widths), and where there are more narrow tiles than the compute units can take one each:
// fewer tiles leave units idle that tiles of half the width would use.  Row tiles are estimated: half a
// tile per group for its tail.  Wide / narrow over 2 to 32 groups of 64 to 700 rows, 640 to 4096 columns, mean of the
// four kernels (smallest and largest): estimates of 200 to 255 narrow tiles 1.20 (0.95, 1.61), 256 1.21 (0.97, 1.41),
// 257 to 287 0.91 (0.75, 1.36), 320 to 359 0.99 (0.61, 1.29: the large ones are groups of whole tiles, which the
// estimate overstates), 360 to 449 0.91.  Measured, narrow -> wide, us: 64 groups, 4032 x 1472 (pads alike), 100 rows each:
// gate/up 394 -> 324, down 186 -> 174, dA 200 -> 176, dX 329 -> 311; 1200 rows each: 2146 -> 1723, 1076 -> 948,
// 1056 -> 980, 1820 -> 1694.  3136 columns (8 % more padding): down 521 -> 534.  8 groups of 512 x 1024, 200
// rows each (few tiles): gate/up 17 -> 22, down 19 -> 26, dA 20 -> 28, dX 27 -> 42; 8 of 4096 x 14336, dX at 32
// rows 416 -> 608, at 200 rows 536 -> 676, at 300 rows (384 narrow tiles) 918 -> 684.
// A width that the 512-column tiles do not divide takes them only where their last round is nearly full (at most 15 %
// idle): the narrow ones then waste less in the last round than the wide ones save.  Wide / narrow for 1408 and 1472
// columns over contractions of 640 to 2048, idle 33 and 28 % (32 groups of 450 rows, 16 of 1000): dA 1.09 to 1.18, down
// 1.00 to 1.12, dX 1.00 to 1.17; idle 4 % (128 groups of 100 rows): 0.92 to 1.12, 0.95 to 1.00, 0.91 to 1.01.  (Gate/up, 256
// columns of each: 0.81 to 1.02 either way.)
// Short contractions (k_dim, over both products where there are two) stay narrow too: two workgroups per unit
// then hide each other's start and epilogue, which weigh more than the loads the wide tile saves.  16 groups of
// 800 rows, 4096 columns, narrow -> wide: down over 64 28 -> 32 us, 128 38 -> 48, 256 59 -> 65, 512 82 -> 92; 64
// groups of 300 rows, 1536 columns: dA over 128 63 -> 73, 512 92 -> 106; gate/up over 128 53 -> 60, over 512 117
// and 121 (its two projections have twice the work per value).  dX over 2 x 512: 115 -> 105.
constexpr int kComputeUnits = 256;
constexpr int kShortDot = 512;
static inline bool row_tiles_wide(int n_dim, int width, int n_rows, int groups, int k_dim)
{
    if (k_dim <= kShortDot) return false;
    const long long wide = (n_dim + width - 1) / width, narrow = (n_dim + width / 2 - 1) / (width / 2);
    const long long row_tiles = std::max((long long)groups, (long long)n_rows / BM + groups / 2);
    const long long tiles = row_tiles * wide, slots = (tiles + kComputeUnits - 1) / kComputeUnits * kComputeUnits;
    const bool full = n_dim % width == 0 || width < 512 || 100 * slots <= 115 * tiles;
    return n_dim >= width && 2 * wide == narrow && row_tiles * narrow > kComputeUnits && full;
}

static int launch_sched(const SchedIn &in, const Sched &s, hipStream_t stream)
{
    RELIBRA_LAUNCH(RELIBRA_K_SCHED, stream, sched_kernel<<<1, 256, (size_t)(in.Gr + 1) * sizeof(int32_t), stream>>>(in, s));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}
// Whether the first kernel of a call works the schedule out itself: where all of its blocks run at once, two to a
// compute unit, each does so beside the others, however many groups it reads; beyond that it is done once per round and
// soon costs more than the launch it saves.  `tiles` is what a row buffer of this size could hold (the groups are
// known on the device only): a call over a few groups of a large buffer counts as a large one.  With the scheduling
// kernel -> without, us a call, repeated in a captured graph, spread 1 to 6 %: 24 tiles (8 groups of 64 rows, 128 x
// 256) forward 12.9 -> 11.6, data gradients 17.7 -> 16.3; 384 (32 of 128, 256 x 768) 31.6 -> 29.3, 40.7 -> 38.5; 281 (250 of 16, 256 x 128)
// 14.4 -> 12.8, 18.0 -> 16.3; 495 (440 of 16, 256 x 128) 19.7 -> 17.1, 24.6 -> 21.9; all of 16 forward and 22 backward sizes of up to 504 gain.
// Beyond: 1566 (440 of 100, 256 x 256) 52.6 -> 50.5, 2248 (500 of 16, 256 x 512) 57.7 -> 62.2, 2250 (1000 of 16, 256 x 256) 57.0 ->
// 65.6.  Whole training steps: 8 experts of 128 x 256, 512 tokens (two calls) 111.5 -> 106.5, spread 7 %; 16 of 256 x 192, 3 x 777
// tokens (six calls) 262 -> 251, spread 4 %.
static inline bool schedules_itself(bool wide, long long tiles) { return !wide && tiles + 8 <= 2 * kComputeUnits; }

// Launch of a row-tiled GEMM kernel template <bool WT, int AW>: narrow (four waves, two workgroups
// per compute unit) or wide (eight waves, one) column tiles.
#define RELIBRA_ROW_LAUNCH(kid, kern, wt_, wide_, AWN, AWW, tiles, ...)                                                      \
    do {                                                                                                                      \
        if (wide_) {                                                                                                          \
            if (wt_) RELIBRA_LAUNCH(kid, stream, (kern<true, AWW><<<grid8(tiles), kWideRowWaves * 64, kLdsBytesWide, stream>>>(__VA_ARGS__)));  \
            else RELIBRA_LAUNCH(kid, stream, (kern<false, AWW><<<grid8(tiles), kWideRowWaves * 64, kLdsBytesWide, stream>>>(__VA_ARGS__)));    \
        } else {                                                                                                              \
            if (wt_) RELIBRA_LAUNCH(kid, stream, (kern<true, AWN><<<grid8(tiles), THREADS, kLdsBytes, stream>>>(__VA_ARGS__)));   \
            else RELIBRA_LAUNCH(kid, stream, (kern<false, AWN><<<grid8(tiles), THREADS, kLdsBytes, stream>>>(__VA_ARGS__)));     \
        }                                                                                                                     \
    } while (0)


// Xrows: the group-ordered rows, or (row_tok != nullptr) the token tensor [T, h] they are gathered from.
static int ffn_fwd_impl(const void *Xrows, const int32_t *row_tok, int T, int n_rows,
                                   const int32_t *group_offset, const int32_t *group_expert,
                                   int G, int g_begin, int g_end, int E,
                                   const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                   void *Gt_save, void *U_save, void *A_save, void *Yrows, int flags,
                                   void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_,
                                   const float *row_gate = nullptr, void *Ag_save = nullptr)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (flags & ~RELIBRA_FWD_TRANSPOSED_WEIGHTS) return RELIBRA_EINVAL;
    if ((row_gate == nullptr) != (Ag_save == nullptr) || !aligned16(Ag_save)) return RELIBRA_EINVAL;   // Ag_save == A_save: gated in place
    const bool wt = (flags & RELIBRA_FWD_TRANSPOSED_WEIGHTS) != 0;
    const FfnArgs a{n_rows, G, g_begin, g_end, E, h, hff};
    if (int rc = check_ffn_args(a)) return rc;
    const int Gr = g_end - g_begin;
    if (Gr == 0 || n_rows == 0) return RELIBRA_OK;
    if (!Xrows || !group_offset || !group_expert || !Wg || !Wu || !Wd || !Gt_save || !U_save || !A_save ||
        !Yrows || !ws || !err_flag)
        return RELIBRA_EINVAL;
    if (!aligned16(Xrows) || !aligned16(Wg) || !aligned16(Wu) || !aligned16(Wd) || !aligned16(A_save) ||
        !aligned16(Gt_save) || !aligned16(U_save) || !aligned16(Yrows) || !aligned16(ws))
        return RELIBRA_EINVAL;
    if (ws_bytes < ffn_ws_bytes(n_rows, Gr, hff, false)) return RELIBRA_EWORKSPACE;
    if (int rc = ensure_lds_limits()) return rc;
    Sched s = carve(ws, n_rows, Gr, hff, false);
    const long long R = max_row_tiles(n_rows, Gr);
    const bool wide1 = row_tiles_wide(hff, 256, n_rows, Gr, 2 * h), wide2 = row_tiles_wide(h, 512, n_rows, Gr, hff);
    const int ct1 = wide1 ? (hff + 255) / 256 : (hff + 127) / 128, ct2 = wide2 ? (h + 511) / 512 : (h + 255) / 256;
    SchedIn in{group_offset, group_expert, nullptr, g_begin, Gr, n_rows, E, 0, (int)R, err_flag};
    const bool inside = schedules_itself(wide1, R * ct1);
    if (!inside) {
        if (int rc = launch_sched(in, s, stream)) return rc;
        in.group_offset = nullptr;
    }
    RELIBRA_ROW_LAUNCH(RELIBRA_K_FWD_GATE_UP, fwd_gate_up_kernel, wt, wide1, 128, 256, R * ct1 + (inside ? 8 : 0),
                       s, (const bf16_t *)Xrows, row_tok, T - 1, (const bf16_t *)Wg, (const bf16_t *)Wu, h, hff, ct1,
                       (bf16_t *)Gt_save, (bf16_t *)U_save, (bf16_t *)A_save, row_gate, (bf16_t *)Ag_save, in);
    RELIBRA_HIP_TRY(launch_check());
    RELIBRA_ROW_LAUNCH(RELIBRA_K_FWD_DOWN, fwd_down_kernel, wt, wide2, 256, 512, R * ct2,
                       s, (const bf16_t *)A_save, (const bf16_t *)Wd, h, hff, ct2, (bf16_t *)Yrows);
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" int relibra_moe_ffn_fwd(const void *Xrows, int n_rows,
                                   const int32_t *group_offset, const int32_t *group_expert,
                                   int G, int g_begin, int g_end, int E,
                                   const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                   void *Gt_save, void *U_save, void *A_save, void *Yrows, int flags,
                                   void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_)
{
    return ffn_fwd_impl(Xrows, nullptr, 1, n_rows, group_offset, group_expert, G, g_begin, g_end, E, Wg, Wu, Wd, h, hff,
                        Gt_save, U_save, A_save, Yrows, flags, ws, ws_bytes, err_flag, stream_);
}

extern "C" int relibra_moe_ffn_fwd_gather(const void *X, int T, const int32_t *row_tok, int n_rows,
                                          const int32_t *group_offset, const int32_t *group_expert,
                                          int G, int g_begin, int g_end, int E,
                                          const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                          void *Gt_save, void *U_save, void *A_save, void *Yrows, int flags,
                                          void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_)
{
    if (T < 1 || !row_tok) return RELIBRA_EINVAL;
    return ffn_fwd_impl(X, row_tok, T, n_rows, group_offset, group_expert, G, g_begin, g_end, E, Wg, Wu, Wd, h, hff,
                        Gt_save, U_save, A_save, Yrows, flags, ws, ws_bytes, err_flag, stream_);
}

extern "C" int relibra_moe_ffn_fwd_gated(const void *X, int T, const int32_t *row_tok, const float *row_gate, int n_rows,
                                         const int32_t *group_offset, const int32_t *group_expert,
                                         int G, int g_begin, int g_end, int E,
                                         const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                         void *Gt_save, void *U_save, void *A_save, void *Ag_save, void *Yrows, int flags,
                                         void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_)
{
    if (T < 1 || !row_tok || !row_gate || !Ag_save) return RELIBRA_EINVAL;
    return ffn_fwd_impl(X, row_tok, T, n_rows, group_offset, group_expert, G, g_begin, g_end, E, Wg, Wu, Wd, h, hff,
                        Gt_save, U_save, A_save, Yrows, flags, ws, ws_bytes, err_flag, stream_, row_gate, Ag_save);
}

// Per-micro-batch weight gradients in 256 x 256 tiles of eight waves: half the operand bytes per flop and 1 KiB of
// a row per store, but one workgroup per compute unit, whose start, reads of old gradients and stores nobody covers, and
// whose last round is as long as the others.  `padded`: the tiles with both launches' last rounds filled up; `small`: the
// same work in 128 x 128 tiles, four to a unit (in tiles of 256 x 256).  Small tiles (from 512 rows on: 256 x 128)
// -> these, kernel times, by rows per group:
//   written       padded/small   128   192   256   384   512   1024  2048      added         512   1024  1536  2048
//   64 x 4096 x 1536      1.0   1.04  0.93  0.88  0.87  0.88                                1.11
//   8 x 4096 x 4096       1.0   1.03  1.06  1.01  0.93  0.85  0.82  0.88                    1.05  1.03  0.95  0.95
//   128 x 2048 x 768      1.0   0.93  0.85  0.85  0.88  0.93  0.89                          1.04  1.01  0.96
//   20 x 2880 x 2880      1.11  1.05  0.96  0.93  0.90  0.90  0.90                          1.03  1.00  0.98
//   18 x 1024 x 2048      1.19  0.96  0.92  0.91  0.93  0.96  0.93  0.93                    1.10  1.06  1.03  0.98
//   40 x 896 x 1152       1.35  1.06  1.03  1.03  1.04  1.06  1.03  1.03                    1.11  1.08  1.08  1.04
//   16 x 640 x 1536       1.78  1.22  1.22  1.21  1.24  1.15  1.06  1.01                    1.16  1.11  1.05  1.04
// So from 192 rows per group on where gradients are written and at most a fifth is padding, and from 1536 on where they
// are added to and next to nothing is.
static inline bool wgrad_tiles_wide(int n_rows, int groups, int h, int hff, bool add)
{
    const auto cut = [](long long n, long long by) { return (n + by - 1) / by; };
    const long long down = groups * cut(h, 256) * cut(hff, 256), gate_up = groups * cut(hff, 128) * cut(h, 256);
    const long long padded = (cut(down, kComputeUnits) + cut(gate_up, kComputeUnits)) * kComputeUnits;
    const long long small4 = groups * (cut(h, 128) * cut(hff, 128) + cut(hff, 64) * cut(h, 128));     // four times `small`
    return h >= 256 && hff >= 256 && down >= kComputeUnits && (long long)n_rows >= (add ? 1536LL : 192LL) * groups &&
           100 * 4 * padded <= (add ? 105 : 120) * small4;
}

// Whether the gradient tensors (fp32, `values` in each) are larger than the 256 MB last-level cache together.
static inline int streams_dw(size_t values) { return 3 * values * sizeof(float) > ((size_t)256 << 20) ? 1 : 0; }

// Gate-fused form of the backward call: the upstream gradient comes from the token tensor.
struct GatedBwd {
    const void *dOut;
    int T;
    const int32_t *row_tok;
    const float *row_gate;
    const int32_t *src_of;   // optional
    float *dgate;
    void *scratch;
    size_t scratch_bytes;
};

static int ffn_bwd_impl(const void *dYrows, const void *Xrows,
                                   const void *Gt_save, const void *U_save, const void *A_save, int n_rows,
                                   const int32_t *group_offset, const int32_t *group_expert,
                                   const int32_t *group_dw_slot,
                                   int G, int g_begin, int g_end, int E, int n_dw_slots,
                                   const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                   void *dXrows, float *dWg, float *dWu, float *dWd, int flags,
                                   void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_,
                                   const GatedBwd *gb)
{
    hipStream_t stream = (hipStream_t)stream_;
    const FfnArgs a{n_rows, G, g_begin, g_end, E, h, hff};
    if (int rc = check_ffn_args(a)) return rc;
    if (n_dw_slots < E) return RELIBRA_EINVAL;
    if (gb) {
        if (!(flags & RELIBRA_BWD_DEFER_WGRAD) || gb->T < 1 || !gb->dOut || !gb->row_tok || !gb->row_gate || !gb->dgate ||
            !gb->scratch || !aligned16(gb->dOut) || !aligned16(gb->scratch))
            return RELIBRA_EINVAL;
        if (gb->scratch_bytes < dgate_scratch_bytes(n_rows, hff)) return RELIBRA_EWORKSPACE;
        dYrows = gb->dOut;                       // the argument checks below see the tensor the kernels read
    }
    const int Gr = g_end - g_begin;
    if (Gr == 0) return RELIBRA_OK;
    const bool defer = (flags & RELIBRA_BWD_DEFER_WGRAD) != 0;    // then dW is not touched and may be null
    // Xrows is an operand of the weight gradients only
    if (!dYrows || !Gt_save || !U_save || !A_save || !group_offset || !group_expert || !group_dw_slot ||
        !Wg || !Wu || !Wd || !dXrows || !ws || !err_flag || (!defer && (!Xrows || !dWg || !dWu || !dWd)))
        return RELIBRA_EINVAL;
    if (!aligned16(dYrows) || !aligned16(Xrows) || !aligned16(A_save) || !aligned16(Gt_save) || !aligned16(U_save) ||
        !aligned16(Wg) || !aligned16(Wu) || !aligned16(Wd) || !aligned16(dXrows) || !aligned16(dWg) ||
        !aligned16(dWu) || !aligned16(dWd) || !aligned16(ws))
        return RELIBRA_EINVAL;
    if (ws_bytes < ffn_ws_bytes(n_rows, Gr, hff, true)) return RELIBRA_EWORKSPACE;
    if (int rc = ensure_lds_limits()) return rc;
    Sched s = carve(ws, n_rows, Gr, hff, true);
    // the slot table matters only to kernels that write dW or read replica parameters
    const int32_t *slot_table = (defer && !(flags & RELIBRA_BWD_REPLICA_WEIGHTS)) ? nullptr : group_dw_slot;
    const long long R = max_row_tiles(n_rows, Gr);
    const bool wide_h = row_tiles_wide(h, 512, n_rows, Gr, 2 * hff);
    // (the activation backward on transposed weight copies keeps whole tiles: its partial gate sums belong to columns)
    const bool wide_ff = row_tiles_wide(hff, 512, n_rows, Gr, h) && (hff % 512 == 0 || !(flags & RELIBRA_BWD_TRANSPOSED_WEIGHTS));
    const int ct_ff = wide_ff ? (hff + 511) / 512 : (hff + 255) / 256, ct_h = wide_h ? (h + 511) / 512 : (h + 255) / 256;
    SchedIn in{group_offset, group_expert, slot_table, g_begin, Gr, n_rows, E, n_dw_slots, (int)R, err_flag};
    const bool inside = n_rows > 0 && schedules_itself(wide_ff, R * ct_ff);
    if (!inside) {
        if (int rc = launch_sched(in, s, stream)) return rc;
        in.group_offset = nullptr;
    }
    const long long act_blocks = R * ct_ff + (inside ? 8 : 0);
    const int accumulate = (flags & RELIBRA_BWD_ACCUMULATE) ? 1 : 0;
    const int w_from_slot = (flags & RELIBRA_BWD_REPLICA_WEIGHTS) ? 1 : 0;
    if (n_rows > 0) {
        const bf16_t *wd = (const bf16_t *)Wd, *wg = (const bf16_t *)Wg, *wu = (const bf16_t *)Wu;
        const bf16_t *dy = (const bf16_t *)dYrows, *gt = (const bf16_t *)Gt_save, *us = (const bf16_t *)U_save;
        const bool wt = (flags & RELIBRA_BWD_TRANSPOSED_WEIGHTS) != 0;
        GateFusion gf;
        gf.n_rows = n_rows;
        if (gb) {
            gf.row_tok = gb->row_tok;
            gf.tok_last = gb->T - 1;
            gf.row_gate = gb->row_gate;
            gf.dgate_part = (float *)gb->scratch;
        }
#define RELIBRA_BWD_ACT(WT_, GATED_)                                                                                              \
    do {                                                                                                                          \
        if (wide_ff) RELIBRA_LAUNCH(RELIBRA_K_BWD_ACT, stream, (bwd_act_kernel<WT_, GATED_, 512><<<grid8(act_blocks), kWideRowWaves * 64, kLdsBytesWide, stream>>>( \
            s, dy, wd, gt, us, h, hff, ct_ff, w_from_slot, gf, in)));                                                                 \
        else RELIBRA_LAUNCH(RELIBRA_K_BWD_ACT, stream, (bwd_act_kernel<WT_, GATED_, 256><<<grid8(act_blocks), THREADS, kLdsBytes, stream>>>(         \
            s, dy, wd, gt, us, h, hff, ct_ff, w_from_slot, gf, in)));                                                                 \
    } while (0)
        if (wt) { if (gb) RELIBRA_BWD_ACT(true, true); else RELIBRA_BWD_ACT(true, false); }
        else { if (gb) RELIBRA_BWD_ACT(false, true); else RELIBRA_BWD_ACT(false, false); }
#undef RELIBRA_BWD_ACT
        RELIBRA_HIP_TRY(launch_check());
        if (wt) RELIBRA_ROW_LAUNCH(RELIBRA_K_BWD_DX, bwd_dx_kernel, true, wide_h, 256, 512, R * ct_h,
                                   s, wg, wu, h, hff, ct_h, w_from_slot, (bf16_t *)dXrows);
        else RELIBRA_ROW_LAUNCH(RELIBRA_K_BWD_DX, bwd_dx_kernel, false, wide_h, 256, 512, R * ct_h,
                                s, wg, wu, h, hff, ct_h, w_from_slot, (bf16_t *)dXrows);
        RELIBRA_HIP_TRY(launch_check());
        if (gb) {
            RELIBRA_LAUNCH(RELIBRA_K_DGATE_REDUCE, stream, dgate_reduce_kernel<<<std::min(1024, (n_rows + 255) / 256), 256, 0, stream>>>(
                (const float *)gb->scratch, kDgateParts * ((hff + 255) / 256), n_rows, group_offset, g_begin, g_end, gb->src_of, gb->dgate, err_flag));
            RELIBRA_HIP_TRY(launch_check());
        }
    }
    if (defer) return RELIBRA_OK;                                  // dGt, dU stay in the workspace
    // short groups (few rows per group on average): the small, high-occupancy geometry
    const bool wide_tiles = wgrad_tiles_wide(n_rows, Gr, h, hff, accumulate != 0);
    const bool small_tiles = !wide_tiles && (long long)n_rows < 512LL * Gr;
    const int wgm = small_tiles ? 128 : 256, wgn = wide_tiles ? 256 : WGN;
    const long long t_down = (long long)Gr * ((h + wgm - 1) / wgm) * ((hff + wgn - 1) / wgn);              // dWd: m in h, n in h'
    const long long t_gu = (long long)Gr * ((hff + wgm / 2 - 1) / (wgm / 2)) * ((h + wgn - 1) / wgn);      // dWg, dWu: m in h', n in h
    const int stream_dw = streams_dw((size_t)n_dw_slots * h * hff);
#define RELIBRA_WGRAD(WGM_, WN_)                                                                                                           \
    do {                                                                                                                                   \
        using CF = WgradCfg<WGM_, false, WN_>;                                                                                             \
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_DOWN, stream, (wgrad_kernel<1, WGM_, WN_><<<grid8(t_down), CF::NWV * 64, CF::LDS, stream>>>(        \
            s, (const bf16_t *)dYrows, nullptr, (const bf16_t *)A_save, h, hff, E, accumulate, stream_dw, (int)t_down, dWd, nullptr)));    \
        RELIBRA_HIP_TRY(launch_check());                                                                                                   \
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_GATE_UP, stream, (wgrad_kernel<2, WGM_, WN_><<<grid8(t_gu), CF::NWV * 64, CF::LDS, stream>>>(       \
            s, s.dGt, s.dU, (const bf16_t *)Xrows, hff, h, E, accumulate, stream_dw, (int)t_gu, dWg, dWu)));                               \
        RELIBRA_HIP_TRY(launch_check());                                                                                                   \
    } while (0)
    if (wide_tiles) {
        RELIBRA_WGRAD(256, 256);
    } else if (!small_tiles) {
        RELIBRA_WGRAD(256, 128);
    } else if (std::max(t_down, t_gu) <= 2 * kComputeUnits) {
        const unsigned blocks_gu = grid8(t_gu);
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_PAIR, stream, (wgrad_pair_kernel<128><<<blocks_gu + grid8(t_down), THREADS, (WgradCfg<128, true>::LDS), stream>>>(
            s, (const bf16_t *)dYrows, (const bf16_t *)A_save, (const bf16_t *)Xrows, h, hff, E, accumulate, stream_dw, (int)t_down, (int)t_gu,
            (int)blocks_gu, dWg, dWu, dWd)));
        RELIBRA_HIP_TRY(launch_check());
    } else {
        RELIBRA_WGRAD(128, 128);
    }
#undef RELIBRA_WGRAD
    if (!(flags & RELIBRA_BWD_NO_REPLICA_SUM) && n_dw_slots > E) {
        const size_t vec4 = (size_t)h * hff / 4;
        const int grid = (int)((vec4 + 255) / 256 < 4096 ? (vec4 + 255) / 256 : 4096);
        RELIBRA_LAUNCH(RELIBRA_K_REPLICA_SUM, stream, replica_sum_kernel<<<dim3(grid, 3), 256, 0, stream>>>(
            s, vec4, (float4 *)dWg, (float4 *)dWu, (float4 *)dWd));
        RELIBRA_HIP_TRY(launch_check());
    }
    return RELIBRA_OK;
}

extern "C" int relibra_moe_ffn_bwd(const void *dYrows, const void *Xrows,
                                   const void *Gt_save, const void *U_save, const void *A_save, int n_rows,
                                   const int32_t *group_offset, const int32_t *group_expert,
                                   const int32_t *group_dw_slot,
                                   int G, int g_begin, int g_end, int E, int n_dw_slots,
                                   const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                   void *dXrows, float *dWg, float *dWu, float *dWd, int flags,
                                   void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_)
{
    return ffn_bwd_impl(dYrows, Xrows, Gt_save, U_save, A_save, n_rows, group_offset, group_expert, group_dw_slot, G, g_begin,
                        g_end, E, n_dw_slots, Wg, Wu, Wd, h, hff, dXrows, dWg, dWu, dWd, flags, ws, ws_bytes, err_flag, stream_,
                        nullptr);
}

extern "C" int relibra_moe_ffn_bwd_gated(const void *dOut, int T, const int32_t *row_tok, const float *row_gate,
                                         const int32_t *src_of,
                                         const void *Gt_save, const void *U_save, int n_rows,
                                         const int32_t *group_offset, const int32_t *group_expert,
                                         const int32_t *group_dw_slot,
                                         int G, int g_begin, int g_end, int E, int n_dw_slots,
                                         const void *Wg, const void *Wu, const void *Wd, int h, int hff,
                                         void *dXrows, float *dgate, int flags,
                                         void *ws, size_t ws_bytes, void *dgate_scratch, size_t dgate_scratch_bytes_,
                                         int32_t *err_flag, relibra_stream stream_)
{
    if (flags & ~(RELIBRA_BWD_REPLICA_WEIGHTS | RELIBRA_BWD_TRANSPOSED_WEIGHTS | RELIBRA_BWD_DEFER_WGRAD)) return RELIBRA_EINVAL;
    const GatedBwd gb{dOut, T, row_tok, row_gate, src_of, dgate, dgate_scratch, dgate_scratch_bytes_};
    // the saved activations are an operand of the weight gradients only: Gt stands in for the pointer check
    return ffn_bwd_impl(nullptr, nullptr, Gt_save, U_save, Gt_save, n_rows, group_offset, group_expert, group_dw_slot, G, g_begin,
                        g_end, E, n_dw_slots, Wg, Wu, Wd, h, hff, dXrows, nullptr, nullptr, nullptr,
                        flags | RELIBRA_BWD_DEFER_WGRAD, ws, ws_bytes, err_flag, stream_, &gb);
}

extern "C" int relibra_moe_ffn_wgrad_batched(const relibra_wgrad_mb *mbs, int n_mb, int n_rows,
                                             int G, int inst_cap, int E, int h, int hff,
                                             float *dWg, float *dWu, float *dWd, int flags,
                                             void *ws, size_t ws_bytes, int32_t *err_flag, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (flags & ~(RELIBRA_WGRAD_ACCUMULATE | RELIBRA_WGRAD_TILE_NARROW | RELIBRA_WGRAD_TILE_WIDE)) return RELIBRA_EINVAL;
    if ((flags & RELIBRA_WGRAD_TILE_NARROW) && (flags & RELIBRA_WGRAD_TILE_WIDE)) return RELIBRA_EINVAL;
    const int accumulate = (flags & RELIBRA_WGRAD_ACCUMULATE) ? 1 : 0;
    const FfnArgs a{n_rows, G, 0, G, E, h, hff};
    if (int rc = check_ffn_args(a)) return rc;
    if (!mbs || n_mb < 1 || n_mb > kMaxWgradMb || inst_cap < 1 || E > 4096) return RELIBRA_EINVAL;
    if (!dWg || !dWu || !dWd || !ws || !err_flag || !aligned16(dWg) || !aligned16(dWu) || !aligned16(dWd) || !aligned16(ws))
        return RELIBRA_EINVAL;
    if (ws_bytes < relibra_workspace_bytes(RELIBRA_WS_WGRAD_BATCHED, 0, 1, E, G, h, hff)) return RELIBRA_EWORKSPACE;
    MbTable tb;
    tb.dy_tokens = 0;
    for (int mb = 0; mb < kMaxWgradMb; ++mb) {
        const relibra_wgrad_mb &m = mbs[mb < n_mb ? mb : 0];
        if (mb < n_mb) {
            const bool gathered = m.Xrows_dev == nullptr;
            if (!m.dYrows_dev && (!m.dOut_dev || !gathered || !aligned16(m.dOut_dev))) return RELIBRA_EINVAL;
            if (!m.A_save_dev || !m.bwd_workspace_dev || !m.inst_ptr_dev || !m.inst_group_dev ||
                !m.group_offset_dev || (gathered && (!m.X_dev || !m.row_tok_dev || m.n_tokens < 1)))
                return RELIBRA_EINVAL;
            if (!aligned16(m.dYrows_dev) || !aligned16(gathered ? m.X_dev : m.Xrows_dev) || !aligned16(m.A_save_dev) ||
                !aligned16(m.bwd_workspace_dev))
                return RELIBRA_EINVAL;
        }
        const Sched s = carve(const_cast<void *>(m.bwd_workspace_dev), n_rows, G, hff, true);
        tb.dY[mb] = (const bf16_t *)(m.dYrows_dev ? m.dYrows_dev : m.dOut_dev);
        if (!m.dYrows_dev) tb.dy_tokens |= 1ull << mb;
        tb.X[mb] = (const bf16_t *)(m.Xrows_dev ? m.Xrows_dev : m.X_dev);
        tb.rtok[mb] = m.Xrows_dev ? nullptr : m.row_tok_dev;
        tb.tok_last[mb] = m.Xrows_dev ? 0 : m.n_tokens - 1;
        tb.A[mb] = (const bf16_t *)m.A_save_dev;
        tb.dGt[mb] = s.dGt;
        tb.dU[mb] = s.dU;
        tb.iptr[mb] = m.inst_ptr_dev;
        tb.igrp[mb] = m.inst_group_dev;
        tb.goff[mb] = m.group_offset_dev;
    }
    if (int rc = ensure_lds_limits()) return rc;
    if (inst_cap > E + G) return RELIBRA_EINVAL;               // an instance is a group: at most G of them
    const WgradPlan w = carve_wgrad(ws, E, G);
    RELIBRA_LAUNCH(RELIBRA_K_WGRAD_ORDER, stream, wgrad_order_kernel<<<1, 256, E * sizeof(int32_t), stream>>>(
        tb, n_mb, G, inst_cap, n_rows, E, h, hff, w, err_flag));
    RELIBRA_HIP_TRY(launch_check());
    auto grid_of = [&](long long tiles_per_expert) {          // blocks: 8 XCDs x chunks per XCD x tiles per chunk
        const long long chunks = ((long long)E * tiles_per_expert + kWgradChunk - 1) / kWgradChunk;
        return (unsigned)(8 * ((chunks + 7) / 8) * kWgradChunk);
    };
    // Tile width.  The 256-column tile moves two thirds of the operand bytes per flop and is the
    // default wherever the output is at least that wide (measured on every workload shape: 3-10 %
    // faster), with one exception: dWd with a narrow h' and a short contraction, where its three
    // tile columns lose to the narrow tile's six (h' = 768, 8 k rows per expert: 3.76 against 3.62 ms).
    const bool long_k = (long long)n_rows * n_mb >= (long long)16384 * E;
    const bool forced = (flags & (RELIBRA_WGRAD_TILE_NARROW | RELIBRA_WGRAD_TILE_WIDE)) != 0;
    const bool want_wide = (flags & RELIBRA_WGRAD_TILE_WIDE) != 0;
    const bool wide_down = forced ? want_wide : (hff >= 1024 || (long_k && hff >= 256));
    const bool wide_gu = forced ? want_wide : h >= 256;
    const int wn_down = wide_down ? 256 : 128, wn_gu = wide_gu ? 256 : 128;
    const unsigned g_down = grid_of((long long)((h + 255) / 256) * ((hff + wn_down - 1) / wn_down));  // dWd: m in h, n in h'
    const unsigned g_gu = grid_of((long long)((hff + 127) / 128) * ((h + wn_gu - 1) / wn_gu));        // dWg, dWu: m in h', n in h
    const int stream_dw = streams_dw((size_t)E * h * hff);
    const long long tiles = (long long)E * ((h + 255) / 256 * ((hff + wn_down - 1) / wn_down) + (hff + 127) / 128 * ((h + wn_gu - 1) / wn_gu));
    if (wide_down == wide_gu && tiles <= kComputeUnits) {
        if (wide_gu) RELIBRA_LAUNCH(RELIBRA_K_WGRAD_PAIR, stream, (wgrad_batched_pair_kernel<256, kWideWaves><<<g_gu + g_down, kWideWaves * 64, WgradWide<256>::LDS, stream>>>(
            E, h, hff, w, accumulate, stream_dw, (int)g_gu, dWg, dWu, dWd)));
        else RELIBRA_LAUNCH(RELIBRA_K_WGRAD_PAIR, stream, (wgrad_batched_pair_kernel<128><<<g_gu + g_down, THREADS, WgradWide<128>::LDS, stream>>>(
            E, h, hff, w, accumulate, stream_dw, (int)g_gu, dWg, dWu, dWd)));
        RELIBRA_HIP_TRY(launch_check());
        return RELIBRA_OK;
    }
    if (wide_down) {
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_DOWN, stream, (wgrad_batched_kernel<1, 256, kWideWaves><<<g_down, kWideWaves * 64, WgradWide<256>::LDS, stream>>>(
            E, h, hff, w, accumulate, stream_dw, dWd, nullptr)));
    } else {
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_DOWN, stream, wgrad_batched_kernel<1, 128><<<g_down, THREADS, WgradWide<128>::LDS, stream>>>(
            E, h, hff, w, accumulate, stream_dw, dWd, nullptr));
    }
    RELIBRA_HIP_TRY(launch_check());
    if (wide_gu) {
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_GATE_UP, stream, (wgrad_batched_kernel<2, 256, kWideWaves><<<g_gu, kWideWaves * 64, WgradWide<256>::LDS, stream>>>(
            E, hff, h, w, accumulate, stream_dw, dWg, dWu)));
    } else {
        RELIBRA_LAUNCH(RELIBRA_K_WGRAD_GATE_UP, stream, wgrad_batched_kernel<2, 128><<<g_gu, THREADS, WgradWide<128>::LDS, stream>>>(
            E, hff, h, w, accumulate, stream_dw, dWg, dWu));
    }
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" int relibra_transpose_experts(const void *in_dev, int n_blocks, int rows, int cols, void *out_dev,
                                         relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (n_blocks < 0 || rows < 8 || cols < 8 || rows % 8 || cols % 8 || n_blocks > 65535) return RELIBRA_EINVAL;
    if (n_blocks == 0) return RELIBRA_OK;
    if (!in_dev || !out_dev || in_dev == out_dev || !aligned16(in_dev) || !aligned16(out_dev)) return RELIBRA_EINVAL;
    if ((rows + 63) / 64 > 65535) return RELIBRA_EUNSUPPORTED;
    const dim3 grid((cols + kTrTile - 1) / kTrTile, (rows + kTrTile - 1) / kTrTile, n_blocks);
    RELIBRA_LAUNCH(RELIBRA_K_TRANSPOSE, stream, transpose_experts_kernel<<<grid, 256, 0, stream>>>(
        (const bf16_t *)in_dev, rows, cols, (bf16_t *)out_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}
