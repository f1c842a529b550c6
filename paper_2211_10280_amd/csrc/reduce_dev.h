// The segmented reduction of the gradient calculation: duplicates of a row summed in sorted order (see grad.hip).  What
// its two forms have in common -- a row per wave (reduce.hip), several per wave (reduce_sub.hip): the window of entries
// that a wave works on, and the kernels that chain the partials of long rows.
#pragma once
#include "aux_dev.h"
#include "dev_common.h"
#include "group_dev.h"
#include "kernels.h"

#ifndef SEG_UNROLL
#define SEG_UNROLL 4
#endif
#ifndef SEG_RUNS
#define SEG_RUNS 1
#endif

// One wave per tile of up to 32 sorted entries.  A row (segment) of at most a tile's entries is
// "short": it is summed completely, in sorted order, by the wave whose tile contains its first
// entry, even where it runs into the next tile, and written once.  Longer rows are "long": every
// tile sums the part of the row that lies inside it into a partial (part[tile][0] for a row that
// began in an earlier tile, part[tile][1] for one that begins here), and k_segfixup chains the
// partials in tile order.  Work per wave is bounded by two tiles whatever the skew of the ids.
struct SegWindow {
    int tile, t0, avail, tile_len;   // the tile, its first entry, entries in the window (two tiles), in the tile
    int tile_size;
    int seg_l;                       // lane l: row and value of entry t0 + l
    u32 val_l;
    int first_start;                 // first entry of the row that entry t0 belongs to
    u64 heads;                       // bit l: entry t0 + l opens a row
    bool at_end;                     // the window reaches the end of the list
    // entries this wave sums: from the first row it owns (or its share of a long row that
    // began earlier) to the end of the last row that begins in the tile (or the tile end if long)
    int e_begin, e_end;
    int dest;                        // of the row at e_begin: 0 out_rows, 1 part[tile][0], 2 part[tile][1]
    int last_dest;                   // of the row at e_end - 1

    // end (relative) of the row whose first entry in the window is at e, or -1 if it runs past the window
    __device__ __forceinline__ int row_end(int e) const
    {
        const u64 later = (e + 1 < 64) ? (heads >> (e + 1)) : 0ull;
        if (later) return e + 1 + (int)__builtin_ctzll(later);
        return at_end ? avail : -1;
    }
    __device__ __forceinline__ int row_dest(int e) const   // of a row that begins at e
    {
        const int end = row_end(e);
        return ((end < 0) || (end - e) > tile_size) ? 2 : 0;
    }
    // rows and values of the window; false: no such tile
    __device__ __forceinline__ bool load(const SegReduceArgs &a, int tile_)
    {
        static_assert(2 * TN_SEG_MAX_TILE <= WAVE, "a wave keeps the metadata of two tiles in its lanes");
        tile = tile_;
        tile_size = 1 << a.shift;
        t0 = tile << a.shift;
        if (t0 >= a.n) return false;
        tile_len = min(a.n, t0 + tile_size) - t0;
        avail = min(2 * tile_size, a.n - t0);
        const int lane = lane_id();
        seg_l = -1;
        val_l = 0;
        if (lane < avail) {
            seg_l = a.seg_of[t0 + lane];
            val_l = a.vals[t0 + lane];
        }
        return true;
    }
    // false: nothing to sum
    __device__ __forceinline__ bool split(const SegReduceArgs &a)
    {
        const int lane = lane_id();
        const int seg_up = __shfl_up(seg_l, 1, WAVE);
        const int first_row = rd_lane(seg_l, 0);
        first_start = a.seg_start[first_row];
        heads = __ballot((lane < avail) && (lane == 0 ? (first_start == t0) : (seg_l != seg_up)));
        at_end = (t0 + avail == a.n);
        e_begin = dest = last_dest = 0;
        const int fe = row_end(0);
        const bool lead_long = (fe < 0) || (t0 + fe - first_start) > tile_size;
        if (first_start < t0) {
            if (lead_long) dest = 1;
            else e_begin = fe;                          // short row owned by an earlier tile
        } else {
            dest = lead_long ? 2 : 0;
        }
        const u64 in_tile = heads & ((tile_len < 64) ? ((1ull << tile_len) - 1ull) : ~0ull);
        if (in_tile) {
            const int h_last = 63 - (int)__builtin_clzll(in_tile);
            last_dest = row_dest(h_last);
            e_end = last_dest ? tile_len : row_end(h_last);
        } else {
            last_dest = 1;
            e_end = (first_start < t0 && lead_long) ? tile_len : e_begin;
        }
        // first tile of a block of tiles: tell k_segcross whether a long row crosses the block's border
        if (a.cross && (tile % TN_SEG_XBLOCK) == 0 && tile > 0 && lane == 0)
            a.xinfo[tile / TN_SEG_XBLOCK] = (first_start < t0 && dest == 1) ? 1 : 0;
        if (e_begin >= e_end) return false;
        if (e_begin > 0) dest = row_dest(e_begin);   // the first owned row begins at e_begin
        return true;
    }
};

// a long row begins in this tile: leave it, and where it ends, for the kernel that chains the partials
// (integer counter; the order of the list does not matter, every chain is independent)
__device__ __forceinline__ void seg_note_long(const SegReduceArgs &a, int tile, int row)
{
    if (lane_id() != 0) return;
    const int end = a.seg_start[row + 1], word = a.long_mask != nullptr ? a.row_ids[row] : 0;
    a.long_list[atomicAdd(a.long_cnt, 1)] = make_int4(tile, row, ((end - 1) >> a.shift) - tile, word);
    if (a.long_mask != nullptr) atomicOr((unsigned long long *)&a.long_mask[word >> 6], 1ull << (word & 63));
}

// ---------------------------------------------------------------- chains of partials
// (512-thread workgroups: 1024-thread ones wait for a whole compute unit's worth of free wave
// slots when another kernel fills the chip, which starved this kernel for hundreds of microseconds)
#define FIXUP_THREADS 512
#define FIXUP_WAVES (FIXUP_THREADS / WAVE)

// The sum of `n` rows of D floats, the j-th at src(j), in FIXUP_WAVES shares, several by each of the workgroup's WAVES waves,
// side by side where it has fewer: a share goes to its row of red; `first` (may be NULL) comes on top.  A row per wave (float4
// registers per lane: ITERS) ...
template <int ITERS>
struct WideChain {
    static constexpr int row = ITERS * WAVE * 4;
    template <int WAVES = FIXUP_WAVES, typename Src>
    static __device__ __forceinline__ void sum(int D, int n, const float *first, Src src, float (*red)[row])
    {
        constexpr int SHARES = FIXUP_WAVES / WAVES, UNROLL = SHARES * ITERS > 2 && SHARES > 1 ? SEG_UNROLL / 2 : SEG_UNROLL;
        const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id(), C4 = D >> 2;
        float4 acc[SHARES][ITERS];
#pragma unroll
        for (int h = 0; h < SHARES; ++h) zero_row<ITERS>(acc[h]);
        if (first && wave == 0) load_row<float, ITERS>(acc[0], first, C4, lane);
        for (int j0 = wave; j0 < n; j0 += FIXUP_WAVES * UNROLL) {
            float4 r[UNROLL][SHARES][ITERS];
#pragma unroll
            for (int x = 0; x < UNROLL; ++x)
#pragma unroll
                for (int h = 0; h < SHARES; ++h) {
                    const int j = j0 + x * FIXUP_WAVES + h * WAVES;
                    const float *p = src(j);
                    if (j < n) load_row<float, ITERS>(r[x][h], p, C4, lane);
                    else zero_row<ITERS>(r[x][h]);
                }
#pragma unroll
            for (int x = 0; x < UNROLL; ++x)
#pragma unroll
                for (int h = 0; h < SHARES; ++h) add_row<ITERS>(acc[h], r[x][h]);
        }
#pragma unroll
        for (int h = 0; h < SHARES; ++h)
#pragma unroll
            for (int it = 0; it < ITERS; ++it) *(float4 *)&red[wave + h * WAVES][(lane + WAVE * it) * 4] = acc[h][it];
    }
};
// ... or one per group of SUB lanes (rows of at most 4 * SUB elements)
template <int SUB>
struct GroupChain {
    static constexpr int row = SUB * 4;
    template <int WAVES = FIXUP_WAVES, typename Src>
    static __device__ __forceinline__ void sum(int D, int n, const float *first, Src src, float (*red)[row])
    {
        constexpr int RPW = WAVE / SUB, STEP = FIXUP_WAVES * RPW, SHARES = FIXUP_WAVES / WAVES;
        const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
        const int slot = lane / SUB, sl = lane % SUB, g = wave * RPW + slot;
        const bool in = sl < (D >> 2);
        float4 acc[SHARES];
#pragma unroll
        for (int h = 0; h < SHARES; ++h) acc[h] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (first && in && g == 0) acc[0] = ld4(first + 4 * sl);
        for (int j0 = g; j0 - slot < n; j0 += STEP * SEG_UNROLL) {
            float4 r[SEG_UNROLL][SHARES];
#pragma unroll
            for (int x = 0; x < SEG_UNROLL; ++x)
#pragma unroll
                for (int h = 0; h < SHARES; ++h) {
                    const int j = j0 + x * STEP + h * WAVES * RPW;
                    r[x][h] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (in && j < n) r[x][h] = ld4(src(j) + 4 * sl);
                }
#pragma unroll
            for (int x = 0; x < SEG_UNROLL; ++x)
#pragma unroll
                for (int h = 0; h < SHARES; ++h) axpy4(acc[h], 1.0f, r[x][h]);
        }
#pragma unroll
        for (int h = 0; h < SHARES; ++h) {
            acc[h] = sum_groups<SUB>(acc[h]);
            if (slot == 0) *(float4 *)&red[wave + h * WAVES][4 * sl] = acc[h];
        }
    }
};

// the waves' shares -> the row
template <typename Chain>
__device__ __forceinline__ void chain_store(float *dst, int D, float (*red)[Chain::row])
{
    __syncthreads();
    for (int e = threadIdx.x; e < D; e += FIXUP_THREADS) {
        float s = red[0][e];
#pragma unroll
        for (int w = 1; w < FIXUP_WAVES; ++w) s += red[w][e];
        dst[e] = s;
    }
}

// Chains the partials of a long row that the reduction listed, in tile order: the waves share the chain
// part[tile][1], part[tile+1][0], ...
template <typename Chain, int WAVES>
__device__ __forceinline__ void segfixup_row(const SegReduceArgs &a, int4 entry, float (*red)[Chain::row])
{
    const int tile = uniform(entry.x), len = uniform(entry.z);   // tiles after this one that hold a leading partial
    // the chain: leading partials of the tiles up to the next border of a tile block, then one
    // partial per tile block (k_segcross), the last of which ends where the row ends
    const int b1 = tile / TN_SEG_XBLOCK + 1;
    const int to_border = a.cross ? b1 * TN_SEG_XBLOCK - 1 - tile : len;   // no block partials: walk it all
    const int nd = len < to_border ? len : to_border;
    const int nc = (len > to_border) ? ((tile + len) / TN_SEG_XBLOCK - b1 + 1) : 0;
    // the j-th partial by selects (with a branch per partial the chain is longer: gradient of 6 000 centers, 100 words, 2 600 partials
    // of D = 300 in the longest row 147 us, by selects 138)
    const u32 near_step = 2 * (u32)a.D, far_step = (u32)a.D;
    const float *near = a.part + (size_t)(tile + 1) * near_step, *far = a.cross + (i64)(b1 - nd) * a.D;
    Chain::template sum<WAVES>(a.D, nd + nc, a.part + ((size_t)tile * 2 + 1) * a.D,
                               [=](int j) { return (j < nd ? near : far) + (size_t)(u32)j * (j < nd ? near_step : far_step); }, red);
}
// one workgroup per long row
template <typename Chain>
__device__ __forceinline__ void segfixup_rows(const SegReduceArgs &a, int first, int stride, float (*red)[Chain::row])
{
    int4 entry = a.long_list[first];        // there is one per tile, and no more workgroups: with the count, not after it
    const int count = *a.long_cnt;
    for (int i = first; i < count; i += stride) {
        if (i > first) entry = a.long_list[i];
        segfixup_row<Chain, FIXUP_WAVES>(a, entry, red);
        chain_store<Chain>(a.out_rows + (size_t)uniform(entry.y) * a.D, a.D, red);
        __syncthreads();
    }
}

// A long row's chain of partials can be very long (a hot word of a skewed stream takes a large share of
// all entries), and one workgroup walking it alone would bound the whole step.  The tiles are therefore
// grouped in blocks of TN_SEG_XBLOCK; at most one long row crosses the border at the start of a block,
// and this kernel sums that row's leading partials inside the block into cross[block], all blocks in
// parallel.  k_segfixup then adds one partial per block instead of one per tile.
template <typename Chain>
__device__ __forceinline__ void segcross_block(const SegReduceArgs &a, int b, float (*red)[Chain::row])
{
    const int t0 = b * TN_SEG_XBLOCK;
    const i64 e0 = (i64)t0 << a.shift;
    if (b < 1 || e0 >= a.n || a.xinfo[b] == 0) return;
    const int row = a.seg_of[e0];
    const int start = a.seg_start[row];
    const int end = a.seg_start[row + 1];
    if (start >= e0 || end - start <= (1 << a.shift)) return;   // no row crosses the border, or a short one (no partials)
    const int last_tile = (end - 1) >> a.shift;
    const int cnt = (last_tile < t0 + TN_SEG_XBLOCK - 1 ? last_tile : t0 + TN_SEG_XBLOCK - 1) - t0 + 1;
    Chain::sum(a.D, cnt, nullptr, [&](int j) { return a.part + (size_t)(t0 + j) * 2 * a.D; }, red);
    chain_store<Chain>(a.cross + (size_t)b * a.D, a.D, red);
}

template <typename Chain>
__global__ void __launch_bounds__(FIXUP_THREADS) k_segcross(SegReducePair p)
{
    __shared__ float red[FIXUP_WAVES][Chain::row];
    const int b = blockIdx.x;
    if (b < p.blocks_in) segcross_block<Chain>(p.in, b, red);
    else segcross_block<Chain>(p.out, b - p.blocks_in, red);
}

template <typename Chain>
__global__ void __launch_bounds__(FIXUP_THREADS) k_segfixup(SegReducePair p, PrepPhase rider)
{
    if ((int)blockIdx.x < rider.blocks) {
        prep_block<FIXUP_THREADS, false>(rider, (int)blockIdx.x, ride_lds);
        return;
    }
    float (*red)[Chain::row] = (float (*)[Chain::row])ride_lds;
    const int b = (int)blockIdx.x - rider.blocks, blocks = (int)gridDim.x - rider.blocks;
    if (b < p.blocks_in) segfixup_rows<Chain>(p.in, b, p.blocks_in, red);
    else segfixup_rows<Chain>(p.out, b - p.blocks_in, blocks - p.blocks_in, red);
}

// the launches of a reduction; reduce(workgroups of the two problems): its own
template <typename Chain, typename Reduce>
static void launch_segreduce_tiles(SegReducePair &p, const PrepPhase &rider, hipStream_t st, Reduce reduce)
{
    p.out.shift = tn_seg_shift(p.out.n, p.out.D);
    p.in.shift = tn_seg_shift(p.in.n, p.in.D);
    const int tiles_out = p.out.n > 0 ? (int)tn_seg_tiles(p.out.n, p.out.D) : 0;
    const int tiles_in = p.in.n > 0 ? (int)tn_seg_tiles(p.in.n, p.in.D) : 0;
    if (tiles_out <= TN_SEG_CROSS_MIN) p.out.cross = nullptr;
    if (tiles_in <= TN_SEG_CROSS_MIN) p.in.cross = nullptr;
    const int blocks_out = (tiles_out + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    p.blocks_in = (tiles_in + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    reduce(p.blocks_in + blocks_out);
    // Partials per block of tiles, for problems large enough that one row's chain could hold up the step:
    // up to TN_SEG_CROSS_MIN tiles even a row that takes every entry is walked by one workgroup in well
    // under a fifth of a millisecond, and the extra launch would cost every step several microseconds.
    const int xb_out = tiles_out > TN_SEG_CROSS_MIN ? (tiles_out + TN_SEG_XBLOCK - 1) / TN_SEG_XBLOCK : 0;
    const int xb_in = tiles_in > TN_SEG_CROSS_MIN ? (tiles_in + TN_SEG_XBLOCK - 1) / TN_SEG_XBLOCK : 0;
    if (xb_out + xb_in > 0) {
        p.blocks_in = xb_in;
        hipLaunchKernelGGL((k_segcross<Chain>), dim3(xb_in + xb_out), dim3(FIXUP_THREADS), 0, st, p);
    }
    const int fix_out = tn_seg_chains(p.out.n, p.out.D), fix_in = tn_seg_chains(p.in.n, p.in.D);
    if (fix_out + fix_in > 0 && p.out.long_mask == nullptr) {
        p.blocks_in = fix_in;
        const unsigned own = 4u * FIXUP_WAVES * Chain::row, riding = ride_lds_bytes<FIXUP_THREADS>(rider);
        hipLaunchKernelGGL((k_segfixup<Chain>), dim3(rider.blocks + fix_out + fix_in), dim3(FIXUP_THREADS),
                           own > riding ? own : riding, st, p, rider);
    }
}
