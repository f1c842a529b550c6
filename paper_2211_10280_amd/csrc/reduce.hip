// The segmented reduction of the gradient calculation: duplicates of a row summed in sorted order (see grad.hip).
#include <string.h>

#include "aux_dev.h"
#include "dev_common.h"
#include "kernels.h"
#include "rows_dev.h"

#ifndef SEG_UNROLL
#define SEG_UNROLL 4
#endif
#ifndef SEG_RUNS
#define SEG_RUNS 1
#endif

// rows in flight per wave in the segmented reduction
template <typename T, int NQ, bool TAIL>
struct SegShape {
    static constexpr int regs = (sizeof(T) == 2 ? 2 : 4) * NQ + (TAIL ? 1 : 0);
    static constexpr int unroll = regs <= 5 ? 2 * SEG_UNROLL : SEG_UNROLL;
};

// ---------------------------------------------------------------- segmented reduction
// Contribution of sorted entry e: scale * row, both fetched by the wave.
template <typename T, int MODE>
__device__ __forceinline__ void entry_source(const SegReduceArgs &a, u32 val, const T *&row,
                                             float &scale)
{
    if (MODE == 0) {
        int c = a.pair_center[val / (u32)a.Np1];
        row = (const T *)a.table + (size_t)c * a.stride;
        scale = a.g[val];
    } else {
        row = (const T *)a.center_part + (size_t)val * a.D;
        scale = 1.0f;
    }
}

// One wave per tile of TILE (<= 32) sorted entries.  A row (segment) of at most TILE entries is
// "short": it is summed completely, in sorted order, by the wave whose tile contains its first
// entry, even where it runs into the next tile, and written once.  Longer rows are "long": every
// tile sums the part of the row that lies inside it into a partial (part[tile][0] for a row that
// began in an earlier tile, part[tile][1] for one that begins here), and k_segfixup chains the
// partials in tile order.  Work per wave is bounded by 2*TILE entries whatever the skew of the ids.
template <typename T, int NQ, bool TAIL, int MODE, int TILE>
__device__ __forceinline__ void segreduce_tile(const SegReduceArgs &a, int block)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = SegShape<T, NQ, TAIL>::unroll;
    static_assert(2 * TILE <= WAVE, "a wave keeps the metadata of two tiles in its lanes");
    // the wave index is made explicitly wave-uniform so that all the control flow below is scalar
    const int tile = block * WAVES_PER_BLOCK + uniform((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    const int t0 = tile * TILE;
    if (t0 >= a.n) return;
    const int t1 = min(a.n, t0 + TILE);

    // lane l holds the metadata of entry t0 + l, for this tile and the next
    const int avail = min(2 * TILE, a.n - t0);
    int seg_l = -1;
    u32 val_l = 0;
    if (lane < avail) {
        seg_l = a.seg_of[t0 + lane];
        val_l = a.vals[t0 + lane];
    }
    const T *row_l = nullptr;
    float scale_l = 0.f;
    if (lane < avail) entry_source<T, MODE>(a, val_l, row_l, scale_l);

    // heads inside the two-tile window (bit l: entry t0+l opens a row); bit `avail` closes the list
    const int seg_up = __shfl_up(seg_l, 1, WAVE);
    const int first_row = rd_lane(seg_l, 0);
    const int first_start = a.seg_start[first_row];          // the only dependent load of the wave
    const bool head_l = (lane < avail) && (lane == 0 ? (first_start == t0) : (seg_l != seg_up));
    const u64 heads = __ballot(head_l);
    const bool at_end = (t0 + avail == a.n);                 // the window reaches the end of the list
    // end (relative) of the row whose first entry in the window is at e, or -1 if it runs past the window
    auto row_end = [&](int e) -> int {
        const u64 later = (e + 1 < 64) ? (heads >> (e + 1)) : 0ull;
        if (later) return e + 1 + (int)__builtin_ctzll(later);
        return at_end ? avail : -1;
    };
    const int tile_len = t1 - t0;
    // range of entries this wave sums: from the first row it owns (or its share of a long row that
    // began earlier) to the end of the last row that begins in the tile (or the tile end if long)
    int e_begin = 0, e_end;
    int dest = 0;                    // of the current row: 0 out_rows, 1 part[tile][0], 2 part[tile][1]
    {
        const int fe = row_end(0);
        const bool lead_long = (fe < 0) || (t0 + fe - first_start) > TILE;
        if (first_start < t0) {
            if (lead_long) dest = 1;
            else e_begin = fe;                          // short row owned by an earlier tile
        } else {
            dest = lead_long ? 2 : 0;
        }
        const u64 in_tile = heads & ((tile_len < 64) ? ((1ull << tile_len) - 1ull) : ~0ull);
        if (in_tile) {
            const int h_last = 63 - (int)__builtin_clzll(in_tile);
            const int end = row_end(h_last);
            const bool is_long = (end < 0) || (end - h_last) > TILE;
            e_end = is_long ? tile_len : end;
        } else {
            e_end = (first_start < t0 && lead_long) ? tile_len : e_begin;
        }
    }
    // first tile of a block of tiles: tell k_segcross whether a long row crosses the block's border
    if (a.cross && (tile % TN_SEG_XBLOCK) == 0 && tile > 0 && lane == 0)
        a.xinfo[tile / TN_SEG_XBLOCK] = (first_start < t0 && dest == 1) ? 1 : 0;
    if (e_begin >= e_end) return;
    Row acc;
    acc.zero();
    float *part = a.part + (size_t)tile * 2 * a.D;
    int cur = rd_lane(seg_l, e_begin);
    if (e_begin > 0) {   // the first owned row begins at e_begin
        const int end = row_end(e_begin);
        dest = ((end < 0) || (end - e_begin) > TILE) ? 2 : 0;
    }
    // a finished gradient row is next read by the table update, long after this kernel: it is written
    // around the caches (with ordinary stores the update ran 4 % slower, paying for the write-back of
    // these lines), while partials are read again at once
    auto flush = [&]() {
        if (dest == 0) acc.template store<true>(a.out_rows + (size_t)cur * a.D, a.D, lane);
        else acc.template store<false>(dest == 1 ? part : part + a.D, a.D, lane);
    };

    if constexpr (MODE == 0 && SEG_RUNS) {
        // Runs.  The occurrences of one center position follow one another in the sorted list of a row, and
        // where a word is frequent a position has many of them (the most frequent word of a steep distribution
        // is drawn as a negative dozens of times per position): consecutive entries of a row that take the same
        // center's row are one run, their scales are summed first (in a fixed order: a segmented scan across the
        // lanes) and the row is fetched and added once, scaled by the sum.
        const u64 rp = (u64)row_l;
        const u32 up_lo = (u32)__shfl_up((int)(u32)rp, 1, WAVE), up_hi = (u32)__shfl_up((int)(u32)(rp >> 32), 1, WAVE);
        const bool in_range = lane >= e_begin && lane < e_end;
        const bool rh_l = in_range && (lane == e_begin || seg_l != seg_up || (u32)rp != up_lo || (u32)(rp >> 32) != up_hi);
        const u64 rheads = __ballot(rh_l);
        const u64 upto = rheads & ((lane == 63) ? ~0ull : ((2ull << lane) - 1ull));
        const int my_head = (in_range && upto) ? 63 - (int)__builtin_clzll(upto) : lane;
        float xs = in_range ? scale_l : 0.f;   // becomes the sum of the scales from the run's first entry to this one
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const float y = __shfl_up(xs, o, WAVE);
            if (lane - o >= my_head) xs += y;
        }
        u64 rmask = rheads;
        while (rmask) {
            LoadedRow<T, NQ, TAIL> r[UNROLL];
            float sc[UNROLL];
            int hd[UNROLL];
#pragma unroll
            for (int x = 0; x < UNROLL; ++x) {
                hd[x] = -1;
                if (rmask) {
                    const int h = (int)__builtin_ctzll(rmask);
                    rmask &= rmask - 1ull;
                    const int last = (rmask ? (int)__builtin_ctzll(rmask) : e_end) - 1;
                    hd[x] = h;
                    sc[x] = rd_lane(xs, last);
                    r[x].load((const T *)rd_lane64(rp, h), a.D, lane);
                }
            }
#pragma unroll
            for (int x = 0; x < UNROLL; ++x) {
                if (hd[x] >= 0) {
                    if (hd[x] != e_begin && ((heads >> hd[x]) & 1ull)) {   // a new row begins here
                        flush();
                        acc.zero();
                        cur = rd_lane(seg_l, hd[x]);
                        const int end = row_end(hd[x]);
                        dest = ((end < 0) || (end - hd[x]) > TILE) ? 2 : 0;
                    }
                    acc.axpy(sc[x], r[x]);
                }
            }
        }
    } else
    for (int e0 = e_begin; e0 < e_end; e0 += UNROLL) {
        LoadedRow<T, NQ, TAIL> r[UNROLL];
        float sc[UNROLL];
        int sg[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int e = e0 + x;
            if (e < e_end) {
                sg[x] = rd_lane(seg_l, e);
                sc[x] = rd_lane(scale_l, e);
                const T *row = (const T *)rd_lane64((u64)row_l, e);
                r[x].load(row, a.D, lane);
            }
        }
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int e = e0 + x;
            if (e < e_end) {
                if (sg[x] != cur) {   // row `cur` is complete (or its share of it): write it out
                    flush();
                    acc.zero();
                    cur = sg[x];
                    const int end = row_end(e);
                    dest = ((end < 0) || (end - e) > TILE) ? 2 : 0;
                }
                acc.axpy(sc[x], r[x]);
            }
        }
    }
    flush();
    // a long row begins in this tile: leave its tile for the kernel that chains the partials
    // (integer counter; the order of the list does not matter, every chain is independent)
    if (dest == 2 && lane == 0) a.long_list[atomicAdd(a.long_cnt, 1)] = tile;
}

// The W_out-side and the W_in-side reduction of a mini-batch are independent: one launch runs both
// (workgroups [0, blocks_in) take the in-side problem, the rest the out-side one), so that the small
// in-side problem costs no launch of its own and its few workgroups start first.
struct SegReducePair {
    SegReduceArgs out, in;
    int blocks_in;    // workgroups of the in-side problem at the front of the grid
};

template <typename T, int NQ, bool TAIL, int TILE_OUT, int TILE_IN>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(NQ == 1 || (NQ == 2 && sizeof(T) == 2 && !TAIL) ? 8 : NQ == 4 ? 5 : 1)))
k_segreduce(SegReducePair p, AuxWork aux)
{
    // the first aux.total workgroups carry the small jobs that ride with this launch
    if ((int)blockIdx.x < aux.total) {
        aux_block<true, false>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    const int b = (int)blockIdx.x - aux.total;
    if (b < p.blocks_in) segreduce_tile<float, NQ, TAIL, 1, TILE_IN>(p.in, b);
    else segreduce_tile<T, NQ, TAIL, 0, TILE_OUT>(p.out, b - p.blocks_in);
}

// Chains the partials of long rows in tile order: one workgroup per long row (grid-strided
// over the list the reduction left), its waves sharing the chain part[tile][1], part[tile+1][0], ...
// (512-thread workgroups: 1024-thread ones wait for a whole compute unit's worth of free wave
// slots when another kernel fills the chip, which starved this kernel for hundreds of microseconds)
#define FIXUP_THREADS 512
template <int ITERS, int TILE>
__device__ __forceinline__ void segfixup_rows(const SegReduceArgs &a, int first, int stride,
                                              float (*red)[ITERS * WAVE * 4])
{
    constexpr int NW = FIXUP_THREADS / WAVE;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int C4 = a.D >> 2;
    const int count = *a.long_cnt;
    for (int i = first; i < count; i += stride) {
        const int tile = a.long_list[i];
        const int t1 = min(a.n, tile * TILE + TILE);
        const int row = a.seg_of[t1 - 1];
        const int end = a.seg_start[row + 1];
        const int len = (end - 1) / TILE - tile;   // tiles after this one that hold a leading partial
        // the chain: leading partials of the tiles up to the next border of a tile block, then one
        // partial per tile block (k_segcross), the last of which ends where the row ends
        const int b1 = tile / TN_SEG_XBLOCK + 1;
        const int to_border = a.cross ? b1 * TN_SEG_XBLOCK - 1 - tile : len;   // no block partials: walk it all
        const int nd = len < to_border ? len : to_border;
        const int nc = (len > to_border) ? ((tile + len) / TN_SEG_XBLOCK - b1 + 1) : 0;
        float4 acc[ITERS];
        zero_row<ITERS>(acc);
        if (wave == 0) load_row<float, ITERS>(acc, a.part + ((size_t)tile * 2 + 1) * a.D, C4, lane);
        for (int j0 = wave; j0 < nd + nc; j0 += NW * SEG_UNROLL) {
            float4 r[SEG_UNROLL][ITERS];
#pragma unroll
            for (int x = 0; x < SEG_UNROLL; ++x) {
                const int j = j0 + x * NW;
                const float *src = (j < nd) ? a.part + (size_t)(tile + 1 + j) * 2 * a.D
                                            : a.cross + (size_t)(b1 + j - nd) * a.D;
                if (j < nd + nc) load_row<float, ITERS>(r[x], src, C4, lane);
                else zero_row<ITERS>(r[x]);
            }
#pragma unroll
            for (int x = 0; x < SEG_UNROLL; ++x) add_row<ITERS>(acc, r[x]);
        }
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            int e = (lane + WAVE * it) * 4;
            red[wave][e + 0] = acc[it].x;
            red[wave][e + 1] = acc[it].y;
            red[wave][e + 2] = acc[it].z;
            red[wave][e + 3] = acc[it].w;
        }
        __syncthreads();
        float *dst = a.out_rows + (size_t)row * a.D;
        for (int e = threadIdx.x; e < a.D; e += FIXUP_THREADS) {
            float s = red[0][e];
#pragma unroll
            for (int w = 1; w < NW; ++w) s += red[w][e];
            dst[e] = s;
        }
        __syncthreads();
    }
}

// A long row's chain of partials can be very long (a hot word of a skewed stream takes a large share of
// all entries), and one workgroup walking it alone would bound the whole step.  The tiles are therefore
// grouped in blocks of TN_SEG_XBLOCK; at most one long row crosses the border at the start of a block,
// and this kernel sums that row's leading partials inside the block into cross[block], all blocks in
// parallel.  k_segfixup then adds one partial per block instead of one per tile.
template <int ITERS, int TILE>
__device__ __forceinline__ void segcross_block(const SegReduceArgs &a, int b, float (*red)[ITERS * WAVE * 4])
{
    constexpr int NW = FIXUP_THREADS / WAVE;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int C4 = a.D >> 2;
    const int t0 = b * TN_SEG_XBLOCK;
    const i64 e0 = (i64)t0 * TILE;
    if (b < 1 || e0 >= a.n || a.xinfo[b] == 0) return;
    const int row = a.seg_of[e0];
    const int start = a.seg_start[row];
    const int end = a.seg_start[row + 1];
    if (start >= e0 || end - start <= TILE) return;   // no row crosses the border, or a short one (no partials)
    const int last_tile = (end - 1) / TILE;
    const int cnt = (last_tile < t0 + TN_SEG_XBLOCK - 1 ? last_tile : t0 + TN_SEG_XBLOCK - 1) - t0 + 1;
    float4 acc[ITERS];
    zero_row<ITERS>(acc);
    for (int j0 = wave; j0 < cnt; j0 += NW * SEG_UNROLL) {
        float4 r[SEG_UNROLL][ITERS];
#pragma unroll
        for (int x = 0; x < SEG_UNROLL; ++x) {
            int j = j0 + x * NW;
            if (j < cnt) load_row<float, ITERS>(r[x], a.part + (size_t)(t0 + j) * 2 * a.D, C4, lane);
            else zero_row<ITERS>(r[x]);
        }
#pragma unroll
        for (int x = 0; x < SEG_UNROLL; ++x) add_row<ITERS>(acc, r[x]);
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int e = (lane + WAVE * it) * 4;
        red[wave][e + 0] = acc[it].x;
        red[wave][e + 1] = acc[it].y;
        red[wave][e + 2] = acc[it].z;
        red[wave][e + 3] = acc[it].w;
    }
    __syncthreads();
    float *dst = a.cross + (size_t)b * a.D;
    for (int e = threadIdx.x; e < a.D; e += FIXUP_THREADS) {
        float s = red[0][e];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[w][e];
        dst[e] = s;
    }
}

template <int ITERS, int TILE_OUT, int TILE_IN>
__global__ void __launch_bounds__(FIXUP_THREADS) k_segcross(SegReducePair p)
{
    __shared__ float red[FIXUP_THREADS / WAVE][ITERS * WAVE * 4];
    const int b = blockIdx.x;
    if (b < p.blocks_in) segcross_block<ITERS, TILE_IN>(p.in, b, red);
    else segcross_block<ITERS, TILE_OUT>(p.out, b - p.blocks_in, red);
}

template <int ITERS, int TILE_OUT, int TILE_IN>
__global__ void __launch_bounds__(FIXUP_THREADS) k_segfixup(SegReducePair p, PrepPhase rider)
{
    constexpr int LDS = FIXUP_THREADS / WAVE * ITERS * WAVE * 4;
    __shared__ u32 lds[LDS > PrepLds<FIXUP_THREADS>::words ? LDS : PrepLds<FIXUP_THREADS>::words];
    if ((int)blockIdx.x < rider.blocks) {
        prep_block<FIXUP_THREADS, false>(rider, (int)blockIdx.x, lds);
        return;
    }
    float (*red)[ITERS * WAVE * 4] = (float (*)[ITERS * WAVE * 4])lds;
    const int b = (int)blockIdx.x - rider.blocks, blocks = (int)gridDim.x - rider.blocks;
    if (b < p.blocks_in) segfixup_rows<ITERS, TILE_IN>(p.in, b, p.blocks_in, red);
    else segfixup_rows<ITERS, TILE_OUT>(p.out, b - p.blocks_in, blocks - p.blocks_in, red);
}

// ITERS: float4 registers per lane of a whole row (the chaining kernels' layout); TAIL: the reduction
// holds rows as ITERS-1 float4 and one float per lane instead (dimensions just above a multiple of 256)
template <typename T, int ITERS, bool TAIL, int TILE_OUT, int TILE_IN>
static void launch_segreduce_i(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    constexpr int NQ = TAIL ? ITERS - 1 : ITERS;
    const int tiles_out = p.out.n > 0 ? (p.out.n + TILE_OUT - 1) / TILE_OUT : 0;
    const int tiles_in = p.in.n > 0 ? (p.in.n + TILE_IN - 1) / TILE_IN : 0;
    if (tiles_out <= TN_SEG_CROSS_MIN) p.out.cross = nullptr;
    if (tiles_in <= TN_SEG_CROSS_MIN) p.in.cross = nullptr;
    const int blocks_out = (tiles_out + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    p.blocks_in = (tiles_in + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    hipLaunchKernelGGL((k_segreduce<T, NQ, TAIL, TILE_OUT, TILE_IN>), dim3(aux.total + p.blocks_in + blocks_out),
                       dim3(BLOCK), aux_lds_bytes(aux), st, p, aux);
    // Partials per block of tiles, for problems large enough that one row's chain could hold up the step:
    // up to TN_SEG_CROSS_MIN tiles even a row that takes every entry is walked by one workgroup in well
    // under a fifth of a millisecond, and the extra launch would cost every step several microseconds.
    const int xb_out = tiles_out > TN_SEG_CROSS_MIN ? (tiles_out + TN_SEG_XBLOCK - 1) / TN_SEG_XBLOCK : 0;
    const int xb_in = tiles_in > TN_SEG_CROSS_MIN ? (tiles_in + TN_SEG_XBLOCK - 1) / TN_SEG_XBLOCK : 0;
    if (xb_out + xb_in > 0) {
        p.blocks_in = xb_in;
        hipLaunchKernelGGL((k_segcross<ITERS, TILE_OUT, TILE_IN>), dim3(xb_in + xb_out), dim3(FIXUP_THREADS), 0, st,
                           p);
    }
    const int fix_out = tn_seg_chains(p.out.n), fix_in = tn_seg_chains(p.in.n);
    if (fix_out + fix_in > 0) {
        p.blocks_in = fix_in;
        hipLaunchKernelGGL((k_segfixup<ITERS, TILE_OUT, TILE_IN>), dim3(rider.blocks + fix_out + fix_in),
                           dim3(FIXUP_THREADS), 0, st, p, rider);
    }
}

template <typename T, int ITERS, bool TAIL>
static void launch_segreduce_t(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    const bool so = tn_seg_tile(p.out.n) == 8, si = tn_seg_tile(p.in.n) == 8;
    if (so) si ? launch_segreduce_i<T, ITERS, TAIL, 8, 8>(p, aux, rider, st) : launch_segreduce_i<T, ITERS, TAIL, 8, 32>(p, aux, rider, st);
    else si ? launch_segreduce_i<T, ITERS, TAIL, 32, 8>(p, aux, rider, st) : launch_segreduce_i<T, ITERS, TAIL, 32, 32>(p, aux, rider, st);
}

template <typename T>
static void launch_segreduce_d(SegReducePair &p, int D, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    const int iters = (D / 4 + WAVE - 1) / WAVE;
    const int rest = D - (iters - 1) * 4 * WAVE;   // elements in the last float4 register of a lane's row
    if (iters >= 2 && rest <= WAVE) {              // a short tail: one float per lane
        switch (iters) {
        case 2: launch_segreduce_t<T, 2, true>(p, aux, rider, st); break;
        case 3: launch_segreduce_t<T, 3, true>(p, aux, rider, st); break;
        default: launch_segreduce_t<T, 4, true>(p, aux, rider, st); break;
        }
        return;
    }
    switch (iters) {
    case 1: launch_segreduce_t<T, 1, false>(p, aux, rider, st); break;
    case 2: launch_segreduce_t<T, 2, false>(p, aux, rider, st); break;
    case 3: launch_segreduce_t<T, 3, false>(p, aux, rider, st); break;
    default: launch_segreduce_t<T, 4, false>(p, aux, rider, st); break;
    }
}

// Either problem may be absent (NULL): the other one then runs alone.
void tn_launch_segreduce(const SegReduceArgs *out, const SegReduceArgs *in, const AuxWork *aux, const PrepPhase *rider,
                         hipStream_t st)
{
    AuxWork none;
    PrepPhase no_rider;
    no_rider.kind = PREP_KEYS;
    no_rider.blocks = 0;
    if (!rider) rider = &no_rider;
    if (!aux) {
        tn_aux_none(none);
        aux = &none;
    }
    SegReducePair p;
    memset(&p, 0, sizeof(p));
    if (out && out->n > 0) p.out = *out;
    if (in && in->n > 0) p.in = *in;
    if (p.out.n <= 0 && p.in.n <= 0) return;   // callers attach jobs only to a mini-batch with pairs
    const int D = p.out.n > 0 ? p.out.D : p.in.D;
    if (p.out.n > 0 && p.out.dtype != 0) launch_segreduce_d<bf16_t>(p, D, *aux, *rider, st);
    else launch_segreduce_d<float>(p, D, *aux, *rider, st);
}
