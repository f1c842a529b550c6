// The segmented reduction, a row per wave (see reduce_dev.h).
#include <string.h>

#include <algorithm>

#include "reduce_dev.h"
#include "rows_dev.h"

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

template <typename T, int NQ, bool TAIL, int MODE>
__device__ __forceinline__ void segreduce_tile(const SegReduceArgs &a, int block)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = SegShape<T, NQ, TAIL>::unroll;
    // the wave index is made explicitly wave-uniform so that all the control flow below is scalar
    const int tile = block * WAVES_PER_BLOCK + uniform((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    SegWindow win;
    if (!win.load(a, tile)) return;
    const T *row_l = nullptr;
    float scale_l = 0.f;
    if (lane < win.avail) entry_source<T, MODE>(a, win.val_l, row_l, scale_l);
    if (!win.split(a)) return;
    const int seg_l = win.seg_l, e_begin = win.e_begin, e_end = win.e_end;
    const u64 heads = win.heads;
    int dest = win.dest;             // of the current row: 0 out_rows, 1 part[tile][0], 2 part[tile][1]
    Row acc;
    acc.zero();
    float *part = a.part + (size_t)tile * 2 * a.D;
    int cur = rd_lane(seg_l, e_begin);
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
        const int seg_up = __shfl_up(seg_l, 1, WAVE);
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
                        dest = win.row_dest(hd[x]);
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
                    dest = win.row_dest(e);
                }
                acc.axpy(sc[x], r[x]);
            }
        }
    }
    flush();
    if (dest == 2) seg_note_long(a, tile, cur);
}

template <typename T, int NQ, bool TAIL>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(NQ == 1 || (NQ == 2 && sizeof(T) == 2 && !TAIL) ? 8 : NQ == 4 ? 5 : 1)))
k_segreduce(SegReducePair p, AuxWork aux)
{
    // the first aux.total workgroups carry the small jobs that ride with this launch
    if ((int)blockIdx.x < aux.total) {
        aux_block<true, false>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    const int b = (int)blockIdx.x - aux.total;
    if (b < p.blocks_in) segreduce_tile<float, NQ, TAIL, 1>(p.in, b);
    else segreduce_tile<T, NQ, TAIL, 0>(p.out, b - p.blocks_in);
}

// ITERS: float4 registers per lane of a whole row (the chaining kernels' layout); TAIL: the reduction
// holds rows as ITERS-1 float4 and one float per lane instead (dimensions just above a multiple of 256)
template <typename T, int ITERS, bool TAIL>
static void launch_segreduce_t(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    constexpr int NQ = TAIL ? ITERS - 1 : ITERS;
    launch_segreduce_tiles<WideChain<ITERS>>(p, rider, st, [&](int blocks) {
        hipLaunchKernelGGL((k_segreduce<T, NQ, TAIL>), dim3(aux.total + blocks), dim3(BLOCK), aux_lds_bytes(aux), st, p, aux);
    });
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

// Workgroups for the long rows of either side, fewer than k_segfixup has: in the update's launch one that finds none takes its place and
// registers all the same.  As many as there (1 024 and 1 024), 50 steps of 30 000 to 131 072 occurrences 1.003 of the time in the mean, up to
// 1.017; 16 and 128 1.007, up to 1.08 (1 001 words, D = 500, 532 centers 37.0 / 40.0 us).
void tn_chain_work(ChainWork &c, const SegReduceArgs &out, const SegReduceArgs &in)
{
    memset(&c, 0, sizeof(c));
    c.p.out = out;
    c.p.in = in;
    c.p.out.shift = tn_seg_shift(out.n, out.D);
    c.p.in.shift = tn_seg_shift(in.n, in.D);
    c.p.out.cross = c.p.in.cross = nullptr;
    c.p.blocks_in = std::min(tn_seg_chains(in.n, in.D), 64);
    c.blocks = c.p.blocks_in + std::min(tn_seg_chains(out.n, out.D), 512);
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
    if (D <= TN_SUB_MAX_DIM) tn_launch_segreduce_sub(p, *aux, *rider, st);
    else if (p.out.n > 0 && p.out.dtype != 0) launch_segreduce_d<bf16_t>(p, D, *aux, *rider, st);
    else launch_segreduce_d<float>(p, D, *aux, *rider, st);
}
