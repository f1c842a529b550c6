// Gradient calculation of one mini-batch (calculate_gradient of Algorithm 1; the "GC"
// term of Eq. 1 in TensAIR, arXiv 2211.10280, Section 2.2) for a skip-gram model with
// negative sampling: per pair (c, x) and j in {x, negatives},
//   s = <W_in[c], W_out[j]>,  g = (sigmoid(s) - label)/P,
//   Gin[c] += g W_out[j],     Gout[j] += g W_in[c].
//
// Two passes, both free of atomics:
//   forward   one workgroup per center position: the center row stays in registers, the
//             context/negative rows are gathered once, g is stored per occurrence and the
//             center's share of Gin is combined across waves through LDS;
//   segreduce the occurrences sorted by row id are cut into fixed tiles (of 8, 16 or 32 by their number);
//             a wave sums, in sorted order, the short rows that begin in its tile and its share
//             of long rows, whose partials a second kernel chains in tile order.  Load balance
//             is therefore independent of how hot a row is.
#include <string.h>

#include "aux_dev.h"
#include "dev_common.h"
#include "forward_dev.h"
#include "kernels.h"
#include "rows_dev.h"

// ---------------------------------------------------------------- forward
// rows in flight per wave: as many as fit in 64 registers per lane (8 waves per SIMD).  Measured: with
// the tables in cache (D = 256, 10 k words) 4 rows in flight are 19 % faster than 2; at D = 300 and a
// million words the pass moves 0.46 GB of rows through the fabric at the rate random 1.2 KB gathers
// get (5.7 TB/s) and neither more rows in flight, nor prefetching the row ids, nor software pipelining,
// nor keeping neighbouring centers on one XCD changes its time.
template <typename T, int NQ, bool TAIL>
struct FwdShape {
    static constexpr int regs = (sizeof(T) == 2 ? 2 : 4) * NQ + (TAIL ? 1 : 0);   // of a row as loaded
    static constexpr int unroll = regs <= 5 ? 4 : 2;
    static constexpr int row = (NQ * 4 + (TAIL ? 1 : 0)) * WAVE;                  // floats of a wave's row in LDS
    static constexpr unsigned lds = 4u * (WAVES_PER_BLOCK * row + WAVES_PER_BLOCK);   // bytes of LDS of the pass itself
};

// LOSS: also accumulate the loss terms (only when the caller asked for the mean loss).
// PREP: phases of a preparation may ride.  Their code needs a few registers more than the pass itself: where the pass
// fits 8 waves per SIMD, so must they.  Without them the pass leaves registers to the sort that runs beside it on the
// caller's stream where a large mini-batch is not prepared (step with hot rows: 580 us against 610).
template <typename T, int NQ, bool TAIL, bool LOSS, bool PREP>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(NQ == 1 || (NQ == 2 && !TAIL && !LOSS) ? 8 : 1)))
k_forward(FwdArgs a, AuxWork aux)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = FwdShape<T, NQ, TAIL>::unroll;
    constexpr int ROW = FwdShape<T, NQ, TAIL>::row;
    float (*red)[ROW] = (float (*)[ROW])ride_lds;
    float *lred = (float *)ride_lds + WAVES_PER_BLOCK * ROW;
    // the first aux.total workgroups carry the small jobs that ride with this launch (measured: spread among
    // the centers' workgroups instead, alternating one by one or in runs of eight, they cost the forward pass
    // 25 to 35 us more than in front of it)
    if ((int)blockIdx.x < aux.total) {
        aux_block<PREP, PREP>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    const int i = (int)blockIdx.x - aux.total;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const T *w_in = (const T *)a.w_in;
    const T *w_out = (const T *)a.w_out;
    const int Np1 = a.b.N + 1;
    const FwdCenter at = fwd_center(a, i);

    Row v, acc;
    v.load(w_in + (size_t)at.c * a.stride, a.D, lane);
    acc.zero();
    float loss = 0.f;   // per-lane partial (lanes 0..UNROLL-1 carry it)

    // wave `wave` takes tasks wave, wave+4, ...; UNROLL rows are in flight at a time.  The
    // dot products are reduced one by one, then lane x evaluates the sigmoid of task x, so the
    // transcendental code runs once per group instead of once per task.
    for (int t0 = wave; t0 < at.ntasks; t0 += WAVES_PER_BLOCK * UNROLL) {
        LoadedRow<T, NQ, TAIL> u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            int t = t0 + x * WAVES_PER_BLOCK;
            if (t < at.ntasks) {
                u32 j = a.out_keys[at.occ0 + t];
                u[x].load(w_out + (size_t)j * a.stride, a.D, lane);
            } else {
                u[x].zero();
            }
        }
        float s_l = 0.f;
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            float s = wave_sum_dpp(v.dot(u[x]));
            s_l = (lane == x) ? s : s_l;
        }
        const int t_l = t0 + lane * WAVES_PER_BLOCK;
        const bool live = (lane < UNROLL) && (t_l < at.ntasks);
        const float g_t = task_g<LOSS>((t_l % Np1) == 0, s_l, a.inv_P, loss, live);
        const float g_l = live ? g_t : 0.f;
        if (live) a.g[at.occ0 + t_l] = g_l;
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) acc.axpy(rd_lane(g_l, x), u[x]);
    }
    // combine the four waves in a fixed order
    acc.spill(red[wave], lane);
    if (LOSS) {
        loss = wave_sum_dpp(loss);
        if (lane == 0) lred[wave] = loss;
    }
    __syncthreads();
    float *dst = a.center_part + (size_t)i * a.D;
    for (int e = threadIdx.x; e < a.D; e += BLOCK) {
        float s = red[0][e];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += red[w][e];
        dst[e] = s;
    }
    if (LOSS && threadIdx.x == 0) {
        float s = lred[0];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += lred[w];
        a.center_loss[i] = s;
    }
}

// ---------------------------------------------------------------- forward where words repeat (see RepeatList)
template <typename T, int NQ, bool TAIL, bool LOSS, bool PREP>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8)))
k_forward_repeats(FwdArgs a, AuxWork aux)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = FwdShape<T, NQ, TAIL>::unroll;
    constexpr int ROW = FwdShape<T, NQ, TAIL>::row;
    if ((int)blockIdx.x < aux.total) {
        aux_block<PREP, PREP>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    float (*red)[ROW] = (float (*)[ROW])ride_lds;
    float *lred = (float *)ride_lds + WAVES_PER_BLOCK * ROW;
    const int i = (int)blockIdx.x - aux.total;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const T *w_in = (const T *)a.w_in;
    const T *w_out = (const T *)a.w_out;
    const FwdCenter at = fwd_center(a, i);

    Row v, acc;
    v.load(w_in + (size_t)at.c * a.stride, a.D, lane);
    acc.zero();
    RepeatList words;
    words.build(a, at, ride_lds + WAVES_PER_BLOCK * ROW + WAVES_PER_BLOCK);
    float loss = 0.f;
    for (int t0 = wave; t0 < words.n; t0 += WAVES_PER_BLOCK * UNROLL) {
        LoadedRow<T, NQ, TAIL> u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int t = t0 + x * WAVES_PER_BLOCK;
            if (t < words.n) u[x].load(w_out + (size_t)uniform((int)words.ukey[t]) * a.stride, a.D, lane);
            else u[x].zero();
        }
        float s_l = 0.f;
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const float s = wave_sum_dpp(v.dot(u[x]));
            s_l = (lane == x) ? s : s_l;
        }
        const int t_l = t0 + lane * WAVES_PER_BLOCK;
        float sum = 0.f;
        if (lane < UNROLL && t_l < words.n) sum = words.template scale<LOSS>(t_l, s_l, a.inv_P, loss);
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) acc.axpy(rd_lane(sum, x), u[x]);
    }
    // combine the four waves in a fixed order
    acc.spill(red[wave], lane);
    if (LOSS) {
        loss = wave_sum_dpp(loss);
        if (lane == 0) lred[wave] = loss;
    }
    __syncthreads();
    words.store_g(a, at);
    float *dst = a.center_part + (size_t)i * a.D;
    for (int e = threadIdx.x; e < a.D; e += BLOCK) {
        float s = red[0][e];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += red[w][e];
        dst[e] = s;
    }
    if (LOSS && threadIdx.x == 0) {
        float s = lred[0];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += lred[w];
        a.center_loss[i] = s;
    }
}

template <typename T, int NQ, bool TAIL, bool LOSS>
static void launch_forward_k(const FwdArgs &a, const AuxWork &aux, hipStream_t st)
{
    unsigned lds = FwdShape<T, NQ, TAIL>::lds;
    const unsigned riders = aux_lds_bytes(aux);
    if (lds < riders) lds = riders;
    const dim3 grid(aux.total + a.b.n_centers), blk(BLOCK);
    if constexpr (NQ == 1) {
        if (a.repeats) {
            const unsigned own = FwdShape<T, NQ, TAIL>::lds + 4u * repeat_lds(2 * a.b.w * (a.b.N + 1)).words();
            if (lds < own) lds = own;
            if (aux.prep[0].blocks) hipLaunchKernelGGL((k_forward_repeats<T, NQ, TAIL, LOSS, true>), grid, blk, lds, st, a, aux);
            else hipLaunchKernelGGL((k_forward_repeats<T, NQ, TAIL, LOSS, false>), grid, blk, lds, st, a, aux);
            return;
        }
    }
    if (aux.prep[0].blocks) hipLaunchKernelGGL((k_forward<T, NQ, TAIL, LOSS, true>), grid, blk, lds, st, a, aux);
    else hipLaunchKernelGGL((k_forward<T, NQ, TAIL, LOSS, false>), grid, blk, lds, st, a, aux);
}

template <typename T, bool LOSS>
static void launch_forward_t(const FwdArgs &a, const AuxWork &aux, hipStream_t st)
{
    const int full = a.D / (4 * WAVE);           // float4 registers that every lane uses
    const int rest = a.D - full * 4 * WAVE;      // elements beyond them
    if (rest > 0 && rest <= WAVE && full >= 1) {   // a short tail: one float per lane
        switch (full) {
        case 1: launch_forward_k<T, 1, true, LOSS>(a, aux, st); break;
        case 2: launch_forward_k<T, 2, true, LOSS>(a, aux, st); break;
        default: launch_forward_k<T, 3, true, LOSS>(a, aux, st); break;
        }
        return;
    }
    const int iters = (a.D / 4 + WAVE - 1) / WAVE;
    switch (iters) {
    case 1: launch_forward_k<T, 1, false, LOSS>(a, aux, st); break;
    case 2: launch_forward_k<T, 2, false, LOSS>(a, aux, st); break;
    case 3: launch_forward_k<T, 3, false, LOSS>(a, aux, st); break;
    default: launch_forward_k<T, 4, false, LOSS>(a, aux, st); break;
    }
}

void tn_launch_forward(const FwdArgs &a, const AuxWork *aux, hipStream_t st)
{
    AuxWork none;
    if (!aux) {
        tn_aux_none(none);
        aux = &none;
    }
    if (a.D <= TN_SUB_MAX_DIM) {
        tn_launch_forward_sub(a, *aux, st);
        return;
    }
    const bool loss = a.center_loss != nullptr;
    if (a.dtype == 0) loss ? launch_forward_t<float, true>(a, *aux, st) : launch_forward_t<float, false>(a, *aux, st);
    else loss ? launch_forward_t<bf16_t, true>(a, *aux, st) : launch_forward_t<bf16_t, false>(a, *aux, st);
}

// ---------------------------------------------------------------- loss and the empty batch
__global__ void __launch_bounds__(BLOCK) k_loss(const float *center_loss, int n, float inv_P, float *mean_loss)
{
    __shared__ float sm[WAVES_PER_BLOCK];
    aux_mean_loss(center_loss, n, inv_P, mean_loss, sm);
}

void tn_launch_loss(const float *center_loss, int n_centers, float inv_P, float *mean_loss,
                    hipStream_t st)
{
    hipLaunchKernelGGL(k_loss, dim3(1), dim3(BLOCK), 0, st, center_loss, n_centers, inv_P, mean_loss);
}

__global__ void k_empty_grad(int *n_in, int *n_out, float *mean_loss, int *seg_in, int *seg_out)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        *n_in = 0;
        *n_out = 0;
        if (mean_loss) *mean_loss = 0.f;
        if (seg_in) seg_in[0] = 0;
        if (seg_out) seg_out[0] = 0;
    }
}

void tn_launch_empty_grad(int *n_in, int *n_out, float *mean_loss, int *seg_in, int *seg_out,
                          hipStream_t st)
{
    hipLaunchKernelGGL(k_empty_grad, dim3(1), dim3(WAVE), 0, st, n_in, n_out, mean_loss, seg_in, seg_out);
}
