// The forward pass (see grad.hip) for rows of at most 128 elements.  A whole wave per row would leave half of its lanes
// and more without an element, and the pass is bound by the chain of load, dot product, sigmoid and sum that a wave goes
// through for every few rows: here a wave works on 64 / SUB rows side by side, one per group of SUB lanes (group_dev.h),
// the sigmoid of a group's task is evaluated by all of its lanes, and the groups' sums meet once per position.  With the
// reduction in the same form (reduce_sub.hip): step of 1 327 centers, 4 405 words, D = 92 62.7 -> 48.1 us; 558 centers, 256
// tasks each, D = 56 in bfloat16 76.9 -> 64.6; gradient of 960 centers, 1 443 words, D = 96 64.1 -> 52.9.
#include "aux_dev.h"
#include "dev_common.h"
#include "forward_dev.h"
#include "group_dev.h"
#include "kernels.h"

#ifndef FWD_SUB_UNROLL
#define FWD_SUB_UNROLL 4     // rows in flight per group
#endif
template <int SUB>
struct FwdSubShape {
    static constexpr int row = SUB * 4;                                               // floats of a row in LDS
    static constexpr unsigned lds = 4u * (WAVES_PER_BLOCK * row + WAVES_PER_BLOCK);   // bytes of LDS of the pass itself
};

// `n` rows, the t-th that of word(t); done(t, s, live): what it is scaled by, from its dot product
template <typename T, int SUB, typename Word, typename Done>
__device__ __forceinline__ void forward_rows(const FwdArgs &a, float4 v, float4 &acc, int n, Word word, Done done)
{
    constexpr int RPW = WAVE / SUB, UNROLL = FWD_SUB_UNROLL, STEP = WAVES_PER_BLOCK * RPW;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int slot = lane / SUB, sl = lane % SUB;
    const bool in = sl < (a.D >> 2);
    const T *w_out = (const T *)a.w_out + 4 * sl;
    for (int b = wave * RPW; b < n; b += STEP * UNROLL) {
        u32 key[UNROLL];
        typename Raw4<T>::type u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int t = b + x * STEP + slot;
            key[x] = word(t < n ? t : n - 1);
        }
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            zero_raw(u[x]);
            if (in && b + x * STEP + slot < n) u[x] = ldraw(w_out + (size_t)key[x] * a.stride);
        }
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int t = b + x * STEP + slot;
            const float4 r = widen4(u[x]);
            const float s = group_sum<SUB>(dot4(v, r));
            axpy4(acc, done(t, s, t < n), r);
        }
    }
}

// REPEATS: every different word of a position once (see RepeatList).  PREP: phases of a preparation may ride.
template <typename T, int SUB, bool REPEATS, bool LOSS, bool PREP>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8)))
k_forward_sub(FwdArgs a, AuxWork aux)
{
    constexpr int ROW = FwdSubShape<SUB>::row;
    if ((int)blockIdx.x < aux.total) {
        aux_block<PREP, PREP>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    float (*red)[ROW] = (float (*)[ROW])ride_lds;
    float *lred = (float *)ride_lds + WAVES_PER_BLOCK * ROW;
    const int i = (int)blockIdx.x - aux.total;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int slot = lane / SUB, sl = lane % SUB;
    const FwdCenter at = fwd_center(a, i);

    typename Raw4<T>::type v;
    zero_raw(v);
    if (sl < (a.D >> 2)) v = ldraw((const T *)a.w_in + (size_t)at.c * a.stride + 4 * sl);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float loss = 0.f;       // carried by the first lane of a group
    RepeatList words;
    if constexpr (REPEATS) {
        words.build(a, at, ride_lds + WAVES_PER_BLOCK * ROW + WAVES_PER_BLOCK);
        forward_rows<T, SUB>(a, widen4(v), acc, words.n, [&](int t) { return words.ukey[t]; },
                             [&](int t, float s, bool live) {
                                 float sum = 0.f;
                                 if (live && sl == 0) sum = words.template scale<LOSS>(t, s, a.inv_P, loss);
                                 return __shfl(sum, lane - sl, WAVE);
                             });
    } else {
        const int Np1 = a.b.N + 1;
        const u32 *keys = a.out_keys + at.occ0;
        float *g = a.g + at.occ0;
        forward_rows<T, SUB>(a, widen4(v), acc, at.ntasks, [&](int t) { return keys[t]; },
                             [&](int t, float s, bool live) {
                                 const float x = task_g<LOSS>(t % Np1 == 0, s, a.inv_P, loss, live && sl == 0);
                                 if (live && sl == 0) g[t] = x;
                                 return live ? x : 0.f;
                             });
    }
    // combine the groups, then the waves, in a fixed order
    acc = sum_groups<SUB>(acc);
    if (slot == 0) *(float4 *)&red[wave][4 * sl] = acc;
    if (LOSS) {
        loss = wave_sum_dpp(loss);
        if (lane == 0) lred[wave] = loss;
    }
    __syncthreads();
    if constexpr (REPEATS) words.store_g(a, at);
    if ((int)threadIdx.x < a.D) {
        const int e = threadIdx.x;
        float s = red[0][e];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += red[w][e];
        a.center_part[(size_t)i * a.D + e] = s;
    }
    if (LOSS && threadIdx.x == 0) {
        float s = lred[0];
#pragma unroll
        for (int w = 1; w < WAVES_PER_BLOCK; ++w) s += lred[w];
        a.center_loss[i] = s;
    }
}

template <typename T, int SUB, bool LOSS>
static void launch_forward_sub_k(const FwdArgs &a, const AuxWork &aux, hipStream_t st)
{
    unsigned lds = FwdSubShape<SUB>::lds;
    if (a.repeats) lds += 4u * repeat_lds(2 * a.b.w * (a.b.N + 1)).words();
    const unsigned riders = aux_lds_bytes(aux);
    if (lds < riders) lds = riders;
    const dim3 grid(aux.total + a.b.n_centers), blk(BLOCK);
    const bool prep = aux.prep[0].blocks != 0;
    if (a.repeats) {
        if (prep) hipLaunchKernelGGL((k_forward_sub<T, SUB, true, LOSS, true>), grid, blk, lds, st, a, aux);
        else hipLaunchKernelGGL((k_forward_sub<T, SUB, true, LOSS, false>), grid, blk, lds, st, a, aux);
    } else {
        if (prep) hipLaunchKernelGGL((k_forward_sub<T, SUB, false, LOSS, true>), grid, blk, lds, st, a, aux);
        else hipLaunchKernelGGL((k_forward_sub<T, SUB, false, LOSS, false>), grid, blk, lds, st, a, aux);
    }
}

template <typename T, bool LOSS>
static void launch_forward_sub_t(const FwdArgs &a, const AuxWork &aux, hipStream_t st)
{
    switch (group_lanes(a.D)) {
    case 8: launch_forward_sub_k<T, 8, LOSS>(a, aux, st); break;
    case 16: launch_forward_sub_k<T, 16, LOSS>(a, aux, st); break;
    default: launch_forward_sub_k<T, 32, LOSS>(a, aux, st); break;
    }
}

void tn_launch_forward_sub(const FwdArgs &a, const AuxWork &aux, hipStream_t st)
{
    const bool loss = a.center_loss != nullptr;
    if (a.dtype == 0) loss ? launch_forward_sub_t<float, true>(a, aux, st) : launch_forward_sub_t<float, false>(a, aux, st);
    else loss ? launch_forward_sub_t<bf16_t, true>(a, aux, st) : launch_forward_sub_t<bf16_t, false>(a, aux, st);
}
