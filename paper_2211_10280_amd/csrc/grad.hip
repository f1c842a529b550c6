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
//   segreduce the occurrences sorted by row id are cut into fixed tiles (32, or 8 for small lists);
//             a wave sums, in sorted order, the short rows that begin in its tile and its share
//             of long rows, whose partials a second kernel chains in tile order.  Load balance
//             is therefore independent of how hot a row is.
#include <string.h>

#include "aux_dev.h"
#include "dev_common.h"
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
    const BatchDesc &b = a.b;
    const i64 p = b.begin + i;
    const T *w_in = (const T *)a.w_in;
    const T *w_out = (const T *)a.w_out;
    const int Np1 = b.N + 1;

    int c = b.tok[p];
    if ((u32)c >= (u32)a.V) c = 0;   // flagged by the key kernel; stay in range
    i64 left = p < b.w ? p : b.w;
    i64 right = (b.T - 1 - p) < b.w ? (b.T - 1 - p) : b.w;
    const int ntasks = (int)(left + right) * Np1;
    const i64 occ0 = (pairs_before(p, b.T, b.w) - b.pair_base) * Np1;

    Row v, acc;
    v.load(w_in + (size_t)c * a.stride, a.D, lane);
    acc.zero();
    float loss = 0.f;   // per-lane partial (lanes 0..UNROLL-1 carry it)

    // wave `wave` takes tasks wave, wave+4, ...; UNROLL rows are in flight at a time.  The
    // dot products are reduced one by one, then lane x evaluates the sigmoid of task x, so the
    // transcendental code runs once per group instead of once per task.
    for (int t0 = wave; t0 < ntasks; t0 += WAVES_PER_BLOCK * UNROLL) {
        LoadedRow<T, NQ, TAIL> u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            int t = t0 + x * WAVES_PER_BLOCK;
            if (t < ntasks) {
                u32 j = a.out_keys[occ0 + t];
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
        const bool live = (lane < UNROLL) && (t_l < ntasks);
        const bool pos = (t_l % Np1) == 0;
        // sigmoid(s) - label without cancellation: label 1: -1/(1+e^s), label 0: 1/(1+e^-s)
        const float z = pos ? s_l : -s_l;
        float gg = 1.0f / (1.0f + expf(z));
        gg = pos ? -gg : gg;
        const float g_l = live ? gg * a.inv_P : 0.f;
        if (live) a.g[occ0 + t_l] = g_l;
        if (LOSS) {
            // loss term: softplus(-s) for the context, softplus(s) for a negative
            const float y = -z;
            if (live) loss += fmaxf(y, 0.f) + log1pf(expf(-fabsf(y)));
        }
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

// ---------------------------------------------------------------- forward where words repeat
// Where few words are frequent, a position's tasks name the same word over and over (10 000 words, Zipf exponent 1.5,
// 256 tasks: 126 different ones): every word is gathered and multiplied once here, and its row added once, scaled by
// what its contexts and its negatives receive together.  The workgroup finds the different words with a hash table in
// LDS; they are worked on in the order of their first task, so the result does not depend on the order of insertion.
// g is stored per task as before (the same bits: one dot product, the same lanes).  The pass is bound by the row
// gathers out of L2, and half of them go; what the table costs (two barriers and some LDS traffic per position) is
// more than that where most words are different, so the host asks for it by the noise distribution (FwdArgs::repeats).
// 16 384 centers, 10 000 words, D = 256: 250 -> 175 us beside the sort (step 576 -> 511 us); 500 centers, 2 000 words, D = 32: step
// 60.5 -> 55.7; no gain where nine tenths of the words are different (5 000 words, 60 tasks: step 40.4 -> 40.6).
struct RepeatLds {
    int slots, tasks;      // slots: a power of two, at least twice the tasks
    __host__ __device__ int words() const { return 3 * slots + 4 * tasks + 2 * WAVES_PER_BLOCK; }
};
__host__ __device__ static inline RepeatLds repeat_lds(int tasks)
{
    RepeatLds l;
    l.tasks = tasks;
    l.slots = tasks <= 256 ? 512 : 1024;
    return l;
}

template <typename T, int NQ, bool TAIL, bool LOSS, bool PREP>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8)))
k_forward_repeats(FwdArgs a, AuxWork aux)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = FwdShape<T, NQ, TAIL>::unroll;
    constexpr int ROW = FwdShape<T, NQ, TAIL>::row;
    constexpr int PER = TN_REPEAT_MAX_TASKS / BLOCK;      // tasks per thread
    if ((int)blockIdx.x < aux.total) {
        aux_block<PREP, PREP>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    float (*red)[ROW] = (float (*)[ROW])ride_lds;
    float *lred = (float *)ride_lds + WAVES_PER_BLOCK * ROW;
    const BatchDesc &b = a.b;
    const int Np1 = b.N + 1;
    const RepeatLds l = repeat_lds(2 * b.w * Np1);
    u32 *key = ride_lds + WAVES_PER_BLOCK * ROW + WAVES_PER_BLOCK;   // [slots] word
    u32 *first = key + l.slots;        // [slots] first task that names it, later its place in the list
    u32 *cnt = first + l.slots;        // [slots] contexts + 65536 * negatives
    u32 *ukey = cnt + l.slots, *ucnt = ukey + l.tasks;               // [tasks] the list: word, counts,
    float *gp = (float *)(ucnt + l.tasks), *gn = gp + l.tasks;       // g of a context and of a negative
    u32 *wn = (u32 *)(gn + l.tasks);   // [PER][waves] different words per wave and round
    const int i = (int)blockIdx.x - aux.total;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const i64 p = b.begin + i;
    const T *w_in = (const T *)a.w_in;
    const T *w_out = (const T *)a.w_out;

    int c = b.tok[p];
    if ((u32)c >= (u32)a.V) c = 0;   // flagged by the key kernel; stay in range
    const i64 left = p < b.w ? p : b.w;
    const i64 right = (b.T - 1 - p) < b.w ? (b.T - 1 - p) : b.w;
    const int ntasks = (int)(left + right) * Np1;         // <= l.tasks <= TN_REPEAT_MAX_TASKS
    const i64 occ0 = (pairs_before(p, b.T, b.w) - b.pair_base) * Np1;

    Row v, acc;
    v.load(w_in + (size_t)c * a.stride, a.D, lane);
    acc.zero();
    u32 mine[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int t = r * BLOCK + (int)threadIdx.x;
        mine[r] = t < ntasks ? a.out_keys[occ0 + t] : 0u;
    }
    for (int s = threadIdx.x; s < l.slots; s += BLOCK) {
        key[s] = 0xFFFFFFFFu;          // no word: ids stay below 2^28
        first[s] = 0xFFFFFFFFu;
        cnt[s] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int t = r * BLOCK + (int)threadIdx.x;
        if (t < ntasks) {
            const u32 k = mine[r];
            // a free slot or the word's own is found: there are at least twice as many slots as tasks
            u32 s = (k * 0x9E3779B1u) >> 22;
            for (;; ++s) {
                s &= (u32)l.slots - 1u;
                const u32 was = atomicCAS(&key[s], 0xFFFFFFFFu, k);
                if (was == 0xFFFFFFFFu || was == k) break;
            }
            atomicMin(&first[s], (u32)t);
            atomicAdd(&cnt[s], t % Np1 == 0 ? 1u : 65536u);
            mine[r] = s;
        }
    }
    __syncthreads();
    // the list of different words, in the order of their first tasks
    u64 own[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int t = r * BLOCK + (int)threadIdx.x;
        own[r] = __ballot(t < ntasks && first[mine[r]] == (u32)t);
        if (lane == 0) wn[r * WAVES_PER_BLOCK + wave] = (u32)__popcll(own[r]);
    }
    __syncthreads();
    int nu = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r)
#pragma unroll
        for (int w = 0; w < WAVES_PER_BLOCK; ++w) {
            if (w == wave && ((own[r] >> lane) & 1ull)) {
                const int at = nu + (int)__popcll(own[r] & ((1ull << lane) - 1ull));
                const u32 s = mine[r];
                ukey[at] = key[s];
                ucnt[at] = cnt[s];
                first[s] = (u32)at;
            }
            nu += (int)wn[r * WAVES_PER_BLOCK + w];
        }
    nu = uniform(nu);
    __syncthreads();
    float loss = 0.f;
    for (int t0 = wave; t0 < nu; t0 += WAVES_PER_BLOCK * UNROLL) {
        LoadedRow<T, NQ, TAIL> u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int t = t0 + x * WAVES_PER_BLOCK;
            if (t < nu) u[x].load(w_out + (size_t)uniform((int)ukey[t]) * a.stride, a.D, lane);
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
        if (lane < UNROLL && t_l < nu) {
            // sigmoid(s) - label without cancellation: label 1: -1/(1+e^s), label 0: 1/(1+e^-s)
            const float g1 = -(1.0f / (1.0f + expf(s_l))) * a.inv_P, g0 = 1.0f / (1.0f + expf(-s_l)) * a.inv_P;
            gp[t_l] = g1;
            gn[t_l] = g0;
            const u32 n = ucnt[t_l];
            const float n1 = (float)(n & 0xFFFFu), n0 = (float)(n >> 16);
            sum = fmaf(n1, g1, n0 * g0);
            if (LOSS) {
                // loss terms: softplus(-s) for a context, softplus(s) for a negative; one that does not occur is left
                // out, not taken zero times (it is infinite where the dot product has overflowed)
                const float tail = log1pf(expf(-fabsf(s_l)));
                if (n & 0xFFFFu) loss += n1 * (fmaxf(-s_l, 0.f) + tail);
                if (n >> 16) loss += n0 * (fmaxf(s_l, 0.f) + tail);
            }
        }
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
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int t = r * BLOCK + (int)threadIdx.x;
        if (t < ntasks) {
            const u32 at = first[mine[r]];
            a.g[occ0 + t] = t % Np1 == 0 ? gp[at] : gn[at];
        }
    }
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
