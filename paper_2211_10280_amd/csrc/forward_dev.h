// What the forward passes (grad.hip: a row per wave; grad_sub.hip: several) have in common: a center position and the
// list of different words among its tasks.
#pragma once
#include "aux_dev.h"
#include "dev_common.h"
#include "kernels.h"

struct FwdCenter {
    int c, ntasks;      // the center's word; its tasks: every context's pair with its negatives
    i64 occ0;           // its first occurrence
};
__device__ __forceinline__ FwdCenter fwd_center(const FwdArgs &a, int i)
{
    const BatchDesc &b = a.b;
    const i64 p = b.begin + i;
    FwdCenter x;
    x.c = b.tok[p];
    if ((u32)x.c >= (u32)a.V) x.c = 0;   // flagged by the key kernel; stay in range
    const i64 left = p < b.w ? p : b.w;
    const i64 right = (b.T - 1 - p) < b.w ? (b.T - 1 - p) : b.w;
    x.ntasks = (int)(left + right) * (b.N + 1);
    x.occ0 = (pairs_before(p, b.T, b.w) - b.pair_base) * (b.N + 1);
    return x;
}

// A word that is a context and a negative so many times of one center word, with dot product s: g of a
// context and of a negative, and what the word's row is scaled by; the loss terms come on top of `loss`.
template <bool LOSS>
__device__ __forceinline__ float pair_scale(u32 contexts, u32 negatives, float s, float inv_P, float &loss, float &g1, float &g0)
{
    // sigmoid(s) - label without cancellation: label 1: -1/(1+e^s), label 0: 1/(1+e^-s)
    g1 = -(1.0f / (1.0f + expf(s))) * inv_P;
    g0 = 1.0f / (1.0f + expf(-s)) * inv_P;
    const float n1 = (float)contexts, n0 = (float)negatives;
    if (LOSS) {
        // loss terms: softplus(-s) for a context, softplus(s) for a negative; one that does not occur is left
        // out, not taken zero times (it is infinite where the dot product has overflowed)
        const float tail = log1pf(expf(-fabsf(s)));
        if (contexts) loss += n1 * (fmaxf(-s, 0.f) + tail);
        if (negatives) loss += n0 * (fmaxf(s, 0.f) + tail);
    }
    return fmaf(n1, g1, n0 * g0);
}

// ---------------------------------------------------------------- the different words of a position
// Where few words are frequent, a position's tasks name the same word over and over (10 000 words, Zipf exponent 1.5,
// 256 tasks: 126 different ones): every word is gathered and multiplied once, and its row added once, scaled by
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

struct RepeatList {
    static constexpr int PER = TN_REPEAT_MAX_TASKS / BLOCK;   // tasks per thread
    u32 *ukey, *ucnt;      // [n] word; contexts + 65536 * negatives
    float *gp, *gn;        // [n] g of a context and of a negative: what the pass finds
    u32 *first;            // [slots] place in the list
    u32 mine[PER];         // slot of every task of this thread
    int n;                 // different words

    // lds: RepeatLds::words() words
    __device__ __forceinline__ void build(const FwdArgs &a, const FwdCenter &x, u32 *lds)
    {
        const int Np1 = a.b.N + 1;
        const RepeatLds l = repeat_lds(2 * a.b.w * Np1);
        const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
        u32 *key = lds;                    // [slots] word
        first = key + l.slots;             // [slots] first task that names it, later its place in the list
        u32 *cnt = first + l.slots;        // [slots]
        ukey = cnt + l.slots;
        ucnt = ukey + l.tasks;
        gp = (float *)(ucnt + l.tasks);
        gn = gp + l.tasks;
        u32 *wn = (u32 *)(gn + l.tasks);   // [PER][waves] different words per wave and round
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int t = r * BLOCK + (int)threadIdx.x;
            mine[r] = t < x.ntasks ? a.out_keys[x.occ0 + t] : 0u;     // ntasks <= l.tasks <= TN_REPEAT_MAX_TASKS
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
            if (t < x.ntasks) {
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
            own[r] = __ballot(t < x.ntasks && first[mine[r]] == (u32)t);
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
        n = uniform(nu);
        __syncthreads();
    }
    // word t's dot product is s: stores its two g, returns what its row is scaled by (the loss terms to `loss`)
    template <bool LOSS>
    __device__ __forceinline__ float scale(int t, float s, float inv_P, float &loss) const
    {
        return pair_scale<LOSS>(ucnt[t] & 0xFFFFu, ucnt[t] >> 16, s, inv_P, loss, gp[t], gn[t]);
    }
    // g of every task, after a barrier
    __device__ __forceinline__ void store_g(const FwdArgs &a, const FwdCenter &x) const
    {
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int t = r * BLOCK + (int)threadIdx.x;
            if (t < x.ntasks) {
                const u32 at = first[mine[r]];
                a.g[x.occ0 + t] = t % (a.b.N + 1) == 0 ? gp[at] : gn[at];
            }
        }
    }
};

// g of one task from its dot product: (sigmoid(s) - label) / P without cancellation: label 1: -1/(1+e^s), label 0: 1/(1+e^-s)
template <bool LOSS>
__device__ __forceinline__ float task_g(bool pos, float s, float inv_P, float &loss, bool counts)
{
    const float z = pos ? s : -s;
    float gg = 1.0f / (1.0f + expf(z));
    gg = pos ? -gg : gg;
    if (LOSS) {
        // loss term: softplus(-s) for the context, softplus(s) for a negative
        const float y = -z;
        if (counts) loss += fmaxf(y, 0.f) + log1pf(expf(-fabsf(y)));
    }
    return gg * inv_P;
}
