// Gradient calculation of a very large mini-batch over a small vocabulary whose words repeat: by pairs of words instead of
// occurrences.  Where a few words are frequent, the same center word meets the same context and negative words over and
// over (16 384 positions, 10 000 words, Zipf exponent 1.5: 4.2 million occurrences, 2.1 million different words counted
// position by position, 0.4 million counted by center word).  The dot product, and with
// it the loss and both terms of g, depend on the two words alone.  So the positions are sorted by their center's word, and
//   k_group_count   counts in LDS how often every word of the vocabulary is a context and a negative of a center word, drawing
//                   the negatives itself: of a frequent center word (tn_group_rare) a chunk of its positions at a time, a counter
//                   per word; of a rare one all positions at once, and lists the words that occur, in order, with a bit per word;
//   k_group_rows    takes the frequent center words against all words, 16 by 64 at a time, by matrix instructions; and works on
//                   every listed word of the rare ones once, as many per workgroup as a position has tasks: the words' scales for
//                   the W_out gradient, and a share of the center word's W_in gradient;
//   k_group_any     turns the rare center words' bits into those of the words;
//   k_group_reduce  adds up, for every word, what the frequent center words give it and the rows of the rare ones that have it
//                   (one workgroup per word), and for every center word its shares.
// No occurrence is listed or sorted (unless the negatives or the offsets of the sorted occurrences are asked for) and nothing is
// chained.  The step above takes 191 us; with chunks of up to 128 positions of any center word, listed all of them, and the
// draws made by a launch before, 319; with the occurrences sorted beside a forward pass position by position (see
// prep_dev.h, grad.hip) 472.  Its launches: the centers' sort 26 us (61 with counts in launches of their own and the keys of
// all occurrences), counts 44 (91, bound by scattered 8-byte stores of the chunks' bits; now a chain of round trips: 44 too without the
// additions in LDS, 34 without the draws), rows 50 (77; the frequent words' workgroups alone 36, of which a wave's matrix instructions are 5,
// the rare ones' 37), bits 7, sums 50 (67: row gathers out of L2).
#include "aux_dev.h"
#include "dev_common.h"
#include "forward_dev.h"
#include "kernels.h"
#include "rows_dev.h"
#include <algorithm>

#define GROUP_THREADS 1024
#define GROUP_WAVES (GROUP_THREADS / WAVE)
#define GROUP_HOT TN_GROUP_HOT  // frequent center words at a time
#define GROUP_TURN 2            // groups of 64 words per wave that turns masks
#define GROUP_BLOCKS 256        // workgroups that count: one per compute unit
#define GROUP_SMALL 1024        // tasks of a center word that a wave counts by itself
#define GROUP_MOST_CHUNKS ((65535 + TN_GROUP_MAX_VOCAB) / GROUP_BLOCKS + 1)     // of a workgroup (tn_group_chunks)
#define GROUP_MOST_RARE (TN_GROUP_MAX_VOCAB / GROUP_BLOCKS + 1)
#define SUM_THREADS 512
#define SUM_WAVES (SUM_THREADS / WAVE)

template <typename T, int NQ, bool TAIL>
struct GroupShape {
    static constexpr int regs = (sizeof(T) == 2 ? 2 : 4) * NQ + (TAIL ? 1 : 0);   // of a row as loaded
    static constexpr int unroll = regs <= 5 ? 4 : 2;
    static constexpr int row = (NQ * 4 + (TAIL ? 1 : 0)) * WAVE;                  // floats of a wave's row in LDS
};

// the waves' rows, one after the other in red, summed in order
template <int THREADS>
__device__ __forceinline__ float sum_waves(const float *red, int row, int e)
{
    double s = red[e];
#pragma unroll
    for (int w = 1; w < THREADS / WAVE; ++w) s += red[w * row + e];
    return (float)s;
}

// A wave's row of long sums, in double: a word's over the rows of the rare center words that have it, group by group of four or
// two (12 228 equal ones, added up in fp32, were off by 50 roundings, now by less than 6), and what the slices of the frequent
// center words give it; a center word's over its shares, of which a rare one has one per `per_center` words of its list and a frequent
// one one per 64 words of the vocabulary.  Those are kept in double themselves: few of them are most of a row, and rounding them
// first is not averaged out (16 384 centers, 10 000 words, Zipf exponent 1.5, D = 256: rows of W_in against 64 bits 6.7e-8, now 6.2e-8, over 120
// inputs; rows of W_out 6.2e-8; both by occurrences 8.6e-8).
template <int NQ, bool TAIL>
struct LongRow {
    double q[NQ][4], t;
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) q[it][0] = q[it][1] = q[it][2] = q[it][3] = 0.0;
        t = 0.0;
    }
    __device__ __forceinline__ void add(const WaveRow<NQ, TAIL> &x)
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            q[it][0] += x.q[it].x;
            q[it][1] += x.q[it].y;
            q[it][2] += x.q[it].z;
            q[it][3] += x.q[it].w;
        }
        if (TAIL) t += x.t;
    }
    __device__ __forceinline__ void load64(const double *row, int D, int lane)
    {
        const int C4 = TAIL ? NQ * WAVE : (D >> 2);
        zero();
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const int c = lane + WAVE * it;
            if (c < C4) {
                const double2 lo = *(const double2 *)(row + 4 * c), hi = *(const double2 *)(row + 4 * c + 2);
                q[it][0] = lo.x;
                q[it][1] = lo.y;
                q[it][2] = hi.x;
                q[it][3] = hi.y;
            }
        }
        if (TAIL && 4 * WAVE * NQ + lane < D) t = row[4 * WAVE * NQ + lane];
    }
    __device__ __forceinline__ void add(const LongRow &x)
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it)
#pragma unroll
            for (int j = 0; j < 4; ++j) q[it][j] += x.q[it][j];
        if (TAIL) t += x.t;
    }
    template <typename T>
    __device__ __forceinline__ void axpy(double a, const LoadedRow<T, NQ, TAIL> &x)
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const float4 v = x.chunk(it);
            q[it][0] = fma(a, (double)v.x, q[it][0]);
            q[it][1] = fma(a, (double)v.y, q[it][1]);
            q[it][2] = fma(a, (double)v.z, q[it][2]);
            q[it][3] = fma(a, (double)v.w, q[it][3]);
        }
        if (TAIL) t = fma(a, (double)x.tail(), t);
    }
    __device__ __forceinline__ void round(WaveRow<NQ, TAIL> &x) const
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) x.q[it] = make_float4((float)q[it][0], (float)q[it][1], (float)q[it][2], (float)q[it][3]);
        x.t = (float)t;
    }
};

// ---------------------------------------------------------------- counting
// Task `rem` of the position of center i (its word: c): the word, with TASK_CONTEXT or not, or TASK_NONE beyond an end of
// the stream.  table: the alias table, in LDS or in memory
#define TASK_NONE 0xFFFFu
#define TASK_CONTEXT 0x8000u                                          // words stay below: TN_GROUP_MAX_VOCAB
template <typename Table>
__device__ __forceinline__ u32 group_task(const GroupArgs &a, u32 per_q, int i, u32 rem, int c, Table table)
{
    const BatchDesc &b = a.f.b;
    const u32 q = (rem * per_q) >> 22, k = rem - q * ((u32)b.N + 1u), w = (u32)b.w;
    const i64 p = b.begin + i, of = p + (q < w ? (i64)q - (i64)w : (i64)q - (i64)w + 1);
    if (of < 0 || of >= b.T) return TASK_NONE;
    int ctx = 0;
    if (k == 0 || a.noise.resample) {
        ctx = b.tok[of];
        if ((u32)ctx >= (u32)a.f.V) {
            ctx = 0;
            atomicOr(a.status, ST_BAD_ID);
        }
    }
    if (k == 0) return (u32)ctx | TASK_CONTEXT;
    const philox_out r = noise_block(a.noise, p, q, k - 1u);
    const u32 bucket = noise_bucket(a.noise, r.r0);
    int word = noise_word(bucket, r.r1, table[bucket]);
    if (a.noise.resample && (word == c || word == ctx)) word = noise_again(a.noise, r.r2, r.r3);
    return (u32)word;
}
// x / Np1 = x * per_q >> 22 for x < per_center <= 512
__device__ __forceinline__ u32 group_per_q(const GroupArgs &a) { return (1u << 22) / ((u32)a.f.b.N + 1u) + 1u; }

// `len` sorted positions from e on, all of center word c: cnt[word] += contexts + 65536 * negatives
__device__ __forceinline__ void group_tasks(const GroupArgs &a, int e, int len, int c, const uint2 *table, u32 *cnt)
{
    constexpr int AT_ONCE = 4;
    const u32 pc = (u32)a.per_center, per_q = group_per_q(a);
    const u32 step_j = GROUP_THREADS / pc, step_r = GROUP_THREADS % pc;
    u32 j = threadIdx.x / pc, r = threadIdx.x % pc;
    while (j < (u32)len) {
        u32 rem[AT_ONCE], task[AT_ONCE];
        int at[AT_ONCE];
#pragma unroll
        for (int x = 0; x < AT_ONCE; ++x) {
            at[x] = j < (u32)len ? (int)a.vals[e + j] : -1;
            rem[x] = r;
            j += step_j;
            r += step_r;
            if (r >= pc) {
                r -= pc;
                ++j;
            }
        }
#pragma unroll
        for (int x = 0; x < AT_ONCE; ++x) task[x] = at[x] >= 0 ? group_task(a, per_q, at[x], rem[x], c, table) : TASK_NONE;
#pragma unroll
        for (int x = 0; x < AT_ONCE; ++x)
            if (task[x] != TASK_NONE) atomicAdd(&cnt[task[x] & ~TASK_CONTEXT], task[x] & TASK_CONTEXT ? 1u : 65536u);
    }
}

__device__ __forceinline__ void group_clear(u32 *cnt, int words)
{
    for (int i = threadIdx.x; i < 16 * words; i += GROUP_THREADS) ((uint4 *)cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
}

// the list of a rare center word's different words, in order, and a bit per word; clears the counters behind it
__device__ __forceinline__ void group_list(const GroupArgs &a, int r, int s0, int c, u32 *cnt, u32 *sums)
{
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id(), words = a.words;
    const int per_wave = (words + GROUP_WAVES - 1) / GROUP_WAVES, w0 = wave * per_wave;      // at most 64 (TN_GROUP_MAX_VOCAB)
    const int mine = min(words - w0, per_wave);
    const u64 below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    u64 mask = 0;                                                     // lane l: of the wave's l-th 64 words
    for (int i = 0; i < mine; ++i) {
        const u64 m = __ballot(cnt[64 * (w0 + i) + lane] != 0u);
        if (lane == i) mask = m;
    }
    const u32 n = (u32)__popcll(mask), incl = wave_incl_scan(n, lane);
    if (lane == WAVE - 1) sums[wave] = incl;
    __syncthreads();
    u32 first = incl - n, all = 0;
#pragma unroll
    for (int w = 0; w < GROUP_WAVES; ++w) {
        if (w < wave) first += sums[w];
        all += sums[w];
    }
    if (lane < mine) {
        a.masks[(size_t)r * words + w0 + lane] = mask;
        a.starts[(size_t)r * words + w0 + lane] = (unsigned short)first;
    }
    if (threadIdx.x == 0) a.meta[r] = make_int4(c, s0, (int)all, 0);
    const size_t base = (size_t)s0 * a.per_center;
    for (int i = 0; i < mine; ++i) {
        const u64 m = rd_lane64(mask, i);
        if (m == 0ull) continue;
        const size_t at = base + (u32)rd_lane((int)first, i) + (u32)__popcll(m & below);
        u32 *k = &cnt[64 * (w0 + i) + lane];
        if ((m >> lane) & 1ull) {
            a.list[at] = (u32)(64 * (w0 + i) + lane);
            a.counts[at] = *k;
            *k = 0;
        }
    }
    __syncthreads();
}

// the same for one of at most GROUP_SMALL tasks, by a wave: a bit per word, a counter per set bit.
// room: 10 * words bytes, then 6 per task, of this wave
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
__device__ __forceinline__ void group_list_small(const GroupArgs &a, int r, int s0, int len, int c, u32 *room)
{
    const int lane = lane_id(), words = a.words, tasks = len * a.per_center;
    const u32 per_q = group_per_q(a);
    u32 *bits = room, *cnt = room + 2 * words;
    unsigned short *task = (unsigned short *)(cnt + GROUP_SMALL), *first = task + GROUP_SMALL;
    for (int i = lane; i < 2 * words; i += WAVE) bits[i] = 0u;
    for (int t = lane; t < tasks; t += WAVE) cnt[t] = 0u;
    wave_order();
    constexpr int AT_ONCE = 4;
    for (int t0 = lane; t0 < tasks; t0 += AT_ONCE * WAVE) {
        u32 x[AT_ONCE];
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const int t = t0 + i * WAVE, j = t / a.per_center;
            x[i] = t < tasks ? group_task(a, per_q, (int)a.vals[s0 + j], (u32)(t - j * a.per_center), c, a.noise.draw) : TASK_NONE;
        }
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const int t = t0 + i * WAVE;
            if (t < tasks) task[t] = (unsigned short)x[i];
            const u32 word = x[i] & ~TASK_CONTEXT;
            if (x[i] != TASK_NONE) atomicOr(&bits[word >> 5], 1u << (word & 31));
        }
    }
    wave_order();
    u32 n = 0;
    for (int w0 = 0; w0 < words; w0 += WAVE) {
        const int wd = w0 + lane;
        const u64 m = wd < words ? ((u64)bits[2 * wd + 1] << 32) | bits[2 * wd] : 0ull;
        const u32 k = (u32)__popcll(m), incl = wave_incl_scan(k, lane);
        if (wd < words) {
            first[wd] = (unsigned short)(n + incl - k);
            a.masks[(size_t)r * words + wd] = m;
            a.starts[(size_t)r * words + wd] = (unsigned short)(n + incl - k);
        }
        n += (u32)rd_lane((int)incl, WAVE - 1);
    }
    if (lane == 0) a.meta[r] = make_int4(c, s0, (int)n, 0);
    wave_order();
    const size_t base = (size_t)s0 * a.per_center;
    for (int t = lane; t < tasks; t += WAVE) {
        const u32 x = task[t], word = x & ~TASK_CONTEXT, wd = word >> 6;
        if (x == TASK_NONE) continue;
        const u64 m = ((u64)bits[2 * wd + 1] << 32) | bits[2 * wd];
        const u32 at = first[wd] + (u32)__popcll(m & ((1ull << (word & 63)) - 1ull));
        atomicAdd(&cnt[at], x & TASK_CONTEXT ? 1u : 65536u);
        a.list[base + at] = word;                                     // the same from each of the word's tasks
    }
    wave_order();
    for (u32 i = lane; i < n; i += WAVE) a.counts[base + i] = cnt[i];
    wave_order();
}
__host__ __device__ static inline int group_room(int words) { return (10 * words + 6 * GROUP_SMALL + 15) / 16 * 4; }   // 32-bit words

// (The table in LDS: every draw reads 8 bytes of it at random, a line of L2 each time: chunks of 79 positions 62 us with 512 threads
// and the table in L2.)
// GROUP_BLOCKS workgroups, which share out the chunks of the frequent center words, then the rare center words, the many that
// have few tasks to a wave each.  The alias table lies in LDS beside a counter per word.
__global__ void __launch_bounds__(GROUP_THREADS) k_group_count(GroupArgs a)
{
    __shared__ u32 sums[2 * GROUP_WAVES];
    __shared__ int4 chunks[GROUP_MOST_CHUNKS];                        // row, chunk of the row, chunk of all
    __shared__ int rare[GROUP_MOST_RARE], small[GROUP_MOST_RARE], found[3];
    u32 *cnt = ride_lds;                                              // [64 * words]
    uint2 *table = (uint2 *)(ride_lds + 64 * a.words);                // [V]
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id(), b = (int)blockIdx.x, turn = GROUP_BLOCKS - 1 - b;
    for (int i = threadIdx.x; i < (int)a.f.V; i += GROUP_THREADS) table[i] = a.noise.draw[i];
    group_clear(cnt, a.words);
    if (b == 0)
        for (int i = threadIdx.x; i < a.words; i += GROUP_THREADS) a.any[i] = 0ull;
    if (threadIdx.x < 3) found[threadIdx.x] = 0;
    // what there is to share out, and this workgroup's part of it
    const int U = *a.n_in;
    u32 run0 = 0, run1 = 0;             // chunks + 65536 * frequent words, rare words + 65536 * small ones so far
    __syncthreads();
    for (int r0 = 0; r0 < U; r0 += GROUP_THREADS) {
        const int r = r0 + (int)threadIdx.x;
        int s0 = 0, len = 0;
        if (r < U) {
            s0 = a.seg_start[r];
            len = a.seg_start[r + 1] - s0;
        }
        const bool hot = len > a.rare, little = len > 0 && !hot && len * a.per_center <= GROUP_SMALL;
        const u32 pieces = hot ? (u32)((len + a.chunk - 1) / a.chunk) : 0u;
        const u32 x0 = hot ? pieces + 65536u : 0u, x1 = little ? 65536u : len > 0 && !hot ? 1u : 0u;
        const u32 i0 = wave_incl_scan(x0, lane), i1 = wave_incl_scan(x1, lane);
        if (lane == WAVE - 1) {
            sums[wave] = i0;
            sums[GROUP_WAVES + wave] = i1;
        }
        __syncthreads();
        u32 e0 = run0 + i0 - x0, e1 = run1 + i1 - x1;
#pragma unroll
        for (int w = 0; w < GROUP_WAVES; ++w) {
            if (w < wave) {
                e0 += sums[w];
                e1 += sums[GROUP_WAVES + w];
            }
            run0 += sums[w];
            run1 += sums[GROUP_WAVES + w];
        }
        if (hot) {
            const int at = (int)(e0 & 0xFFFFu), rank = (int)(e0 >> 16);
            for (int i = (b - at) & (GROUP_BLOCKS - 1); i < (int)pieces; i += GROUP_BLOCKS) chunks[atomicAdd(&found[0], 1)] = make_int4(r, i, at + i, 0);
            if (b == 0) {
                const int c = a.in_ids[r];
                a.frequent[rank] = make_int4(c, r, (int)pieces, at);
                a.meta[r] = make_int4(c, s0, 0, 1 + rank);
            }
        } else if (little) {
            if ((int)((e1 >> 16) & (GROUP_BLOCKS - 1)) == turn) small[atomicAdd(&found[2], 1)] = r;
        } else if (len > 0) {
            if ((int)(e1 & (GROUP_BLOCKS - 1)) == turn) rare[atomicAdd(&found[1], 1)] = r;
        }
        __syncthreads();
    }
    if (b == 0 && threadIdx.x == 0) *a.n_frequent = (int)(run0 >> 16);
    const int n_chunks = uniform(found[0]), n_rare = uniform(found[1]), n_small = uniform(found[2]);
    for (int x = 0; x < n_chunks; ++x) {
        const int r = uniform(chunks[x].x), i = uniform(chunks[x].y);
        const int e = uniform(a.seg_start[r]) + i * a.chunk, end = uniform(a.seg_start[r + 1]);
        group_tasks(a, e, min(a.chunk, end - e), uniform(a.in_ids[r]), table, cnt);
        __syncthreads();
        uint4 *dst = (uint4 *)(a.dense + (size_t)uniform(chunks[x].z) * (64 * a.words));
        for (int k = threadIdx.x; k < 16 * a.words; k += GROUP_THREADS) {
            dst[k] = ((uint4 *)cnt)[k];
            ((uint4 *)cnt)[k] = make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
    }
    for (int x = 0; x < n_rare; ++x) {
        const int r = uniform(rare[x]), s0 = uniform(a.seg_start[r]), c = uniform(a.in_ids[r]);
        group_tasks(a, s0, uniform(a.seg_start[r + 1]) - s0, c, table, cnt);
        __syncthreads();
        group_list(a, r, s0, c, cnt, sums);
    }
    __syncthreads();
    for (int x = wave; x < n_small; x += GROUP_WAVES) {
        const int r = uniform(small[x]), s0 = uniform(a.seg_start[r]);
        group_list_small(a, r, s0, uniform(a.seg_start[r + 1]) - s0, uniform(a.in_ids[r]), ride_lds + wave * group_room(a.words));
    }
}

// ---------------------------------------------------------------- frequent center words
// 64 words of the vocabulary against the frequent center words, GROUP_HOT at a time (every `slices` times as many: the
// workgroups of a slice; of `parts` workgroups, where that would be too few, each has all dot products and a part of the
// rows): their counts, dot products by matrix instructions, scales, then the words' sums over the center words
// and the center words' sums over the words, all but the sigmoid in double: a pair's scale stands for up to all of its tasks, and
// its rounding is not averaged over many of them.
typedef double v4d __attribute__((ext_vector_type(4)));
struct HotLds {
    union {
        struct {
            u32 ctx[GROUP_HOT][WAVE], neg[GROUP_HOT][WAVE];
        };
        double scale[GROUP_HOT][WAVE + 1];     // (rows of 64 would lie in the same banks)
    };
    float s[GROUP_HOT][WAVE];
    u64 met[GROUP_HOT];
    float loss[WAVES_PER_BLOCK];
    u32 odd;               // a row of these is not finite
};
// s[h][w]: dot product of row words[h] of w_in and row first + w of w_out, for 16 of each, by one wave.  A matrix instruction takes
// 4 elements of 16 rows of each table, a lane one of each row; a lane loads 4 neighbouring ones for four instructions.  In double
// (a score's rounding is in all of its tasks); rows of more than 512 elements, of which the forward pass adds up 12 and more in a
// chain too, 16 at a time in fp32: a quarter of the time (40 words, D = 1 024, 2 355 centers of 512 tasks: step 85 / 74 us) for an
// error of the rows against 64 bits that is up to 3 % larger (250 inputs, 10 000 words, D = 1 024 6.7 -> 6.8e-8, 40 words, D = 768 6.2 -> 6.4) and
// below that of pairs whose scores are sums in fp32 throughout (120 inputs, D = 516 6.2 / 6.5, D = 1 024 6.4 / 6.9, 40 words, D = 768 6.6 / 7.0).
template <typename T>
__device__ __forceinline__ void hot_dots(const FwdArgs &f, int word_l, int first, float (*s)[WAVE], int col, int lane, u32 &odd)
{
    constexpr int STEPS = 4;
    const bool wide = f.D > 512;
    const int part = lane >> 4, mine = lane & 15;
    const T *a = (const T *)f.w_in + (size_t)word_l * f.stride, *b = (const T *)f.w_out + (size_t)min(first + mine, (int)f.V - 1) * f.stride;
    v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll 1
    for (int k0 = 0; k0 < f.D; k0 += 16 * STEPS) {
        typename Raw4<T>::type x[STEPS], y[STEPS];
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int k = k0 + 16 * i + 4 * part;
            zero_raw(x[i]);
            zero_raw(y[i]);
            if (k < f.D) {
                x[i] = ldraw(a + k);
                y[i] = ldraw(b + k);
            }
        }
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const float4 u = widen4(x[i]), v = widen4(y[i]);
            if (wide) {
                v4f sum = {0.f, 0.f, 0.f, 0.f};
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(u.x, v.x, sum, 0, 0, 0);
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(u.y, v.y, sum, 0, 0, 0);
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(u.z, v.z, sum, 0, 0, 0);
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(u.w, v.w, sum, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[0][r] += (double)sum[r];
                continue;
            }
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u.x, (double)v.x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u.y, (double)v.y, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u.z, (double)v.z, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u.w, (double)v.w, acc[1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double x = acc[0][i] + acc[1][i];
        s[wide ? 4 * part + i : 4 * i + part][col + mine] = (float)x;      // the two kinds' layouts
        if (!(fabs(x) <= 1.7e308)) odd = 1u;
    }
}

// elements d0 .. d0 + 63 of the sums, a wave: lane l holds element d0 + 4 * (l % 16) + j of rows 4 * r + l / 16 in sum[j][r]
typedef v4d HotTile[4];
__device__ __forceinline__ void hot_step(HotTile &sum, double scale, float4 x)
{
    sum[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(scale, (double)x.x, sum[0], 0, 0, 0);
    sum[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(scale, (double)x.y, sum[1], 0, 0, 0);
    sum[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(scale, (double)x.z, sum[2], 0, 0, 0);
    sum[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(scale, (double)x.w, sum[3], 0, 0, 0);
}
template <typename T>
__device__ __forceinline__ typename Raw4<T>::type hot_load(const T *row, int d, int D)
{
    typename Raw4<T>::type x;
    zero_raw(x);
    if (d < D) x = ldraw(row + d);
    return x;
}

// of the 64 words, over the center words
template <typename T>
__device__ __forceinline__ void hot_words(const FwdArgs &f, const HotLds &l, bool odd, int nh, int word_l, int d0, double *dst, bool first, int lane)
{
    const int part = lane >> 4, mine = lane & 15, d = d0 + 4 * mine;
    const T *w_in = (const T *)f.w_in;
    typename Raw4<T>::type v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = hot_load<T>(w_in + (size_t)__shfl(word_l, 4 * s + part, WAVE) * f.stride, d, f.D);
#pragma unroll 1
    for (int t = 0; t < WAVE; t += 16) {
        HotTile sum = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
        if (odd) {
            for (int h = 0; h < nh; ++h) {
                const float4 x = widen4(hot_load<T>(w_in + (size_t)rd_lane(word_l, h) * f.stride, d, f.D));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int w = t + 4 * r + part;
                    if (!((l.met[h] >> w) & 1ull)) continue;
                    const double s = l.scale[h][w];
                    sum[0][r] = fma(s, (double)x.x, sum[0][r]);
                    sum[1][r] = fma(s, (double)x.y, sum[1][r]);
                    sum[2][r] = fma(s, (double)x.z, sum[2][r]);
                    sum[3][r] = fma(s, (double)x.w, sum[3][r]);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) hot_step(sum, l.scale[4 * s + part][t + mine], widen4(v[s]));
        }
        if (d >= f.D) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double2 *at = (double2 *)(dst + (size_t)(t + 4 * r + part) * f.D + d);
            double2 lo = make_double2(sum[0][r], sum[1][r]), hi = make_double2(sum[2][r], sum[3][r]);
            if (!first) {
                const double2 x = at[0], y = at[1];
                lo = make_double2(lo.x + x.x, lo.y + x.y);
                hi = make_double2(hi.x + y.x, hi.y + y.y);
            }
            at[0] = lo;
            at[1] = hi;
        }
    }
}

// of the center words, over the 64 words from w0 on; row h at dst + h * pitch
template <typename T>
__device__ __forceinline__ void hot_centers(const FwdArgs &f, const HotLds &l, bool odd, int nh, int w0, int d0, double *dst, size_t pitch, int lane)
{
    constexpr int STEPS = 4;
    const int part = lane >> 4, mine = lane & 15, d = d0 + 4 * mine, last = (int)f.V - 1;
    const T *w_out = (const T *)f.w_out;
    HotTile sum = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    if (odd) {
        for (int w = 0; w < WAVE; ++w) {
            const float4 x = widen4(hot_load<T>(w_out + (size_t)min(w0 + w, last) * f.stride, d, f.D));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int h = 4 * r + part;
                if (!((l.met[h] >> w) & 1ull)) continue;
                const double s = l.scale[h][w];
                sum[0][r] = fma(s, (double)x.x, sum[0][r]);
                sum[1][r] = fma(s, (double)x.y, sum[1][r]);
                sum[2][r] = fma(s, (double)x.z, sum[2][r]);
                sum[3][r] = fma(s, (double)x.w, sum[3][r]);
            }
        }
    } else {
#pragma unroll 1
        for (int s0 = 0; s0 < WAVE / 4; s0 += STEPS) {
            typename Raw4<T>::type u[STEPS];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) u[s] = hot_load<T>(w_out + (size_t)min(w0 + 4 * (s0 + s) + part, last) * f.stride, d, f.D);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) hot_step(sum, l.scale[mine][4 * (s0 + s) + part], widen4(u[s]));
        }
    }
    if (d >= f.D) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = 4 * r + part;
        if (h >= nh) continue;
        double2 *at = (double2 *)(dst + (size_t)h * pitch + d);
        at[0] = make_double2(sum[0][r], sum[1][r]);
        at[1] = make_double2(sum[2][r], sum[3][r]);
    }
}

template <typename T, bool LOSS>
__device__ __forceinline__ void group_hot(const GroupArgs &a, int block, HotLds &l)
{
    constexpr int MINE = WAVE / WAVES_PER_BLOCK;                      // words of a wave
    static_assert(GROUP_HOT == 16 && MINE == 16, "tiles of the matrix instructions");
    const FwdArgs &f = a.f;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int group = block % a.words, slice = block / a.words % a.slices, part = block / a.words / a.slices;
    const int n = uniform(*a.n_frequent);
    const int w0 = 64 * group;
    float loss = 0.f;
    u64 any = 0;
#pragma unroll 1
    for (int h0 = slice * GROUP_HOT; h0 < n; h0 += a.slices * GROUP_HOT) {
        const int nh = min(GROUP_HOT, n - h0);
        for (int i = threadIdx.x; i < GROUP_HOT * WAVE; i += BLOCK) (&l.ctx[0][0])[i] = (&l.neg[0][0])[i] = 0u;
        const int4 h_l = a.frequent[h0 + min(lane & 15, nh - 1)];     // lane: the word of center word lane % 16, its chunks
        if (threadIdx.x == 0) l.odd = 0u;
        const int x0 = rd_lane(h_l.w, 0), x1 = rd_lane(h_l.w, nh - 1) + rd_lane(h_l.z, nh - 1);
        __syncthreads();
#pragma unroll 1
        for (int x = x0 + wave; x < x1; x += 8 * WAVES_PER_BLOCK) {
            u32 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = x + i * WAVES_PER_BLOCK < x1 ? a.dense[(size_t)(x + i * WAVES_PER_BLOCK) * (64 * a.words) + w0 + lane] : 0u;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int h = (int)__popcll(__ballot(lane < nh && h_l.w <= x + i * WAVES_PER_BLOCK)) - 1;      // whose chunk it is
                if (v[i] & 0xFFFFu) atomicAdd(&l.ctx[h][lane], v[i] & 0xFFFFu);
                if (v[i] >> 16) atomicAdd(&l.neg[h][lane], v[i] >> 16);
            }
        }
        hot_dots<T>(f, h_l.x, w0 + wave * MINE, l.s, wave * MINE, lane, l.odd);
        __syncthreads();
        // the scales
        double scale[GROUP_HOT * WAVE / BLOCK];
#pragma unroll
        for (int j = 0; j < GROUP_HOT * WAVE / BLOCK; ++j) {
            const int h = j * WAVES_PER_BLOCK + wave;
            const u32 ctx = h < nh ? l.ctx[h][lane] : 0u, neg = h < nh ? l.neg[h][lane] : 0u;
            const u64 met = __ballot((ctx | neg) != 0u);
            float g1 = 0.f, g0 = 0.f;
            if (ctx | neg) (void)pair_scale<LOSS>(ctx, neg, l.s[h][lane], f.inv_P, loss, g1, g0);
            scale[j] = fma((double)ctx, (double)g1, (double)neg * (double)g0);
            if (lane == 0) l.met[h] = met;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < GROUP_HOT * WAVE / BLOCK; ++j) l.scale[j * WAVES_PER_BLOCK + wave][lane] = scale[j];
        __syncthreads();
        for (int h = 0; h < nh; ++h) any |= l.met[h];
        // Words that did not meet have a scale of zero, which takes nothing from a row unless that is not finite: then the
        // products are made one by one.
        const bool odd = uniform((int)l.odd) != 0;
        for (int d0 = 64 * (wave + WAVES_PER_BLOCK * part); d0 < f.D; d0 += 64 * WAVES_PER_BLOCK * a.parts) {
            hot_words<T>(f, l, odd, nh, h_l.x, d0, a.hot_rows + ((size_t)slice * (64 * a.words) + w0) * f.D, h0 == slice * GROUP_HOT, lane);
            hot_centers<T>(f, l, odd, nh, w0, d0, a.hot_part + ((size_t)h0 * a.words + group) * f.D, (size_t)a.words * f.D, lane);
        }
        __syncthreads();
    }
    if (part != 0) return;
    if (any && threadIdx.x == 0) atomicOr((unsigned long long *)&a.any[group], (unsigned long long)any);
    if (LOSS) {
        loss = wave_sum_dpp(loss);
        if (lane == 0) l.loss[wave] = loss;
        __syncthreads();
        if (threadIdx.x == 0) f.center_loss[f.b.n_centers + block] = sum_waves<BLOCK>(l.loss, 1, 0);
    }
}

// ---------------------------------------------------------------- rows
// The workgroups of frequent center words; then one per sorted position: that of a rare center word's i-th takes the words
// [i, i + 1) * per_center of its list, if there are any: it has no more different words than its positions have tasks.  The last
// positions come first: in front are, mostly, those of the frequent center words, for which there is nothing to do here.
template <typename T, int NQ, bool TAIL, bool LOSS>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
k_group_rows(GroupArgs a, AuxWork aux)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = GroupShape<T, NQ, TAIL>::unroll, ROW = GroupShape<T, NQ, TAIL>::row;
    struct RowsLds {
        float red[WAVES_PER_BLOCK * ROW + WAVES_PER_BLOCK];
        u32 word[TN_REPEAT_MAX_TASKS], count[TN_REPEAT_MAX_TASKS];           // per_center is no more
    };
    __shared__ union {
        RowsLds rows;
        HotLds hot;
    } lds;
    if ((int)blockIdx.x < aux.total) {
        aux_block<false, false>(aux, (int)blockIdx.x, (u32 *)&lds);
        return;
    }
    const int hot = a.words * a.slices * a.parts;
    int b = (int)blockIdx.x - aux.total;
    if (b < hot) {
        group_hot<T, LOSS>(a, b, lds.hot);
        return;
    }
    float *red = lds.rows.red;
    u32 *word = lds.rows.word, *count = lds.rows.count;
    const FwdArgs &f = a.f;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int e = f.b.n_centers - 1 - (b - hot);
    const int r = uniform(a.seg_of[e]);
    const int4 center = a.meta[r];
    const int i = e - uniform(center.y);
    const int n = min(a.per_center, uniform(center.z) - i * a.per_center);
    if (n <= 0) {
        if (LOSS && threadIdx.x == 0) f.center_loss[e] = 0.f;
        return;
    }
    const size_t base = (size_t)e * a.per_center;
    Row v, acc;
    v.load((const T *)f.w_in + (size_t)uniform(center.x) * f.stride, f.D, lane);
    acc.zero();
    float loss = 0.f;
    for (int t = threadIdx.x; t < n; t += BLOCK) {
        word[t] = a.list[base + t];
        count[t] = a.counts[base + t];
    }
    __syncthreads();
    for (int t0 = wave; t0 < n; t0 += WAVES_PER_BLOCK * UNROLL) {
        LoadedRow<T, NQ, TAIL> u[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int t = t0 + x * WAVES_PER_BLOCK;
            if (t < n) u[x].load((const T *)f.w_out + (size_t)uniform((int)word[t]) * f.stride, f.D, lane);
            else u[x].zero();
        }
        const int t_l = t0 + lane * WAVES_PER_BLOCK;
        const bool live = lane < UNROLL && t_l < n;
        float s_l = 0.f;
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const float s = wave_sum_dpp(v.dot(u[x]));
            s_l = (lane == x) ? s : s_l;
        }
        float sum = 0.f;
        if (live) {
            float g1, g0;
            const u32 k = count[t_l];
            sum = pair_scale<LOSS>(k & 0xFFFFu, k >> 16, s_l, f.inv_P, loss, g1, g0);
            f.g[base + t_l] = sum;
        }
        Row part;       // sums of sums: one long chain of additions loses accuracy
        part.zero();
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) part.axpy(rd_lane(sum, x), u[x]);
        acc.axpy(1.0f, part);
    }
    acc.spill(red + wave * ROW, lane);
    if (LOSS) {
        loss = wave_sum_dpp(loss);
        if (lane == 0) red[WAVES_PER_BLOCK * ROW + wave] = loss;
    }
    __syncthreads();
    for (int d = threadIdx.x; d < f.D; d += BLOCK) f.center_part[(size_t)e * f.D + d] = sum_waves<BLOCK>(red, ROW, d);
    if (LOSS && threadIdx.x == 0) f.center_loss[e] = sum_waves<BLOCK>(red + WAVES_PER_BLOCK * ROW, 1, 0);
}

// ---------------------------------------------------------------- the words' rare center words
// grid: (64 rows of center words, groups of 64 words in runs of GROUP_TURN waves): 64 by 64 bits, a row of center words per
// lane, turned into a bit per center word for each of 64 words
__global__ void __launch_bounds__(BLOCK) k_group_any(GroupArgs a)
{
    const int U = *a.n_in, r0 = (int)blockIdx.x * WAVE;
    if (r0 >= U) return;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int w0 = ((int)blockIdx.y * WAVES_PER_BLOCK + wave) * GROUP_TURN;
    const int r = r0 + lane;
    const bool rare = r < U && a.meta[r].z > 0;
    u64 m[GROUP_TURN];
#pragma unroll
    for (int x = 0; x < GROUP_TURN; ++x) m[x] = rare && w0 + x < a.words ? a.masks[(size_t)r * a.words + w0 + x] : 0ull;
#pragma unroll
    for (int x = 0; x < GROUP_TURN; ++x) {
        if (w0 + x >= a.words) break;
        u64 turned = 0;
#pragma unroll
        for (int bit = 0; bit < 64; ++bit) {
            const u64 has = __ballot((m[x] >> bit) & 1ull);
            turned = lane == bit ? has : turned;
        }
        a.turned[(size_t)blockIdx.x * (64 * a.words) + 64 * (w0 + x) + lane] = turned;
        const u64 any = __ballot(turned != 0ull);
        if (lane == 0 && any) atomicOr((unsigned long long *)&a.any[w0 + x], (unsigned long long)any);
    }
}

// ---------------------------------------------------------------- sums
// workgroups: the jobs that ride, the frequent center words, the words, the rare center words (SUM_WAVES each)
template <typename T, int NQ, bool TAIL>
__global__ void __launch_bounds__(SUM_THREADS) __attribute__((amdgpu_waves_per_eu(NQ == 1 ? (TAIL ? 6 : 8) : NQ == 2 ? (TAIL ? 5 : 6) : 4))) k_group_reduce(GroupArgs a, AuxWork aux, int blocks_hot, int blocks_out)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int ROW = GroupShape<float, NQ, TAIL>::row;
    __shared__ float red[SUM_WAVES * ROW];
    __shared__ int ahead[SUM_WAVES];
    if ((int)blockIdx.x < aux.total) {
        if ((int)threadIdx.x < BLOCK) aux_block<false, false>(aux, (int)blockIdx.x, (u32 *)red);
        return;
    }
    const FwdArgs &f = a.f;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int U = *a.n_in;
    int b = (int)blockIdx.x - aux.total;
    LongRow<NQ, TAIL> total;
    total.zero();
    if (b < blocks_hot) {                   // a frequent center word: the shares of all 64 words
        if (b >= *a.n_frequent) return;
        const int r = uniform(a.frequent[b].y);
        constexpr int AT_ONCE = NQ == 1 ? 4 : 2;
        const double *rows = a.hot_part + (size_t)b * a.words * f.D;
        for (int q0 = wave; q0 < a.words; q0 += AT_ONCE * SUM_WAVES) {
            LongRow<NQ, TAIL> x[AT_ONCE];
#pragma unroll
            for (int j = 0; j < AT_ONCE; ++j) {
                if (q0 + j * SUM_WAVES < a.words) x[j].load64(rows + (size_t)(q0 + j * SUM_WAVES) * f.D, f.D, lane);
                else x[j].zero();
            }
#pragma unroll
            for (int j = 0; j < AT_ONCE; ++j) total.add(x[j]);
        }
        Row acc;
        total.round(acc);
        acc.spill(red + wave * ROW, lane);
        __syncthreads();
        for (int d = threadIdx.x; d < f.D; d += SUM_THREADS) a.in_rows[(size_t)r * f.D + d] = sum_waves<SUM_THREADS>(red, ROW, d);
        return;
    }
    b -= blocks_hot;
    if (b >= blocks_out) {                  // a rare center word per wave: the shares of its list
        const int r = (b - blocks_out) * SUM_WAVES + wave;
        if (r >= U) return;
        const int4 center = a.meta[r];
        if (uniform(center.w) != 0) return;
        const int shares = (uniform(center.z) + a.per_center - 1) / a.per_center;
        const float *rows = f.center_part + (size_t)uniform(center.y) * f.D;
        for (int q0 = 0; q0 < shares; q0 += 4) {
            LoadedRow<float, NQ, TAIL> x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (q0 + j < shares) x[j].load(rows + (size_t)(q0 + j) * f.D, f.D, lane);
                else x[j].zero();
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) total.axpy(1.0, x[j]);
        }
        Row acc;
        total.round(acc);
        acc.template store<false>(a.in_rows + (size_t)r * f.D, f.D, lane);
        return;
    }
    // a word: what the frequent center words give it, and the rare ones that have it
    constexpr int UNROLL = GroupShape<T, NQ, TAIL>::unroll;
    const int word = b >> 6, bit = b & 63;
    const bool last = b == (int)f.V - 1;
    const bool here = (a.any[word] >> bit) & 1ull;
    if (!here && !last && bit != 0) return;
    const u64 upto = (1ull << bit) - 1ull;
    int n = 0;                              // rows ahead of this word's
    for (int wd = threadIdx.x; wd <= word; wd += SUM_THREADS) n += (int)__popcll(wd < word ? a.any[wd] : a.any[wd] & upto);
    n = (int)rd_lane((int)wave_incl_scan((u32)n, lane), WAVE - 1);
    if (lane == 0) ahead[wave] = n;
    __syncthreads();
    n = 0;
#pragma unroll
    for (int w = 0; w < SUM_WAVES; ++w) n += ahead[w];
    if (last && threadIdx.x == 0) *a.out_n = n + (here ? 1 : 0);
    if (a.index_mask && bit == 0 && threadIdx.x == 0) {      // the update's index of these rows, a word of it each
        a.index_mask[word] = a.any[word];
        a.index_start[word] = (u32)n;
    }
    if (!here) return;
    if (threadIdx.x == 0) a.out_ids[n] = b;
    const int hot = uniform(*a.n_frequent), slices = min(a.slices, (hot + GROUP_HOT - 1) / GROUP_HOT);
    for (int s = wave; s < slices; s += SUM_WAVES) {
        LongRow<NQ, TAIL> x;
        x.load64(a.hot_rows + ((size_t)s * (64 * a.words) + b) * f.D, f.D, lane);
        total.add(x);
    }
    // a wave takes every SUM_WAVES-th center word
    for (int g0 = 0; g0 < (U + WAVE - 1) / WAVE; g0 += WAVE) {
        u64 has = 0;
        if ((g0 + lane) * WAVE < U) has = a.turned[(size_t)(g0 + lane) * (64 * a.words) + b] & (0x0101010101010101ull << wave);
        while (__ballot(has != 0ull)) {     // one of every lane's at a time
            int c = 0;
            float s_l = 0.f;
            const bool one = has != 0ull;
            if (one) {
                const int r = (g0 + lane) * WAVE + (int)__builtin_ctzll(has);
                has &= has - 1ull;
                const int4 center = a.meta[r];
                const size_t at = (size_t)r * a.words + word;
                c = center.x;
                s_l = f.g[(size_t)center.y * a.per_center + a.starts[at] + (u32)__popcll(a.masks[at] & upto)];
            }
            u64 m = __ballot(one);
            while (m) {
                LoadedRow<T, NQ, TAIL> x[UNROLL];
                int at[UNROLL];
#pragma unroll
                for (int j = 0; j < UNROLL; ++j) {
                    at[j] = -1;
                    if (m) {
                        at[j] = (int)__builtin_ctzll(m);
                        m &= m - 1ull;
                        x[j].load((const T *)f.w_in + (size_t)rd_lane(c, at[j]) * f.stride, f.D, lane);
                    }
                }
                Row part;
                part.zero();
#pragma unroll
                for (int j = 0; j < UNROLL; ++j)
                    if (at[j] >= 0) part.axpy(rd_lane(s_l, at[j]), x[j]);
                total.add(part);
            }
        }
    }
    Row acc;
    total.round(acc);
    acc.spill(red + wave * ROW, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < f.D; i += SUM_THREADS) a.out_rows[(size_t)n * f.D + i] = sum_waves<SUM_THREADS>(red, ROW, i);
}

template <typename T, int NQ, bool TAIL>
static void launch_group_k(const GroupArgs &a, int what, const AuxWork &aux, hipStream_t st)
{
    const int n = a.f.b.n_centers, V = (int)a.f.V, rows = std::min(n, V);
    if (what == GROUP_ROWS) {
        const unsigned lds = 4u * std::max(192u * (unsigned)a.words, GROUP_WAVES * (unsigned)group_room(a.words));
        hipLaunchKernelGGL(k_group_count, dim3(GROUP_BLOCKS), dim3(GROUP_THREADS), lds, st, a);
        const dim3 grid(aux.total + a.words * a.slices * a.parts + n), blk(BLOCK);
        if (a.f.center_loss) hipLaunchKernelGGL((k_group_rows<T, NQ, TAIL, true>), grid, blk, 0, st, a, aux);
        else hipLaunchKernelGGL((k_group_rows<T, NQ, TAIL, false>), grid, blk, 0, st, a, aux);
        return;
    }
    const int blocks_hot = what & GROUP_SUMS_IN ? a.most_frequent : 0, blocks_in = what & GROUP_SUMS_IN ? (rows + SUM_WAVES - 1) / SUM_WAVES : 0;
    const int blocks_out = what & GROUP_SUMS_OUT ? V : 0;
    if (blocks_out) hipLaunchKernelGGL(k_group_any, dim3((rows + WAVE - 1) / WAVE, (a.words + WAVES_PER_BLOCK * GROUP_TURN - 1) / (WAVES_PER_BLOCK * GROUP_TURN)), dim3(BLOCK), 0, st, a);
    hipLaunchKernelGGL((k_group_reduce<T, NQ, TAIL>), dim3(aux.total + blocks_hot + blocks_out + blocks_in), dim3(SUM_THREADS), 0, st, a, aux, blocks_hot, blocks_out);
}

template <typename T>
static void launch_group_t(const GroupArgs &a, int what, const AuxWork &x, hipStream_t st)
{
    const int full = a.f.D / (4 * WAVE), rest = a.f.D - full * 4 * WAVE;   // as in the forward pass
    if (rest > 0 && rest <= WAVE && full >= 1) {
        switch (full) {
        case 1: launch_group_k<T, 1, true>(a, what, x, st); break;
        case 2: launch_group_k<T, 2, true>(a, what, x, st); break;
        default: launch_group_k<T, 3, true>(a, what, x, st); break;
        }
        return;
    }
    switch ((a.f.D / 4 + WAVE - 1) / WAVE) {
    case 1: launch_group_k<T, 1, false>(a, what, x, st); break;
    case 2: launch_group_k<T, 2, false>(a, what, x, st); break;
    case 3: launch_group_k<T, 3, false>(a, what, x, st); break;
    default: launch_group_k<T, 4, false>(a, what, x, st); break;
    }
}

void tn_launch_group(const GroupArgs &a, int what, const AuxWork &aux, hipStream_t st)
{
    if (a.f.dtype == 0) launch_group_t<float>(a, what, aux, st);
    else launch_group_t<bf16_t>(a, what, aux, st);
}
