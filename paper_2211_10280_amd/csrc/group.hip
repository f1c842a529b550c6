// Gradient calculation of a very large mini-batch over a small vocabulary whose words repeat: by pairs of words instead of
// occurrences.  Where a few words are frequent, the same center word meets the same context and negative words over and
// over (16 384 positions, 10 000 words, Zipf exponent 1.5: 4.2 million occurrences, 2.1 million different words counted
// position by position, 0.65 million counted for up to 128 positions of a center word together).  The dot product, and with
// it the loss and both terms of g, depend on the two words alone.  So the positions are sorted by their center's word, and
//   k_group_count   takes up to 128 positions of one center word -- a chunk -- per workgroup, counts in
//                   LDS how often every word of the vocabulary is a context and a negative of theirs, and lists the words
//                   that occur, in order, with a bit per word and chunk;
//   k_group_rows    works on every listed word once, as many per workgroup as a position has tasks: the words' scales for
//                   the W_out gradient, and a share of the center word's W_in gradient;
//   k_group_reduce  adds up, for every word, the rows of the chunks that have it (one workgroup per word, the chunks in
//                   order), and for every center word its shares.
// No occurrence is sorted (unless the offsets of the sorted occurrences are asked for) and nothing is chained.  The last two
// are bound by row gathers out of L2; against sorting the occurrences beside a forward pass position by position (see
// prep_dev.h, grad.hip) the step above takes 319 us, 472 before.  (Counting and rows in one kernel, a chunk per workgroup,
// left most of the chip waiting for the chunks of the frequent center words: 446 us at best.)
#include "aux_dev.h"
#include "dev_common.h"
#include "forward_dev.h"
#include "kernels.h"
#include "rows_dev.h"
#include <algorithm>

#define GROUP_THREADS 512
#define GROUP_WAVES (GROUP_THREADS / WAVE)
#define GROUP_RANGE 2           // sorted positions per workgroup; it takes the chunks that begin there (1 / 2 / 4: step 324 / 319 / 326 us)
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

// A wave's row of long sums.  Hundreds of chunks are added up for a frequent word, and in one chain of fp32 additions that
// loses accuracy (rows of W_out against 64 bits 2.6e-7; sums of four or eight rows added up in fp32 1.3e-7; in double 0.6e-7 to
// 0.9e-7; the reduction of sorted occurrences, whose sums meet in a tree, 0.7e-7 to 1.0e-7.  The shares of a center word are as
// many as it has chunks: 500 000 centers of 2 words 1.5e-7 in fp32, 0.9e-7 in double).
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
    __device__ __forceinline__ void round(WaveRow<NQ, TAIL> &x) const
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) x.q[it] = make_float4((float)q[it][0], (float)q[it][1], (float)q[it][2], (float)q[it][3]);
        x.t = (float)t;
    }
};

// the chunk that begins at sorted position e, the i-th of row r, is number r + (first position of r) / positions + i: the
// chunks of a row are neighbours, and at most one number per row stays unused.  lds: a counter per word, then what the
// words before every 64 come to
__device__ __forceinline__ void group_chunk(const GroupArgs &a, int e, int r, int s0, int end, u32 *lds)
{
    const FwdArgs &f = a.f;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int Np1 = f.b.N + 1, words = a.words;
    const int len = min(a.positions, end - e), chunk = r + s0 / a.positions + (e - s0) / a.positions;
    const u64 below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    u32 *cnt = lds;                                                   // contexts + 65536 * negatives
    u32 *sums = lds + 64 * words;                                     // [words + 1]
    for (int i = threadIdx.x; i < 64 * words; i += GROUP_THREADS) cnt[i] = 0;
    __syncthreads();
    for (int j = wave; j < len; j += 2 * GROUP_WAVES) {               // two positions at a time: their look-ups overlap
        const bool two = j + GROUP_WAVES < len;
        const int p0 = (int)a.vals[e + j], p1 = two ? (int)a.vals[e + j + GROUP_WAVES] : p0;
        const FwdCenter x0 = fwd_center(f, p0), x1 = fwd_center(f, p1);
        const int n0 = x0.ntasks, n1 = two ? x1.ntasks : 0;
        for (int k = lane; k < max(n0, n1); k += 4 * WAVE) {
            u32 key[2][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                key[0][q] = k + q * WAVE < n0 ? f.out_keys[x0.occ0 + k + q * WAVE] : 0xFFFFFFFFu;
                key[1][q] = k + q * WAVE < n1 ? f.out_keys[x1.occ0 + k + q * WAVE] : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32 one = (k + q * WAVE) % Np1 == 0 ? 1u : 65536u;
                if (key[0][q] != 0xFFFFFFFFu) atomicAdd(&cnt[key[0][q]], one);
                if (key[1][q] != 0xFFFFFFFFu) atomicAdd(&cnt[key[1][q]], one);
            }
        }
    }
    __syncthreads();
    for (int wd = wave; wd < words; wd += GROUP_WAVES) {
        const u64 m = __ballot(cnt[64 * wd + lane] != 0u);
        if (lane == 0) {
            sums[wd] = (u32)__popcll(m);
            a.masks[(size_t)wd * a.pitch + chunk] = m;
        }
    }
    __syncthreads();
    if (wave == 0) {
        u32 run = 0;
        for (int w0 = 0; w0 < words; w0 += WAVE) {
            const u32 x = w0 + lane < words ? sums[w0 + lane] : 0u;
            const u32 incl = wave_incl_scan(x, lane);
            if (w0 + lane < words) sums[w0 + lane] = run + incl - x;
            run += (u32)rd_lane((int)incl, WAVE - 1);
        }
        if (lane == 0) a.meta[chunk] = make_int4(fwd_center(f, (int)a.vals[e]).c, e, (int)run, 0);
    }
    __syncthreads();
    const size_t base = (size_t)e * a.per_center;
    for (int wd = wave; wd < words; wd += GROUP_WAVES) {
        const u32 k = cnt[64 * wd + lane];
        const u64 m = __ballot(k != 0u);
        if (k != 0u) {
            const size_t at = base + sums[wd] + (u32)__popcll(m & below);
            a.list[at] = (u32)(64 * wd + lane);
            a.counts[at] = k;
        }
        if (lane == 0) a.starts[(size_t)wd * a.pitch + chunk] = (unsigned short)sums[wd];
    }
    if (e + len == end && chunk + 1 < r + 1 + end / a.positions) {    // the unused number after the row's last chunk
        for (int wd = threadIdx.x; wd < words; wd += GROUP_THREADS) a.masks[(size_t)wd * a.pitch + chunk + 1] = 0ull;
        if (threadIdx.x == 0) a.meta[chunk + 1] = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
}

__global__ void __launch_bounds__(GROUP_THREADS) k_group_count(GroupArgs a)
{
    const int e0 = (int)blockIdx.x * GROUP_RANGE;
    for (int e = e0; e < min(a.f.b.n_centers, e0 + GROUP_RANGE); ++e) {
        const int r = uniform(a.seg_of[e]), s0 = uniform(a.seg_start[r]);
        if ((e - s0) % a.positions == 0) group_chunk(a, e, r, s0, uniform(a.seg_start[r + 1]), ride_lds);
    }
}

// The workgroup of the i-th position of a chunk takes the words [i, i + 1) * per_center of the chunk's list, if there are
// any: a chunk has no more different words than its positions have tasks.
template <typename T, int NQ, bool TAIL, bool LOSS>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(NQ == 1 ? 8 : 1)))
k_group_rows(GroupArgs a, AuxWork aux)
{
    typedef WaveRow<NQ, TAIL> Row;
    constexpr int UNROLL = GroupShape<T, NQ, TAIL>::unroll, ROW = GroupShape<T, NQ, TAIL>::row;
    __shared__ float red[WAVES_PER_BLOCK * ROW + WAVES_PER_BLOCK];
    __shared__ u32 word[TN_REPEAT_MAX_TASKS], count[TN_REPEAT_MAX_TASKS];    // per_center is no more
    if ((int)blockIdx.x < aux.total) {
        aux_block<false, false>(aux, (int)blockIdx.x, (u32 *)red);
        return;
    }
    const FwdArgs &f = a.f;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int e = (int)blockIdx.x - aux.total;
    const int r = uniform(a.seg_of[e]), s0 = uniform(a.seg_start[r]), i = (e - s0) % a.positions;
    const int4 chunk = a.meta[r + s0 / a.positions + (e - s0) / a.positions];
    const int n = min(a.per_center, uniform(chunk.z) - i * a.per_center);
    if (n <= 0) {
        if (LOSS && threadIdx.x == 0) f.center_loss[e] = 0.f;
        return;
    }
    const size_t base = (size_t)e * a.per_center;
    Row v, acc;
    v.load((const T *)f.w_in + (size_t)uniform(chunk.x) * f.stride, f.D, lane);
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
            sum = pair_scale<LOSS>(count[t_l], s_l, f.inv_P, loss, g1, g0);
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

// the words that any chunk has; a workgroup per 64 of them
__global__ void __launch_bounds__(BLOCK) k_group_any(GroupArgs a)
{
    __shared__ u64 part[WAVES_PER_BLOCK];
    const int chunks = *a.n_in + a.f.b.n_centers / a.positions;
    u64 m = 0;
    for (int i = threadIdx.x; i < chunks; i += BLOCK) m |= a.masks[(size_t)blockIdx.x * a.pitch + i];
    const u64 all = ((u64)wave_or((u32)(m >> 32)) << 32) | wave_or((u32)m);
    if (lane_id() == 0) part[threadIdx.x >> 6] = all;
    __syncthreads();
    if (threadIdx.x == 0) a.any[blockIdx.x] = part[0] | part[1] | part[2] | part[3];
}

// workgroups: the jobs that ride, W_in's rows, the words
template <typename T, int NQ, bool TAIL>
__global__ void __launch_bounds__(SUM_THREADS) k_group_reduce(GroupArgs a, AuxWork aux, int blocks_in)
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
    float *dst;
    if (b < blocks_in) {                    // a center word: the shares of its chunks, a chunk per wave
        if (b >= U) return;
        const int s0 = a.seg_start[b], chunks = (a.seg_start[b + 1] - s0 + a.positions - 1) / a.positions;
        for (int i = wave; i < chunks; i += SUM_WAVES) {
            const int n = uniform(a.meta[b + s0 / a.positions + i].z);
            const int shares = (n + a.per_center - 1) / a.per_center;
            const float *rows = f.center_part + (size_t)(s0 + i * a.positions) * f.D;
            Row of_chunk;
            of_chunk.zero();
            for (int q0 = 0; q0 < shares; q0 += 4) {
                LoadedRow<float, NQ, TAIL> x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (q0 + j < shares) x[j].load(rows + (size_t)(q0 + j) * f.D, f.D, lane);
                    else x[j].zero();
                }
                Row part;
                part.zero();
#pragma unroll
                for (int j = 0; j < 4; ++j) part.axpy(1.0f, x[j]);
                of_chunk.axpy(1.0f, part);
            }
            total.add(of_chunk);
        }
        dst = a.in_rows + (size_t)b * f.D;
    } else {                                // a word: the chunks that have it
        constexpr int UNROLL = 2 * GroupShape<T, NQ, TAIL>::unroll;
        b -= blocks_in;
        const int word = b >> 6, bit = b & 63;
        const bool last = b == (int)f.V - 1;
        const bool here = (a.any[word] >> bit) & 1ull;
        if (!here && !last) return;
        const u64 upto = (1ull << bit) - 1ull;
        int n = 0;                          // rows ahead of this word's
        for (int wd = threadIdx.x; wd <= word; wd += SUM_THREADS) n += (int)__popcll(wd < word ? a.any[wd] : a.any[wd] & upto);
        n = (int)rd_lane((int)wave_incl_scan((u32)n, lane), WAVE - 1);
        if (lane == 0) ahead[wave] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < SUM_WAVES; ++w) n += ahead[w];
        if (last && threadIdx.x == 0) *a.out_n = n + (here ? 1 : 0);
        if (!here) return;
        if (threadIdx.x == 0) a.out_ids[n] = b;
        const int chunks = U + f.b.n_centers / a.positions;      // numbers in use and the few between them
        for (int c0 = wave * WAVE; c0 < chunks; c0 += SUM_WAVES * WAVE) {
            u64 mk = 0;
            int4 meta = make_int4(0, 0, 0, 0);
            float s_l = 0.f;
            if (c0 + lane < chunks) {
                mk = a.masks[(size_t)word * a.pitch + c0 + lane];
                meta = a.meta[c0 + lane];
            }
            const bool has = (mk >> bit) & 1ull;
            if (has) s_l = f.g[(size_t)meta.y * a.per_center + a.starts[(size_t)word * a.pitch + c0 + lane] + (u32)__popcll(mk & upto)];
            u64 m = __ballot(has);
            while (m) {
                LoadedRow<T, NQ, TAIL> x[UNROLL];
                int at[UNROLL];
#pragma unroll
                for (int j = 0; j < UNROLL; ++j) {
                    at[j] = -1;
                    if (m) {
                        at[j] = (int)__builtin_ctzll(m);
                        m &= m - 1ull;
                        x[j].load((const T *)f.w_in + (size_t)rd_lane(meta.x, at[j]) * f.stride, f.D, lane);
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
        dst = a.out_rows + (size_t)n * f.D;
    }
    Row acc;
    total.round(acc);
    acc.spill(red + wave * ROW, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < f.D; i += SUM_THREADS) dst[i] = sum_waves<SUM_THREADS>(red, ROW, i);
}

template <typename T, int NQ, bool TAIL>
static void launch_group_k(const GroupArgs &a, int what, const AuxWork &aux, hipStream_t st)
{
    const int n = a.f.b.n_centers, V = (int)a.f.V;
    if (what == GROUP_ROWS) {
        hipLaunchKernelGGL(k_group_count, dim3((n + GROUP_RANGE - 1) / GROUP_RANGE), dim3(GROUP_THREADS), 4u * (unsigned)(65 * a.words + 1), st, a);
        const dim3 grid(aux.total + n), blk(BLOCK);
        if (a.f.center_loss) hipLaunchKernelGGL((k_group_rows<T, NQ, TAIL, true>), grid, blk, 0, st, a, aux);
        else hipLaunchKernelGGL((k_group_rows<T, NQ, TAIL, false>), grid, blk, 0, st, a, aux);
        return;
    }
    const int blocks_in = what & GROUP_SUMS_IN ? std::min(n, V) : 0, blocks_out = what & GROUP_SUMS_OUT ? V : 0;
    if (blocks_out) hipLaunchKernelGGL(k_group_any, dim3(a.words), dim3(BLOCK), 0, st, a);
    hipLaunchKernelGGL((k_group_reduce<T, NQ, TAIL>), dim3(aux.total + blocks_in + blocks_out), dim3(SUM_THREADS), 0, st, a, aux, blocks_in);
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
