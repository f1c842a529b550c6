// Gradient application (apply_gradient of Algorithm 1; the "GA" part of Eq. 1 in TensAIR,
// arXiv 2211.10280, Section 2.2) for the own sparse gradient and the K gradients received
// from peers, merged into one pass over the union of their rows:
//     W[r] <- W[r] - lr * (g_0[r] + g_1[r] + ... + g_K[r])
// The paper reports that this step, not the gradient calculation, limits Word2Vec
// scaling (Section 4.3), so it is organised to move every byte once:
//
//   k_apply_index  each source's id list is strictly ascending, so for every 64-row word
//                  of the vocabulary the source's rows in that word are a contiguous run
//                  [start, start + popcount(mask)).  One pass over each id list writes
//                  start[word][k] and mask[word][k]; a wave combines the bits of the ids it
//                  holds with a segmented OR, so only words that straddle two waves need an
//                  (integer, order-independent) atomic.  No sort of the union is needed.
//   k_apply        one wave owns G consecutive vocabulary rows of both tables: a lane holds one
//                  source's (start, mask); rows present in any source are visited in ascending order,
//                  their source rows are streamed (all loads of a row issued together),
//                  summed in source order and applied with one fused multiply-add.  A row
//                  is written by exactly one wave: no write conflicts, fixed order of additions.
//
// Measured and rejected: splitting the update into the rows the own gradient does not touch (which
// could run next to the gradient calculation) and the rows it touches.  The two halves read every
// peer block with holes, lose 20 % of the bandwidth between them, and the gradient calculation is
// itself bound by memory traffic, so nothing was gained by the overlap.

#include <string.h>

#include "apply_kernels.h"
#include "aux_dev.h"
#include "dev_common.h"
#include "kernels.h"

// ---------------------------------------------------------------- index
// (the work itself is in aux_dev.h: inside tensair_step it rides at the front of other launches)
__global__ void __launch_bounds__(BLOCK) k_apply_clear(u64 *m0, u64 *m1, size_t n)
{
    aux_clear_masks(m0, m1, n, (int)blockIdx.x);
}

// grid: (blocks, sources, 2 tables); every wave takes 64 consecutive ids of source k0 + blockIdx.y.
__global__ void __launch_bounds__(BLOCK) k_apply_index(ApplyArgs a, int k0)
{
    aux_index_source(a, k0 + (int)blockIdx.y, (int)blockIdx.z, (int)blockIdx.x, (int)gridDim.x);
}

static int index_blocks_for(const ApplyArgs &a, int k_begin, int k_end)
{
    // enough waves to cover the largest possible id list, grid-strided
    i64 maxcap = 1;
    for (int tb = 0; tb < 2; ++tb)
        for (int k = k_begin; k < k_end; ++k)
            if (a.src[tb][k].ids && a.src[tb][k].capacity > maxcap) maxcap = a.src[tb][k].capacity;
    i64 want = (maxcap + BLOCK * AUX_INDEX_UNROLL - 1) / (BLOCK * AUX_INDEX_UNROLL);
    return (int)(want > 2048 ? 2048 : want);
}

#ifndef AUX_COPY_BLOCKS
#define AUX_COPY_BLOCKS 32
#endif
#ifndef AUX_INDEX_BLOCKS
#define AUX_INDEX_BLOCKS 256
#endif
void tn_aux_none(AuxWork &x) { memset(&x, 0, sizeof(x)); }

static void aux_sum(AuxWork &x)
{
    x.total = x.prep[0].blocks + x.prep[1].blocks + (x.mean_loss ? 1 : 0) + x.clear_blocks + 2 * x.copy_blocks +
              2 * (x.k_end - x.k_begin) * x.index_blocks;
}

void tn_aux_add_prep(AuxWork &x, const PrepPhase &p)
{
    x.prep[x.prep[0].blocks ? 1 : 0] = p;
    aux_sum(x);
}

void tn_aux_add_loss(AuxWork &x, const float *center_loss, int n_centers, float inv_P, float *mean_loss)
{
    x.center_loss = center_loss;
    x.n_centers = n_centers;
    x.inv_P = inv_P;
    x.mean_loss = mean_loss;
    aux_sum(x);
}

void tn_aux_add_clear(AuxWork &x, u64 *mask_in, u64 *mask_out, size_t n)
{
    x.clear_mask[0] = mask_in;
    x.clear_mask[1] = mask_out;
    x.clear_n = n;
    x.clear_blocks = (int)((x.clear_n + BLOCK - 1) / BLOCK);
    aux_sum(x);
}

void tn_aux_add_copy(AuxWork &x, const RowIndexCopy &c, i64 max_rows)
{
    x.copy = c;
    i64 want = (max_rows + 1 + BLOCK - 1) / BLOCK;
    x.copy_blocks = (int)(want > AUX_COPY_BLOCKS ? AUX_COPY_BLOCKS : want);
    aux_sum(x);
}

void tn_aux_add_index(AuxWork &x, const ApplyArgs &a, int k_begin, int k_end)
{
    if (k_end <= k_begin) return;
    x.apply = a;
    x.k_begin = k_begin;
    x.k_end = k_end;
    // few workgroups per id list, each striding over it: riding in front of another kernel's grid, every
    // workgroup that finds nothing to do still delays that kernel's own
    x.index_blocks = index_blocks_for(a, k_begin, k_end);
    if (x.index_blocks > AUX_INDEX_BLOCKS) x.index_blocks = AUX_INDEX_BLOCKS;
    aux_sum(x);
}

void tn_launch_apply_clear(const ApplyArgs &a, hipStream_t st)
{
    const size_t words = (size_t)((a.V + 63) >> 6);
    const size_t n = words * (size_t)a.n_src;
    hipLaunchKernelGGL(k_apply_clear, dim3((unsigned)((n + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, st,
                       a.mask[0], a.mask[1], n);
}

// index of the sources k_begin .. k_end-1 (the masks must have been cleared)
void tn_launch_apply_index(const ApplyArgs &a, int k_begin, int k_end, hipStream_t st)
{
    if (k_end <= k_begin) return;
    const int blocks = index_blocks_for(a, k_begin, k_end);
    hipLaunchKernelGGL(k_apply_index, dim3(blocks, k_end - k_begin, 2), dim3(BLOCK), 0, st, a, k_begin);
}

void tn_launch_apply_update(const ApplyArgs &a, const PrepPhase *rider, const ChainWork *chain, hipStream_t st)
{
    if (chain) tn_launch_apply_update_chaining(a, rider, *chain, st);
    else if (rider) tn_launch_apply_update_riding(a, *rider, st);
    else launch_apply(a, NoRider(), st);
}

// ---------------------------------------------------------------- sum of sparse gradients
// Algorithm 1 keeps the gradients a Model instance has computed and not yet sent in a buffer
// ("gradients += gradient") and broadcasts the buffer every maxGradBuffer steps.  In the sparse form
// that sum lists the union of the rows: a row one source has is taken over, a row several have is
// added in source order (fp32, one rounding per addition).  The same per-word index as for the table
// update tells where every source's rows are; a scan over the popcounts of the united masks gives each
// 64-row word its place in the output, so ids come out ascending without any sort or merge.
#ifndef GRADSUM_G
#define GRADSUM_G 8   // vocabulary rows per wave in the sum of two gradients (4 / 8 / 16 / 32: 0.213 / 0.185 / 0.186 / 0.206 ms)
#endif
#define UNION_WPT (TN_UNION_WORDS / BLOCK)

__device__ __forceinline__ u64 united_mask(const u64 *mask, size_t words, size_t word, int ns)
{
    u64 u = 0;
    for (int k = 0; k < ns; ++k) u |= mask[idx_at((i64)words, k, (i64)word)];
    return u;
}

// block-wide exclusive scan of one int per thread; total = block total
__device__ __forceinline__ int block_scan1(int x, int &total, int *sm)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int incl = (int)wave_incl_scan((u32)x, lane);
    if (lane == WAVE - 1) sm[wave] = incl;
    __syncthreads();
    int off = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < WAVES_PER_BLOCK; ++w) {
        if (w < wave) off += sm[w];
        total += sm[w];
    }
    __syncthreads();
    return off + incl - x;
}

// grid (blocks, 2 tables): rows of the union inside each block of TN_UNION_WORDS words
__global__ void __launch_bounds__(BLOCK) k_union_count(GradSumArgs g)
{
    __shared__ int sm[WAVES_PER_BLOCK];
    const int tb = blockIdx.y, ns = g.a.n_src;
    const size_t words = (size_t)((g.a.V + 63) >> 6);
    const size_t w0 = ((size_t)blockIdx.x * BLOCK + threadIdx.x) * UNION_WPT;
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < UNION_WPT; ++j)
        if (w0 + j < words) cnt += __popcll(united_mask(g.a.mask[tb], words, w0 + j, ns));
    int total;
    block_scan1(cnt, total, sm);
    if (threadIdx.x == 0) g.wblk[tb][blockIdx.x] = (u32)total;
}

// grid (blocks, 2 tables): place of every word in the output; the last block writes the row count
__global__ void __launch_bounds__(BLOCK) k_union_offsets(GradSumArgs g)
{
    __shared__ int sm[WAVES_PER_BLOCK];
    const int tb = blockIdx.y, ns = g.a.n_src;
    const size_t words = (size_t)((g.a.V + 63) >> 6);
    int before = 0;
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += BLOCK) before += (int)g.wblk[tb][j];
    int prefix;
    block_scan1(before, prefix, sm);   // prefix = rows of the union in all earlier blocks
    const size_t w0 = ((size_t)blockIdx.x * BLOCK + threadIdx.x) * UNION_WPT;
    int c[UNION_WPT];
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < UNION_WPT; ++j) {
        c[j] = (w0 + j < words) ? __popcll(united_mask(g.a.mask[tb], words, w0 + j, ns)) : 0;
        cnt += c[j];
    }
    int total;
    int run = prefix + block_scan1(cnt, total, sm);
#pragma unroll
    for (int j = 0; j < UNION_WPT; ++j) {
        if (w0 + j < words) g.wbase[tb][w0 + j] = (u32)run;
        run += c[j];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        i64 U = (i64)prefix + total;
        if (U > g.out_cap[tb]) {
            U = g.out_cap[tb];
            atomicOr(g.a.status, ST_OVERFLOW);
        }
        *g.out_n[tb] = (int)U;
    }
}

// one wave per G consecutive vocabulary rows of both tables, as in k_apply; SWEEP: one group after the other, as there
template <int ITERS, int G, bool SWEEP>
__global__ void __launch_bounds__(BLOCK) k_grad_sum(GradSumArgs g, int nblocks)
{
    const ApplyArgs &a = g.a;
    constexpr int GPW = 64 / G;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int words = (int)((a.V + 63) >> 6);
    const int groups = words * GPW, stride = SWEEP ? nblocks * WAVES_PER_BLOCK : groups;
    int gw = blockIdx.x * WAVES_PER_BLOCK + wave;
    if (gw >= groups) return;
    const int ns = a.n_src;
    const int C4 = a.D >> 2;

    int U = 0;
    u64 rows_ptr = 0;
    u64 mk_next = 0, mk_after = 0;   // index words of the coming group and, in a sweep, of the one after it
    u32 st_next = 0, st_after = 0, base_next = 0, base_after = 0;
    const u64 *masks = nullptr;
    const u32 *starts = nullptr;
    const u32 *bases = g.wbase[lane >> 5];
    {
        const int tb = lane >> 5, k = lane & 31;
        if (k < ns) {
            const ApplySrc &s = a.src[tb][k];
            if (s.ids != nullptr) {
                masks = a.mask[tb] + idx_at(words, k, 0);
                starts = a.start[tb] + idx_at(words, k, 0);
                mk_next = masks[gw / GPW];
                st_next = starts[gw / GPW];
                if (SWEEP && gw + stride < groups) {
                    mk_after = masks[(gw + stride) / GPW];
                    st_after = starts[(gw + stride) / GPW];
                }
                U = *s.n_rows;
                if ((i64)U > s.capacity) U = (int)s.capacity;
                rows_ptr = (u64)s.rows;
            }
        }
    }
    base_next = bases[gw / GPW];
    if (SWEEP && gw + stride < groups) base_after = bases[(gw + stride) / GPW];
    for (;; gw += stride) {
        const int word = gw / GPW, lo = (gw - word * GPW) * G;
        const u64 mk = mk_next;
        const u32 st = st_next, base_l = base_next;
        if (SWEEP) {
            mk_next = mk_after;
            st_next = st_after;
            base_next = base_after;
            if (gw + 2 * (i64)stride < groups) {
                if (masks != nullptr) {
                    mk_after = masks[(gw + 2 * stride) / GPW];
                    st_after = starts[(gw + 2 * stride) / GPW];
                }
                base_after = bases[(gw + 2 * stride) / GPW];
            }
        }
        const i64 row0 = (i64)word * 64;
        u32 u_lo[2], u_hi[2];               // rows of the word that any source has
        half_or((u32)mk, u_lo[0], u_lo[1]);
        half_or((u32)(mk >> 32), u_hi[0], u_hi[1]);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const bool mine = (lane >> 5) == tb;
            const u64 uw = ((u64)u_hi[tb] << 32) | u_lo[tb];
            u64 um = (G == 64) ? uw : ((uw >> lo) & ((1ull << (G & 63)) - 1ull));
            const u32 base = (u32)rd_lane((int)base_l, 32 * tb);
            while (um) {
                const int b = lo + (int)__builtin_ctzll(um);
                um &= um - 1ull;
                const i64 r = row0 + b;
                const i64 dst = (i64)base + __popcll(uw & ((1ull << b) - 1ull));
                if (r >= a.V || dst >= g.out_cap[tb]) break;   // corrupt index or overflow (both flagged)
                const u32 pos = st + (u32)__popcll(mk & ((1ull << b) - 1ull));
                const bool ok = mine && ((mk >> b) & 1ull) && (pos < (u32)U);
                u64 S = __ballot(ok);
                float4 acc[ITERS];
                zero_row<ITERS>(acc);
                while (S) {
                    float4 x[4][ITERS];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (S) {
                            const int k = (int)__builtin_ctzll(S);
                            S &= S - 1ull;
                            const float *src = (const float *)rd_lane64(rows_ptr, k) + (size_t)(u32)rd_lane((int)pos, k) * a.D;
                            load_row_s<float, ITERS>(x[j], src, C4, lane);   // read once: around the caches
                        } else {
                            zero_row<ITERS>(x[j]);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) add_row<ITERS>(acc, x[j]);
                }
                store_row_s<float, ITERS>(g.out_rows[tb] + (size_t)dst * a.D, acc, C4, lane);
                if (lane == 0) g.out_ids[tb][dst] = (int)r;
            }
        }
        if (!SWEEP || gw + stride >= groups) break;
    }
}

// index of the sources and place of every word in the output
void tn_launch_grad_sum_index(const GradSumArgs &g, hipStream_t st)
{
    const ApplyArgs &a = g.a;
    tn_launch_apply_clear(a, st);
    tn_launch_apply_index(a, 0, a.n_src, st);
    const int words = (int)((a.V + 63) >> 6);
    const int sblocks = (words + TN_UNION_WORDS - 1) / TN_UNION_WORDS;
    hipLaunchKernelGGL(k_union_count, dim3(sblocks, 2), dim3(BLOCK), 0, st, g);
    hipLaunchKernelGGL(k_union_offsets, dim3(sblocks, 2), dim3(BLOCK), 0, st, g);
}

template <int G, bool SWEEP>
static void launch_grad_sum(const GradSumArgs &g, hipStream_t st)
{
    const ApplyArgs &a = g.a;
    const int words = (int)((a.V + 63) >> 6);
    const int iters = (a.D / 4 + WAVE - 1) / WAVE;
    const i64 nwaves = (i64)words * (64 / G);
    int nblocks = (int)((nwaves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    if (SWEEP) nblocks = sweep_blocks(nblocks);
    dim3 grid(nblocks), blk(BLOCK);
    switch (iters) {
    case 1: hipLaunchKernelGGL((k_grad_sum<1, G, SWEEP>), grid, blk, 0, st, g, nblocks); break;
    case 2: hipLaunchKernelGGL((k_grad_sum<2, G, SWEEP>), grid, blk, 0, st, g, nblocks); break;
    case 3: hipLaunchKernelGGL((k_grad_sum<3, G, SWEEP>), grid, blk, 0, st, g, nblocks); break;
    default: hipLaunchKernelGGL((k_grad_sum<4, G, SWEEP>), grid, blk, 0, st, g, nblocks); break;
    }
}

// Where few of a large vocabulary's rows are touched a sweep, as for the table update; buffer and message, whole calls,
// sweep in groups of 8 / of 4 / no sweep: 200 000 words, D = 256 36.1 / 31.7 / 34.8 us; 500 000 44.2 / 43.1 / 49.1; a million
// 52.6 / 57.1 / 70.9 and, more touched, 108 / 114 / 126; 2 million 47.2 / 63.7 / 88.6 and 150 / 165 / 190; D = 64 43.8 / 61.9 /
// 83.8 and 86.6 / 101 / 132.
void tn_launch_grad_sum_rows(const GradSumArgs &g, hipStream_t st)
{
    if (!sweep_union(g.a)) launch_grad_sum<GRADSUM_G, false>(g, st);
    else if (g.a.V < 524288) launch_grad_sum<4, true>(g, st);
    else launch_grad_sum<8, true>(g, st);
}
